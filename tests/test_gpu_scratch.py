"""The memory that calls take for themselves (stream-ordered, from one pool per
device): what is given back, and when."""
import os
import subprocess
import sys
import time

import pytest

from paper_2609_16915_amd import rosetta as R

from gpu_helpers import require_gpu, say

pytestmark = pytest.mark.gpu
ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

ONLY_KEY_SWITCHES = """
import time

import torch
from paper_2609_16915_amd import rosetta as R
prm = dict(n=1024, k=1, N=2048, pbs_level=3, pbs_base_log=8, ks_level=6, ks_base_log=3, msg_bits=6)
ksk = R.ksk_prepare(torch.zeros(R.ksk_words(prm), dtype=torch.int64, device="cuda"), prm)
big = torch.zeros((14336, 2049), dtype=torch.int64, device="cuda")
out = R.empty((14336, 1025))
R.keyswitch(big[:1].contiguous(), ksk, prm)
torch.cuda.synchronize()
before = torch.cuda.mem_get_info()[0]
for _ in range(8):
    R.keyswitch(big, ksk, prm, out=out)
R.shutdown()  # with the key switches still running
torch.cuda.synchronize()
for _ in range(20):  # the device's count of free memory lags a little
    time.sleep(0.1)
    held = before - torch.cuda.mem_get_info()[0]
    if held < 32 << 20:
        break
print("HELD", held, flush=True)
"""


def test_shutdown_gives_back_what_key_switches_took():
    """In a process of its own, which calls nothing else: the 168 MiB of digits
    are given back although their free is pending when shutdown is called."""
    require_gpu()
    say("[scratch] key switches only")
    r = subprocess.run([sys.executable, "-c", ONLY_KEY_SWITCHES], cwd=ROOT, capture_output=True,
                       text=True, timeout=100)
    assert r.returncode == 0, r.stderr[-2000:]
    held = int(r.stdout.split("HELD")[1])
    assert held < 32 << 20, f"{held >> 20} MiB held after shutdown"


def _held(torch, before, limit):
    """Bytes of device memory taken since `before` (polled down to limit: the
    device's count of free memory lags a little)."""
    for _ in range(20):
        held = before - torch.cuda.mem_get_info()[0]
        if held <= limit:
            break
        time.sleep(0.1)
    return held


@pytest.mark.parametrize("N,streams", [(2048, 1), (4096, 3)])
def test_idle_pool_keeps_little(N, streams):
    """Calls that expand their key to 576 MiB (N = 2048) or 1.1 GiB, waited for:
    at most 256 MiB of that stays taken."""
    torch = require_gpu()
    say(f"[scratch] idle N={N} streams={streams}")
    prm = dict(n=1024, k=1, N=N, pbs_level=3, pbs_base_log=8, ks_level=3, ks_base_log=4, msg_bits=4)
    bsk = R.bsk_prepare(torch.zeros(R.bsk_words(prm), dtype=torch.int64, device="cuda"), prm)
    lut = torch.zeros(N, dtype=torch.int64, device="cuda")
    lwe = torch.zeros((2, 1025), dtype=torch.int64, device="cuda")
    jobs = [(torch.cuda.Stream(), R.empty((2, N + 1))) for _ in range(streams)]
    torch.cuda.synchronize()

    def calls():
        for st, out in jobs:
            R.blind_rotate_extract(lwe, bsk, lut, prm, out=out, stream=st)
        torch.cuda.synchronize()

    calls()
    R.shutdown()
    torch.cuda.synchronize()
    time.sleep(0.3)
    before = torch.cuda.mem_get_info()[0]
    calls()
    limit = (256 << 20) + (32 << 20)
    assert _held(torch, before, limit) <= limit
