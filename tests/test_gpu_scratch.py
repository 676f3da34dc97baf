"""The memory that calls take for themselves (stream-ordered, from one pool per
device): what is given back, and when; and what a call leaves behind that found
no memory."""
import os
import subprocess
import sys

import numpy as np
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


def test_failed_call_leaves_no_error_for_the_next(O):
    """A workspace larger than the device is refused, and the next call, with
    one that fits, works (the inputs are as large as the batch says; nothing
    is launched for it)."""
    torch = require_gpu()
    say("[scratch] workspace larger than the device")
    prm = dict(n=1, k=1, N=4096, pbs_level=1, pbs_base_log=8, ks_level=1, ks_base_log=4, msg_bits=4)
    rng = np.random.default_rng(4)
    words = lambda *shape: rng.integers(0, R.P, shape, dtype=np.uint64)
    bsk_std, ksk_std, lut, cts = words(R.bsk_words(prm)), words(R.ksk_words(prm)), words(4096), words(3, 2)
    bsk = R.bsk_prepare(R.to_device(bsk_std), prm)
    ksk = R.ksk_prepare(R.to_device(ksk_std), prm)
    total = torch.cuda.get_device_properties(0).total_memory
    batch = total // (4097 * 8) + 1
    with pytest.raises(R.RosettaError) as e:
        R.pbs_batch(torch.zeros((batch, 2), dtype=torch.int64, device="cuda"), bsk, ksk, R.to_device(lut), prm)
    assert R.STATUS[e.value.status] == "ROSETTA_ERR_NOMEM"
    got = R.to_host(R.pbs_batch(R.to_device(cts), bsk, ksk, R.to_device(lut), prm))
    op = O.Params.make(**{k: v for k, v in prm.items() if k != "k"})
    assert np.array_equal(got, O.pbs(op, cts, bsk_std, ksk_std, lut, O.NTT))


def test_no_room_for_the_expanded_key_runs_the_modular_kernel():
    """With less memory free than the expanded key takes (3.2 GB at the largest
    set), the call gives the words that the allocation-free one does, and the
    same again once there is room."""
    torch = require_gpu()
    prm = dict(n=2048, k=1, N=4096, pbs_level=3, pbs_base_log=14, ks_level=1, ks_base_log=4, msg_bits=4)
    rng = np.random.default_rng(5)
    words = lambda *shape: R.to_device(rng.integers(0, R.P, shape, dtype=np.uint64))
    bsk, ksk = R.bsk_prepare(words(R.bsk_words(prm)), prm), R.ksk_prepare(words(R.ksk_words(prm)), prm)
    lut, cts, want = words(4096), words(3, 2049), R.empty((3, 2049))
    out = R.empty((3, 2049))
    R.pbs_batch_noalloc(cts, bsk, ksk, lut, prm, want)
    ws = R.empty(R.pbs_workspace_bytes(prm, 3) // 8)
    torch.cuda.synchronize()
    torch.cuda.empty_cache()
    R.shutdown()
    held = torch.empty(torch.cuda.mem_get_info()[0] - (1500 << 20), dtype=torch.uint8, device="cuda")
    say(f"[scratch] {torch.cuda.mem_get_info()[0] >> 20} MiB free")
    try:
        assert torch.cuda.mem_get_info()[0] < 3 << 30
        R.pbs_batch_ws(cts, bsk, ksk, lut, prm, ws, out=out)
        torch.cuda.synchronize()
        assert torch.equal(out, want)
    finally:
        del held
        torch.cuda.empty_cache()
    R.pbs_batch_ws(cts, bsk, ksk, lut, prm, ws, out=out)
    torch.cuda.synchronize()
    assert torch.equal(out, want)
