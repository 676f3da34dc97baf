"""The key switch's three matrix-core kernels give the same words: batches
small enough for the split contraction, batches whose digits are made once
(across row-block and scratch-cut edges), and the kernel that needs no
scratch (a captured call, and the batches that are better off with it), each
also against the oracle on a few rows.  Which kernel a batch takes is asked of
the rule itself (csrc/internal.hpp, compiled for the host)."""
import numpy as np
import pytest

from paper_2609_16915_amd import rosetta as R
from test_dispatch_cpu import DIGITS, MFMA, SPLIT, build_rule

from gpu_helpers import require_gpu, say

pytestmark = pytest.mark.gpu
P = R.P
EDGES = np.array([0, 1, P - 1, (P - 1) // 2, (P + 1) // 2, 1 << 63, (1 << 63) - 1, P - (1 << 45)],
                 dtype=np.uint64)


@pytest.fixture(scope="module")
def rule(tmp_path_factory):
    return build_rule(tmp_path_factory.mktemp("dispatch"))


def _cus(torch):
    return torch.cuda.get_device_properties(0).multi_processor_count


def _setup(n, N, level, base, seed):
    prm = dict(n=n, k=1, N=N, pbs_level=1, pbs_base_log=8, ks_level=level, ks_base_log=base, msg_bits=4)
    rng = np.random.default_rng(seed)
    ksk = rng.integers(0, P, R.ksk_words(prm), dtype=np.uint64)
    ksk[rng.integers(0, ksk.size, 4096)] = EDGES[rng.integers(0, len(EDGES), 4096)]
    return prm, rng, ksk, R.ksk_prepare(R.to_device(ksk), prm)


@pytest.mark.parametrize("n,N,level,base,large", [
    (1024, 2048, 6, 3, DIGITS), (31, 256, 3, 4, DIGITS), (32, 4096, 8, 2, DIGITS), (742, 512, 1, 7, DIGITS),
    (63, 1024, 5, 3, DIGITS), (64, 512, 3, 4, DIGITS), (15, 256, 1, 4, MFMA), (2047, 256, 1, 4, MFMA)])
def test_batches_across_the_kernels(O, rule, n, N, level, base, large):
    torch = require_gpu()
    cus = _cus(torch)
    route = lambda b: rule([("ks", n, N, level, base, b, cus)])[0]
    prm, rng, ksk, dev = _setup(n, N, level, base, n + N)
    split = 16 * (cus // ((n + 32) // 32))       # the largest batch that is split
    edge = (split + 256) // 256 * 256            # a whole number of 256-row blocks past it
    rows = edge + 300
    big = rng.integers(0, P, (rows, N + 1), dtype=np.uint64)
    big[rng.random(big.shape) < 0.05] = EDGES[1]
    big[:40:3] = EDGES[rng.integers(0, len(EDGES), (14, N + 1))]
    d = R.to_device(big)
    say(f"[ks split] n={n} N={N} {level}x{base} split up to {split}, rows {rows}")
    # pieces of up to 16 rows run the split kernel
    want = np.concatenate([R.to_host(R.keyswitch(d[i:i + 16].contiguous(), dev, prm))
                           for i in range(0, rows, 16)])
    op = O.Params.make(**{k: v for k, v in prm.items() if k != "k"})
    pick = [0, 15, 16, split, rows - 1]
    for q in pick:
        assert np.array_equal(want[q], O.keyswitch(op, big[q], ksk))
    for batch, kernel in [(1, SPLIT), (15, SPLIT), (17, SPLIT), (split, SPLIT), (split + 1, large),
                          (edge - 1, large), (edge, large), (edge + 1, large), (rows, large)]:
        assert route(batch) == kernel, batch
        got = R.to_host(R.keyswitch(d[:batch].contiguous(), dev, prm))
        assert np.array_equal(got, want[:batch]), batch
    # without scratch: a captured call past the split, replayed on new inputs too
    held = edge + 1
    src = d[:held].clone()
    out = R.empty((held, n + 1))
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        R.keyswitch(src, dev, prm, out=out)
    for lo in (0, 200, 100):
        src.copy_(d[lo:lo + held])
        graph.replay()
        torch.cuda.synchronize()
        assert np.array_equal(R.to_host(out), want[lo:lo + held])


def test_batch_beyond_one_scratch_cut(rule):
    """At N = 4096, 8 levels a cut is 16384 rows; rows on both sides of it."""
    torch = require_gpu()
    prm, rng, _, dev = _setup(40, 4096, 8, 2, 5)
    batch = 16384 + 300
    assert rule([("ks", 40, 4096, 8, 2, batch, _cus(torch))])[0] == DIGITS
    d = R.to_device(rng.integers(0, P, (batch, 4097), dtype=np.uint64))
    say("[ks split] cut")
    got = R.to_host(R.keyswitch(d, dev, prm))
    for lo in (0, 16384 - 16, 16384, batch - 16):
        assert np.array_equal(got[lo:lo + 16],
                              R.to_host(R.keyswitch(d[lo:lo + 16].contiguous(), dev, prm)))
