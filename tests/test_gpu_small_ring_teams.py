"""Blind rotation of few ciphertexts on small rings (one team of waves per
gadget digit) against the kernel for many ciphertexts, which the same
ciphertexts reach inside a larger batch, and against the oracle, bit for bit:
every gadget length, the widest digits, 32- and 64-bit digit registers, both
sides of the rule that chooses (two ciphertexts per CU)."""
import numpy as np
import pytest

from paper_2609_16915_amd import rosetta as R
from test_gpu_fft_blind_rotate import _params, _words

from gpu_helpers import require_gpu, say

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("N", [256, 512, 1024])
@pytest.mark.parametrize("l,beta", [(1, 1), (1, 15), (1, 30), (2, 8), (2, 15), (2, 16), (3, 10), (3, 11), (4, 7),
                                    (4, 15)])
def test_teams_equal_the_large_batch_kernel(O, N, l, beta):
    torch = require_gpu()
    cus = torch.cuda.get_device_properties(0).multi_processor_count
    prm = _params(N, l, beta, 7)
    rng = np.random.default_rng(N + 100 * l + beta)
    bsk_std = _words(rng, R.bsk_words(prm))
    bsk = R.bsk_prepare(R.to_device(bsk_std), prm)
    op = O.Params.make(**{k: v for k, v in prm.items() if k != "k"})
    many = 2 * cus + 1
    say(f"[teams] N={N} l={l} beta={beta}")
    cts = _words(rng, many, prm["n"] + 1)
    cts[0, :3] = 0                      # steps that rotate by nothing
    d_in = R.to_device(cts)
    lut = R.to_device(_words(rng, N))
    tp_std = _words(rng, many, 2 * N)
    tp = R.to_device(tp_std)
    wide = R.to_host(R.blind_rotate_extract(d_in, bsk, lut, prm))
    wide_glwe = R.to_host(R.blind_rotate_glwe(d_in, bsk, tp, prm, group=1))
    want = O.blind_rotate_glwe_batch(op, cts[:2], bsk_std, tp_std[:2], O.NTT)
    assert np.array_equal(wide_glwe[:2], want.reshape(wide_glwe[:2].shape))
    for batch in (1, 2 * cus):
        few = d_in[:batch].contiguous()
        assert np.array_equal(R.to_host(R.blind_rotate_extract(few, bsk, lut, prm)), wide[:batch])
        got = R.to_host(R.blind_rotate_glwe(few, bsk, tp[:batch].contiguous(), prm, group=1))
        assert np.array_equal(got, wide_glwe[:batch])
