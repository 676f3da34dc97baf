"""Work that programs give this library, as cases that can be timed and compared.

Every case is one call, or one short chain of calls, through the Python
binding: whole bootstraps at the repository's parameter sets from one
ciphertext to the FFN width of LLaMA-3-8B, the encrypted lookup (Algorithm 1)
and its steps, the key switch, and the ring products underneath.  Sizes are
those of paper_2609_16915_amd/workloads.py and bench.py, with odd batches
among them.

Key words, ciphertext words and GLWE test polynomials are uniform below the
modulus: encryptions are indistinguishable from that, and no step's work or
branch depends on the words (the modulus-switched rotation amounts are
uniform in earnest too).  Tables are the workloads' own.
"""
import math

import torch

from paper_2609_16915_amd import rosetta as R
from paper_2609_16915_amd import workloads as W

TRACE_LEVEL, TRACE_BASE_LOG = 4, 12  # bench.py's trace
LOOKUP = dict(nseg=4, margin=32, sx=40, sv=18, sc=57, refine=5)  # bench.py's lookup


def listed():
    return [
        # the smallest call: the eight ciphertexts of the tiny parameter set
        dict(name="pbs_tiny_8", kind="pbs", set="tiny", n=64, batch=8),
        # latency of a single bootstrap at the headline parameters
        dict(name="pbs_one", kind="pbs", set="llama3_8b_silu", n=1024, batch=1),
        # the reciprocals of the 32 softmax row sums of one decoded token
        dict(name="pbs_softmax_recip_32", kind="pbs", set="llama3_8b_softmax_recip", n=1024,
             batch=32),
        # GELU over GPT-2's FFN width, one decoded token
        dict(name="pbs_gpt2_gelu_3072", kind="pbs", set="gpt2_gelu", n=742, batch=3072),
        # the headline: SiLU over LLaMA-3-8B's FFN width, one decoded token
        dict(name="pbs_llama_silu_14336", kind="pbs", set="llama3_8b_silu", n=1024, batch=14336),
        # softmax exponentials of one head's 2048-token row
        dict(name="pbs_softmax_exp_2048", kind="pbs", set="llama3_8b_softmax_exp", n=1024,
             batch=2048),
        # lookup select on an odd batch: blind rotation of encrypted test
        # polynomials, then the trace (Steps 2-3 of Algorithm 1)
        dict(name="select_1001", kind="select", set="llama3_8b_silu", n=1024, batch=1001,
             group=1),
        # the key switch of a whole FFN layer on its own
        dict(name="keyswitch_14336", kind="keyswitch", set="llama3_8b_silu", n=1024,
             batch=14336),
        # the RLWE traces of a whole FFN layer
        dict(name="trace_14336", kind="trace", set="llama3_8b_lookup", n=1024, batch=14336),
        # Algorithm 1 (Steps 1-3) for a small batch of inputs
        dict(name="lookup_eval_64", kind="lookup", set="llama3_8b_lookup", n=1024, batch=64),
        # construct and recombine: four segment lines per input (Step 3)
        dict(name="construct_4096", kind="construct", set="llama3_8b_lookup", n=1024,
             batch=4096, count=4),
        # plain negacyclic products, an odd count
        dict(name="poly_mul_5001", kind="poly_mul", set="llama3_8b_silu", n=1024, batch=5001),
    ]


SETS = ("tiny", "gpt2_gelu", "tinyllama_silu", "llama3_8b_silu", "llama3_8b_softmax_exp",
        "llama3_8b_lookup")
RINGS = ("gpt2_gelu", "llama3_8b_silu", "llama3_8b_softmax_exp", "llama3_8b_lookup")


def _spread(rng, lo, hi):
    """An integer of [lo, hi], uniform in its logarithm."""
    return max(lo, min(hi, int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))))


def draw(rng):
    kind = rng.choice(["pbs"] * 5 + ["select", "select", "keyswitch", "trace", "lookup",
                                     "construct", "poly_mul"])
    if kind == "pbs":
        name = rng.choice(SETS)
    elif kind == "lookup":
        name = "llama3_8b_lookup"
    else:
        name = rng.choice(RINGS)
    w = W.get(name)
    # the set's own LWE dimension, or another of the same range
    n = w.n if name == "tiny" or rng.random() < 0.5 else rng.randint(500, 1024)
    case = dict(kind=kind, set=name, n=n)
    if kind == "select":
        case["group"] = rng.choice([1, 1, 4])
    if kind == "construct":
        case["count"] = rng.choice([1, 2, 4, 8])
    top = dict(pbs=14336, select=4096, keyswitch=16384, trace=16384, lookup=512,
               construct=4096, poly_mul=16384)[kind]
    # no more than half the headline's blind rotations
    head = W.get(W.HEADLINE)
    limit = 0.5 * head.br_modmul_per_pbs() * head.batch
    one = _rotations(dict(case, batch=1)) * w.br_modmul_per_pbs()
    if one:
        top = min(top, int(limit / one))
    case["batch"] = _spread(rng, 1, max(1, top))
    return case


def _rotations(case):
    """Blind rotations of one pass."""
    b = case["batch"]
    if case["kind"] == "pbs":
        return b
    if case["kind"] == "select":
        return b * case["group"]
    if case["kind"] == "lookup":
        return b * (3 * (LOOKUP["nseg"] - 1) + LOOKUP["nseg"] + 2)
    return 0


def _params(case):
    return dict(W.get(case["set"]).params(), n=case["n"])


def _uniform(gen, *shape):
    """Words uniform below the modulus, as int64 tensors (raw 64-bit words)."""
    x = torch.randint(-2 ** 63, 2 ** 63 - 1, shape, dtype=torch.int64, device="cuda",
                      generator=gen)
    # words in [p, 2^64) are -2^32 + 1 .. -1 as signed integers
    return torch.where((x < 0) & (x > -2 ** 32), x + 2 ** 40, x)


def prepare(case, seed):
    kind, b = case["kind"], case["batch"]
    w, prm = W.get(case["set"]), _params(case)
    p = R.Params.from_dict(prm)
    n, N = p.n, p.N
    gen = torch.Generator(device="cuda")
    gen.manual_seed(seed)
    s = dict(kind=kind, prm=p, case=case)
    if kind in ("pbs", "select", "lookup"):
        s["bsk"] = R.bsk_prepare(_uniform(gen, R.bsk_words(p)), p)
    if kind in ("pbs", "keyswitch", "lookup"):
        s["ksk"] = R.ksk_prepare(_uniform(gen, R.ksk_words(p)), p)
    if kind in ("select", "trace", "lookup"):
        s["autk"] = R.autk_prepare(_uniform(gen, R.autk_words(p, TRACE_LEVEL)), p, TRACE_LEVEL)
    if kind == "pbs":
        s["lwe"] = _uniform(gen, b, n + 1)
        s["lut"] = R.to_device(R.lut_build(p, w.table()))
    elif kind == "select":
        s["lwe"] = _uniform(gen, b, n + 1)
        s["tp"] = _uniform(gen, b * case["group"], 2 * N)
    elif kind == "keyswitch":
        s["big"] = _uniform(gen, b, N + 1)
    elif kind == "trace":
        s["glwe"] = _uniform(gen, b, 2 * N)
    elif kind == "construct":
        s["glwe"] = _uniform(gen, b, 2 * N)
        s["pa"] = R.plain_prepare(_uniform(gen, case["count"], N), N)
        s["pb"] = _uniform(gen, case["count"], N)
        s["exps"] = [i * (N // case["count"]) for i in range(case["count"])]
    elif kind == "poly_mul":
        s["a"], s["b"] = _uniform(gen, b, N), _uniform(gen, b, N)
    elif kind == "lookup":
        L = LOOKUP
        lp = R.LookupParams(nseg=L["nseg"], nbr=N - 2 * L["margin"], margin=L["margin"],
                            x_scale_log=L["sx"],
                            coef_scale_log=63 - int(math.log2(N)) - L["sx"],
                            val_scale_log=L["sv"], cmp_scale_log=L["sc"],
                            trace_level=TRACE_LEVEL, trace_base_log=TRACE_BASE_LOG,
                            cmp_refine_log=L["refine"])
        tau = R.seglut_boundaries(-20.0, 20.0, lp.nseg, "uniform")
        plain, s["consts"] = R.lookup_encode(p, lp, tau, *R.seglut_build("silu", tau, lp.nbr))
        s["plain"] = R.lookup_prepare(R.to_device(plain), p, lp)
        s["x_rlwe"], s["x_cmp"] = _uniform(gen, b, 2 * N), _uniform(gen, b, n + 1)
        s["lp"] = lp
        s["ws"] = R.empty(R.lookup_workspace_bytes(p, lp, b) // 8)
    return s


def run(s):
    kind, p, case = s["kind"], s["prm"], s["case"]
    if kind == "pbs":
        out = R.pbs_batch(s["lwe"], s["bsk"], s["ksk"], s["lut"], p)
    elif kind == "select":
        acc = R.blind_rotate_glwe(s["lwe"], s["bsk"], s["tp"], p, group=case["group"])
        out = R.trace(acc, s["autk"], p, TRACE_LEVEL, TRACE_BASE_LOG)
    elif kind == "keyswitch":
        out = R.keyswitch(s["big"], s["ksk"], p)
    elif kind == "trace":
        out = R.trace(s["glwe"], s["autk"], p, TRACE_LEVEL, TRACE_BASE_LOG)
    elif kind == "construct":
        prods = R.glwe_mul_plain(s["glwe"], s["pa"], s["pb"], p.N)
        out = R.glwe_recombine(prods, case["count"], p.N, exps=s["exps"])
    elif kind == "poly_mul":
        out = R.poly_mul(s["a"], s["b"], p.N)
    else:
        out = R.lookup_eval(s["x_rlwe"], s["x_cmp"], s["bsk"], s["ksk"], s["autk"], s["plain"],
                            s["consts"], p, s["lp"], workspace=s["ws"])
    return out.view(torch.int64)


def work(case):
    """Bytes: inputs and prepared keys read once, outputs written once.
    flops: two (a product and a sum) per modular multiplication of the
    radix-2 transforms and pointwise products, and two per digit
    multiply-add of a key switch."""
    kind, b = case["kind"], case["batch"]
    p = R.Params.from_dict(_params(case))
    n, N, l = p.n, p.N, p.pbs_level
    lg = int(math.log2(N))
    ntt = N // 2 * lg
    bsk, ksk, autk = 4 * n * l * N, R.ksk_device_words(p), lg * TRACE_LEVEL * 2 * N
    br = n * ((2 * l + 2) * ntt + 4 * l * N)
    ks = N * p.ks_level * (n + 1)
    tr = 2 * N + lg * ((TRACE_LEVEL + 2) * ntt + 2 * TRACE_LEVEL * N)
    if kind == "pbs":
        words, mm = bsk + ksk + N + 2 * b * (n + 1), b * (br + ks)
    elif kind == "select":
        g = b * case["group"]
        words, mm = bsk + autk + b * (n + 1) + 4 * g * N, g * (br + tr)
    elif kind == "keyswitch":
        words, mm = ksk + b * (N + n + 2), b * ks
    elif kind == "trace":
        words, mm = autk + 4 * b * N, b * tr
    elif kind == "construct":
        c = case["count"]
        words, mm = 2 * c * N + 4 * b * N, b * (2 * ntt + 2 * c * (ntt + N))
    elif kind == "poly_mul":
        words, mm = 3 * b * N, b * (3 * ntt + N)
    else:
        ns = LOOKUP["nseg"]
        rot, swi, trc, prd = 3 * (ns - 1) + ns + 2, 4 * (ns - 1) + 1, ns + 1, ns + 2
        words = bsk + ksk + autk + (4 + 2 * ns) * N + b * (4 * N + n + 1)
        mm = b * (rot * br + swi * ks + trc * tr + prd * (4 * ntt + 2 * N))
    return {"bytes": 8 * words, "flops": 2 * mm}


def tolerance(case):
    return "exact"  # residues modulo p: one word is right


def exact(case, seed):
    return None  # whole words, compared word for word
