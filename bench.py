#!/usr/bin/env python3
"""Throughput of batched TFHE programmable bootstrapping on one MI355X.

One step = one PBS of the whole batch (modulus switch, blind rotation,
sample extraction, key switching) with inputs and prepared keys resident in
device memory.  Default workload: the LLaMA-3-8B FFN SiLU layer of one
decoded token, n = 1024, N = 2048, l = 3 x 8 bits, batch 14336.

Prints one JSON line.  The timed region is bracketed by device
synchronisations; per-kernel durations come from HIP events recorded on the
stream the kernels are launched on.  A step calls the two entry points that
make up rosetta_pbs_batch (blind rotation + extraction into a workspace,
then key switching) so that the blind-rotation kernel can be timed on its
own for the roofline.
"""
from __future__ import annotations

import argparse
import json
import math
import os
import sys
import time

import numpy as np

ROOT = os.path.dirname(os.path.abspath(__file__))
sys.path.insert(0, ROOT)

# MI355X peaks.  The VALU issues 64 lanes of a full-rate 32-bit instruction
# per clock per CU (4 SIMDs x 16 lanes): 256 CUs x 64 x 2.4 GHz = 39.3e12
# lane-ops/s.  The library's Goldilocks multiplication on the device is 17
# full-rate VALU instructions on gfx950: the 128-bit product from 4
# v_mad_u64_u32 and 4 add-with-carry, the reduction from 2 subtractions with
# borrow, a conditional p (select + 2), one v_mad_u64_u32 folding the 2^64
# limb with its carry-out, a compare, a select and a 64-bit add.  That
# bounds its rate at 39.3e12 / 17 = 2.31e12 modmul/s; the 4 product
# multiply-adds alone bound any 64x64-bit modular product built this way at
# 39.3e12 / 4 = 9.8e12 modmul/s.
HBM_PEAK_GBS = 8000.0
CU, CLOCK_HZ, LANES = 256, 2.4e9, 64
MODMUL_VALU_OPS = 17
MODMUL_PEAK_T = CU * CLOCK_HZ * LANES / MODMUL_VALU_OPS / 1e12   # Tmodmul/s
MULTIPLIER_BOUND_T = CU * CLOCK_HZ * LANES / 4 / 1e12
# Double precision: one fused multiply-add per lane and clock, as any other
# full-rate instruction: 78.6 TFLOP/s.
FP64_PEAK_T = 2 * CU * CLOCK_HZ * LANES / 1e12
INT8_PEAK_P = 5.0   # MI355X dense int8 matrix-core peak, POP/s (no sparsity)
PMC_PROFILE = os.path.join(ROOT, "profiles", "k_blind_rotate_fft_llama3_8b_silu_pmc.md")
KERNEL_SOURCES = ["gl.hpp", "ntt.hpp", "fft.hpp", "exact_fft.hip"]


def kernel_source_digest() -> str:
    """sha256 of the sources of the headline's blind-rotation kernel (gl.hpp,
    ntt.hpp, fft.hpp, exact_fft.hip in that order) with comments and whitespace removed, so that
    it changes with the code and not with its prose."""
    import hashlib
    import re
    h = hashlib.sha256()
    for f in KERNEL_SOURCES:
        with open(os.path.join(ROOT, "paper_2609_16915_amd", "csrc", f)) as fh:
            text = fh.read()
        text = re.sub(r"/\*.*?\*/", " ", text, flags=re.S)
        text = re.sub(r"//[^\n]*", " ", text)
        h.update(re.sub(r"\s+", "", text).encode())
    return h.hexdigest()


def measured_traffic(workload: str, batch: int):
    """Calibrated HBM bytes per blind-rotation launch from the committed
    counter profile, or None unless that profile describes the current
    kernel code and this workload."""
    import re
    from paper_2609_16915_amd import workloads as W
    if workload != W.HEADLINE or batch != W.get(W.HEADLINE).batch:
        return None
    try:
        text = open(PMC_PROFILE).read()
    except OSError:
        return None
    m_sha = re.search(r"kernel_code_sha256: ([0-9a-f]{64})", text)
    m_tb = re.search(r"traffic_bytes_per_launch: ([0-9.eE+]+)", text)
    if not m_sha or not m_tb or m_sha.group(1) != kernel_source_digest():
        return None
    return float(m_tb.group(1))


def _pieces(N: int, rows: int, base_log: int) -> int:
    """fft_pieces_for in csrc/internal.hpp."""
    if N not in (2048, 4096):
        return 0

    def holds(bits):
        e = base_log + bits - 2
        return e < 40 and rows * N * 160 << e <= 1 << 51

    return 3 if holds(22) else 4 if holds(16) else 0


def key_pieces(N: int, level: int, base_log: int) -> int:
    """Pieces the key is cut into for the blind rotation's double-precision
    transforms (the rule of fft_pieces in csrc/internal.hpp), 0 where the
    modular ones run."""
    if level > 3:
        return 0
    pieces = _pieces(N, 2 * level, base_log)
    return 4 if pieces == 3 and level * base_log > 30 else pieces


def trace_pieces(N: int, level: int, base_log: int, batch: int) -> int:
    """The same for the trace (trace_pieces in csrc/internal.hpp)."""
    pieces = _pieces(N, level, base_log)
    if level == 1 and pieces == 4 and (batch > 2 * CU if N == 2048 else batch <= CU):
        return 0
    return pieces


def keyswitch_kernel(n: int, N: int, level: int, base_log: int, batch: int) -> str:
    """The kernel that switches a batch (ks_route in csrc/internal.hpp)."""
    if not (1 <= base_log <= 7 and level * base_log <= 30 and N % 32 == 0
            and N * level * (1 << (base_log - 1)) * 128 < (1 << 31)):
        return "k_keyswitch"
    cols, K, rows = (n + 32) // 32, N * level, -(-batch // 128)
    if -(-batch // 16) * cols <= CU:
        return "k_keyswitch_small"
    if ((cols <= 2 and 16 * rows > (5 if K <= 1024 else 7 if K <= 2048 else 10) * CU)
            or (cols == 3 and K <= 1024 and 16 * rows * cols > 26 * CU and rows * cols <= 2 * CU)
            or (K == 256 and (cols <= 3 or 2 * rows * cols <= 3 * CU))
            or (N == 256 and level == 2 and 2 * rows * cols <= CU)):
        return "k_keyswitch_mfma"
    return "k_keyswitch_gemm"


def fft_flops(N: int, log_bfly: int, forward: int, inverse: int, products: int) -> int:
    """Double-precision operations (a fused multiply-add is two) of complex
    transforms of N/2 points, six multiply-adds per butterfly, and of complex
    products summed up, four per point."""
    C = N // 2
    return 2 * (6 * (C // 2) * log_bfly * (forward + inverse) + 4 * C * products)


def modmul_probe(stream, reps: int = 5) -> float:
    """Empirical product roofline (Tmodmul/s): the library's own modular
    multiplication in 8 independent register-resident chains per thread,
    12 workgroups of 256 threads per CU, median over `reps` launches timed
    with HIP events on the launch stream."""
    import torch
    from paper_2609_16915_amd import rosetta as R
    threads, iters = CU * 12 * 256, 2048
    out = R.empty(threads)
    R.modmul_chain(7, threads, iters, out=out, stream=stream)
    ms = []
    for _ in range(reps):
        a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
        a.record(stream)
        R.modmul_chain(7, threads, iters, out=out, stream=stream)
        b.record(stream)
        b.synchronize()
        ms.append(a.elapsed_time(b))
    return threads * 8 * iters / (float(np.median(ms)) * 1e-3) / 1e12


def log(*a):
    print(*a, file=sys.stderr, flush=True)


def cpu_model() -> str:
    """The host CPU's model name (/proc/cpuinfo, as lscpu reports it)."""
    try:
        with open("/proc/cpuinfo") as fh:
            for line in fh:
                if line.startswith("model name"):
                    return line.split(":", 1)[1].strip()
    except OSError:
        pass
    import platform
    return platform.processor() or "unknown"


def host_threads():
    """(CPUs this process may run on, threads the baseline uses).  The
    baseline takes every CPU of the process's affinity mask, unless
    OMP_NUM_THREADS sets the host share explicitly (as the GPU hosts do:
    16 host threads per GPU)."""
    visible = len(os.sched_getaffinity(0))
    env = os.environ.get("OMP_NUM_THREADS", "")
    use = min(visible, int(env)) if env.isdigit() and int(env) > 0 else visible
    return visible, use


def cpu_baseline(w, keys, cts, v, seconds_target: float):
    """The oracle (tier 2: textbook radix-2 transforms, OpenMP over
    ciphertexts) timed on the host: its once-per-key transform of the
    bootstrapping key on its own, one ciphertext on one thread, then a
    bounded sample of the batch on every thread of the host share."""
    from oracle import oracle as O
    op = O.Params.make(**{k: x for k, x in w.params().items() if k != "k"})
    visible, threads = host_threads()
    t0 = time.perf_counter()
    fbsk = O.bsk_transform(op, keys["bsk"], threads)
    t_key = time.perf_counter() - t0
    t0 = time.perf_counter()
    O.pbs_prepared(op, cts[:1], fbsk, keys["ksk"], v, 1)
    t_one = time.perf_counter() - t0
    rounds = max(1, int(round(seconds_target / max(t_one, 1e-6))))
    sample = min(rounds * threads, cts.shape[0])
    t0 = time.perf_counter()
    O.pbs_prepared(op, cts[:sample], fbsk, keys["ksk"], v, threads)
    dt = time.perf_counter() - t0
    return {"value": sample / dt, "unit": "PBS/s", "cores": threads, "cores_visible": visible,
            "cpu_model": cpu_model(), "kind": "oracle",
            "single_thread_s_per_pbs": round(t_one, 4), "key_transform_s": round(t_key, 3),
            "sample": f"{sample} of the {w.batch} ciphertexts of {w.name} (first {sample}), "
                      f"tier-2 transform oracle on {threads} OpenMP threads, {dt:.1f} s wall; "
                      f"the once-per-key transform of the bootstrapping key "
                      f"({t_key:.2f} s on {threads} threads) is timed apart and not in the rate"}


TRACE_LEVEL, TRACE_BASE_LOG = 4, 12


def lookup_select(R, W, w, p, keys, d_in, bsk, stream, steps):
    """Select step of the lookup protocol over the batch: blind rotation of
    one GLWE test-polynomial ciphertext per input, then the RLWE trace.
    Ciphertext test polynomials are uniform (the work is data-oblivious);
    the automorphism key comes from the library's host helper."""
    import torch
    rng = np.random.default_rng(w.data_seed + 1)
    P = 0xFFFFFFFF00000001
    tp = R.to_device(rng.integers(0, P, (w.batch, 2 * w.N), dtype=np.uint64))
    autk = R.autk_prepare(R.to_device(R.autk_keygen(w.key_seed + 1, p, TRACE_LEVEL, TRACE_BASE_LOG,
                                                    w.sigma_glwe, keys["glwe_key"])),
                          p, TRACE_LEVEL)
    acc = R.empty((w.batch, 2 * w.N))
    out = R.empty((w.batch, 2 * w.N))

    def run(evs=None):
        if evs:
            evs[0].record(stream)
        R.blind_rotate_glwe(d_in, bsk, tp, p, out=acc)
        if evs:
            evs[1].record(stream)
        R.trace(acc, autk, p, TRACE_LEVEL, TRACE_BASE_LOG, out=out)
        if evs:
            evs[2].record(stream)

    run()
    torch.cuda.synchronize()
    ev = [[torch.cuda.Event(enable_timing=True) for _ in range(3)] for _ in range(steps)]
    t0 = time.perf_counter()
    for e in ev:
        run(e)
    torch.cuda.synchronize()
    wall = (time.perf_counter() - t0) / steps
    br_ms = float(np.mean([a.elapsed_time(b) for a, b, _ in ev]))
    tr_ms = float(np.mean([b.elapsed_time(c) for _, b, c in ev]))
    rounds, pieces = int(math.log2(w.N)), trace_pieces(w.N, TRACE_LEVEL, TRACE_BASE_LOG, w.batch)
    if pieces:
        # log2 N rounds of TRACE_LEVEL forward and 2 inverse transforms per piece
        tr_ops = w.batch * rounds * fft_flops(w.N, rounds - 1, TRACE_LEVEL, 2 * pieces,
                                              2 * pieces * TRACE_LEVEL)
        roofline = {"bound": "alu", "kernel": "k_trace_fft", "dtype": "f64", "key_pieces": pieces}
        peak, unit, count = FP64_PEAK_T, "TFLOP/s", "per_launch_flops"
    else:
        tr_ops = w.batch * w.trace_modmul(TRACE_LEVEL)
        roofline = {"bound": "alu", "kernel": "k_trace"}
        peak, unit, count = MODMUL_PEAK_T, "Tmodmul/s", "per_launch_modmul"
    tr_t = tr_ops / (tr_ms * 1e-3) / 1e12
    roofline.update({"achieved": round(tr_t, 4), "peak": round(peak, 4), "unit": unit,
                     "frac": round(tr_t / peak, 4), count: tr_ops, "launch_ms": round(tr_ms, 3)})
    return {"batch": w.batch, "trace_level": TRACE_LEVEL, "trace_base_log": TRACE_BASE_LOG,
            "selects_per_s": round(w.batch / wall, 2), "ms_per_step": round(wall * 1e3, 3),
            "kernels_ms": {"blind_rotate_glwe": round(br_ms, 3), "trace": round(tr_ms, 3)},
            "roofline_trace": roofline}


def lookup_protocol(R, W, stream, steps, batch):
    """The lookup pipeline of Algorithm 1 (Steps 1-3) for SiLU on [-20, 20]
    with 4 uniform segments, at the lookup key set (n = 1024, N = 2048,
    14-bit gadget digits, 8 x 2-bit key switch), a 5-bit refined
    comparison and margins of 32: inputs x ~ N(0, 1) (the FFN activations)
    encrypted as [[x]]_RLWE and [[x]]_cmp with the library's host helpers;
    timed on the device; a sample of outputs is decrypted and compared with
    the cleartext segmented LUT."""
    import torch
    w = W.get("llama3_8b_lookup")
    p = R.Params.from_dict(w.params())
    keys = R.keygen(w.key_seed, p, w.sigma_lwe, w.sigma_glwe)
    bsk = R.bsk_prepare(R.to_device(keys["bsk"]), p)
    ksk = R.ksk_prepare(R.to_device(keys["ksk"]), p)
    sx, sv, sc, margin, nseg, refine = 40, 18, 57, 32, 4, 5
    sp = 63 - int(math.log2(w.N)) - sx
    lp = R.LookupParams(nseg=nseg, nbr=w.N - 2 * margin, margin=margin, x_scale_log=sx,
                        coef_scale_log=sp, val_scale_log=sv, cmp_scale_log=sc,
                        trace_level=TRACE_LEVEL, trace_base_log=TRACE_BASE_LOG,
                        cmp_refine_log=refine)
    tau = R.seglut_boundaries(-20.0, 20.0, nseg, "uniform")
    a, b = R.seglut_build("silu", tau, lp.nbr)
    plain, consts = R.lookup_encode(p, lp, tau, a, b)
    prep = R.lookup_prepare(R.to_device(plain), p, lp)
    autk = R.autk_prepare(R.to_device(R.autk_keygen(w.key_seed + 1, p, TRACE_LEVEL, TRACE_BASE_LOG,
                                                    w.sigma_glwe, keys["glwe_key"])),
                          p, TRACE_LEVEL)
    rng = np.random.default_rng(w.data_seed + 2)
    xs = np.clip(rng.normal(0.0, 1.0, batch), -20.0, 20.0)
    m = np.zeros((batch, w.N), np.uint64)
    m[:, 0] = R.encode_fixed(xs, sx)
    x_rlwe = R.to_device(R.glwe_encrypt(w.enc_seed + 1, p, w.sigma_glwe, keys["glwe_key"], m))
    x_cmp = R.to_device(R.lwe_encrypt_plain(w.enc_seed + 2, p, w.sigma_lwe, keys["lwe_key"],
                                            R.encode_fixed(xs, sc)))
    ws = R.empty(R.lookup_workspace_bytes(p, lp, batch) // 8)
    out = R.empty((batch, 2 * w.N))

    def run():
        R.lookup_eval(x_rlwe, x_cmp, bsk, ksk, autk, prep, consts, p, lp, workspace=ws, out=out)

    run()
    torch.cuda.synchronize()
    e0, e1 = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
    t0 = time.perf_counter()
    e0.record(stream)
    for _ in range(steps):
        run()
    e1.record(stream)
    torch.cuda.synchronize()
    wall = (time.perf_counter() - t0) / steps
    sample = np.arange(0, batch, max(1, batch // 512))
    ph = R.glwe_phase(p, keys["glwe_key"], R.to_host(out)[sample])[:, 0].astype(object)
    P = 0xFFFFFFFF00000001
    got = np.array([(v if v <= P // 2 else v - P) / 2.0 ** (sx + sv) for v in ph], dtype=float)
    err = np.abs(got - R.seglut_eval(tau, a, b, xs[sample]))
    return {"function": "silu", "domain": [-20.0, 20.0], "keys": w.name, "nseg": nseg,
            "nbr": lp.nbr, "margin": margin, "cmp_refine_log": refine,
            "batch": batch, "lookups_per_s": round(batch / wall, 2),
            "ms_per_step": round(wall * 1e3, 3),
            "events_ms_per_step": round(e0.elapsed_time(e1) / steps, 3),
            "per_lookup": {"blind_rotations_step1": (3 if refine else 1) * (nseg - 1),
                           "key_switches_step1": (4 if refine else 1) * (nseg - 1),
                           "blind_rotations_encrypted_tp": nseg + 2,
                           "traces": nseg + 1, "plaintext_products": nseg + 2},
            "decrypt_check": {"sample": int(sample.size), "median_abs_err": float(np.median(err)),
                              "p99_abs_err": float(np.quantile(err, 0.99)),
                              "max_abs_err": float(err.max())}}


# Precision of the encrypted lookup (Algorithm 1) against the paper's
# primitive tables: (function, range, boundary spacing, bits the paper
# reports for its segmented LUT).
PRECISION_CASES = [("silu", -20.0, 20.0, "uniform", 16.8), ("gelu", -20.0, 20.0, "uniform", 15.5),
                   ("inv", 0.01, 10.0, "log", 12.7), ("inv", 0.01, 100.0, "log", 12.5),
                   ("inv_sqrt", 0.01, 10.0, "log", 16.7), ("inv_sqrt", 0.01, 100.0, "log", 12.7)]


def _exact(fn, x):
    import math
    if fn == "silu":
        return x / (1.0 + np.exp(-x))
    if fn == "gelu":
        return 0.5 * x * (1.0 + np.array([math.erf(v / math.sqrt(2.0)) for v in x]))
    if fn == "inv":
        return 1.0 / x
    if fn == "inv_sqrt":
        return 1.0 / np.sqrt(x)
    raise ValueError(fn)


def _bits(err) -> float:
    return float(-np.log2(np.sqrt(np.mean(np.square(err)))))


def _lwe_phase(cts, key):
    """b - <a, s> mod p, exact (Python integers)."""
    P = 0xFFFFFFFF00000001
    n = key.shape[0]
    sel = np.nonzero(key)[0]
    return np.array([(int(c[n]) - sum(int(v) for v in c[sel])) % P for c in cts], dtype=object)


def _modswitched_phase(cts, key, N):
    """b~ - sum a~_i s_i mod 2N with a~ = nearest integer to 2N a / p: the
    rotation a blind rotation by these ciphertexts applies."""
    P = 0xFFFFFFFF00000001
    n = key.shape[0]
    sel = np.nonzero(key)[0]
    ms = lambda a: ((2 * N * int(a) + (P - 1) // 2) // P) % (2 * N)
    return np.array([(ms(c[n]) - sum(ms(v) for v in c[sel])) % (2 * N) for c in cts])


def lookup_precision(R, w, p, keys, bsk, ksk, stream, count: int, variants):
    """Encrypted lookup precision, -log2 RMSE over `count` inputs drawn
    uniformly from each range of the paper's primitive tables, 4 segments,
    at the headline ring and keys.  The error is split into its sources:
    the segmented LUT itself (cleartext, exact indices), the interval the
    blind rotation of Step 3 actually selected (from the decrypted segment
    index S and the modulus-switched selector I, both read from the
    workspace), and what remains (value noise of the traces and products).
    The selector's error is split too: the key switch's noise on I (its
    decrypted phase against the exact t) and the modulus switch's drift
    (the modulus-switched phase against the decrypted one).  `variants`
    lists (comparison refinement bits, margin) pairs to run."""
    import torch
    P = 0xFFFFFFFF00000001
    N, n, nseg = w.N, w.n, 4
    sx = 40
    sp = 63 - int(math.log2(N)) - sx
    autk = R.autk_prepare(R.to_device(R.autk_keygen(w.key_seed + 1, p, TRACE_LEVEL,
                                                    TRACE_BASE_LOG, w.sigma_glwe,
                                                    keys["glwe_key"])), p, TRACE_LEVEL)
    rows = []
    cases = [(refine, margin, k, case) for refine, margin in variants
             for k, case in enumerate(PRECISION_CASES)]
    for refine, margin, k, (fn, lo, hi, spacing, paper) in cases:
        nbr = N - 2 * margin
        tau = R.seglut_boundaries(lo, hi, nseg, spacing)
        a, b = R.seglut_build(fn, tau, nbr)
        grid = np.linspace(lo, hi, 20001)
        fmax = float(np.max(np.abs(_exact(fn, grid))))
        reach = max(max(abs(lo - t), abs(hi - t)) for t in tau[1:-1])
        sc = int(math.floor(math.log2(2.0 ** 62 / reach)))
        sv = int(math.floor(62.5 - math.log2(fmax))) - sx
        lp = R.LookupParams(nseg=nseg, nbr=nbr, margin=margin, x_scale_log=sx,
                            coef_scale_log=sp, val_scale_log=sv, cmp_scale_log=sc,
                            trace_level=TRACE_LEVEL, trace_base_log=TRACE_BASE_LOG,
                            cmp_refine_log=refine)
        plain, consts = R.lookup_encode(p, lp, tau, a, b)
        prep = R.lookup_prepare(R.to_device(plain), p, lp)
        xs = np.random.default_rng(w.data_seed + 10 + k).uniform(lo, hi, count)
        m = np.zeros((count, N), np.uint64)
        m[:, 0] = R.encode_fixed(xs, sx)
        x_rlwe = R.to_device(R.glwe_encrypt(w.enc_seed + 10 + k, p, w.sigma_glwe,
                                            keys["glwe_key"], m))
        x_cmp = R.to_device(R.lwe_encrypt_plain(w.enc_seed + 20 + k, p, w.sigma_lwe,
                                                keys["lwe_key"], R.encode_fixed(xs, sc)))
        ws = R.empty(R.lookup_workspace_bytes(p, lp, count) // 8)
        out = R.lookup_eval(x_rlwe, x_cmp, bsk, ksk, autk, prep, consts, p, lp, workspace=ws)
        torch.cuda.synchronize()
        ph = R.glwe_phase(p, keys["glwe_key"], R.to_host(out))[:, 0].astype(object)
        y = np.array([(v if v <= P // 2 else v - P) / 2.0 ** (sx + sv) for v in ph])
        wsh = R.to_host(ws)
        oS = R.lookup_workspace_offset(p, lp, count, R.LOOKUP_PART_S)
        oI = R.lookup_workspace_offset(p, lp, count, R.LOOKUP_PART_I)
        S_ct = wsh[oS:oS + count * (n + 1)].reshape(count, n + 1)
        I_ct = wsh[oI:oI + count * (n + 1)].reshape(count, n + 1)
        key = keys["lwe_key"]
        S_dec = np.array([int(round(float(v) * 2 * nseg / P)) % (2 * nseg)
                          for v in _lwe_phase(S_ct, key)])
        I_ph = np.array([float(v) * 2 * N / P for v in _lwe_phase(I_ct, key)])
        rot = _modswitched_phase(I_ct, key, N)
        # exact segment, interval and selector value
        S_true = np.array([int(np.sum(x >= tau[1:-1])) for x in xs])
        width = tau[S_true + 1] - tau[S_true]
        t_true = nbr * (xs - tau[S_true]) / width + margin - 0.5
        i_true = np.clip(np.floor(nbr * (xs - tau[S_true]) / width), 0, nbr - 1).astype(int)
        centred = lambda d, M: (d + M / 2) % M - M / 2
        ok = S_dec == S_true
        ks_noise = centred(I_ph - t_true, 2 * N)[ok]
        drift = centred(rot - I_ph, 2 * N)[ok]
        S_used = np.clip(S_dec, 0, nseg - 1)
        # the rotation moves coefficient rot of r_S to the constant term;
        # beyond N the negacyclic wrap negates coefficient rot - N, and
        # coefficient j holds interval clamp(j - margin)
        i_sel = np.clip(rot % N - margin, 0, nbr - 1).astype(int)
        sign = np.where(rot >= N, -1.0, 1.0)
        y_sel = sign * (a[S_used, i_sel] * xs + b[S_used, i_sel])
        y_lut = a[S_true, i_true] * xs + b[S_true, i_true]
        f = _exact(fn, xs)
        sim = R.seglut_precision(fn, tau, a, b, xs,
                                 np.rint(np.random.default_rng(7).normal(
                                     0, float(np.sqrt(np.mean(np.square(ks_noise + drift)))),
                                     count)).astype(np.int32))
        rows.append({"function": fn, "range": [lo, hi], "spacing": spacing, "inputs": count,
                     "cmp_refine_log": refine, "margin": margin, "nbr": nbr,
                     "scales": {"x": sx, "coef": sp, "val": sv, "cmp": sc},
                     "bits_vs_exact": round(_bits(y - f), 2),
                     "bits_vs_cleartext_lut": round(_bits(y - y_lut), 2),
                     "paper_bits": paper,
                     "sources_bits": {"cleartext_lut_vs_exact": round(_bits(y_lut - f), 2),
                                      "selection_vs_cleartext_lut": round(_bits(y_sel - y_lut), 2),
                                      "value_noise": round(_bits(y - y_sel), 2)},
                     "segment_misses": int(np.sum(~ok)),
                     "selector_steps_rms": {"key_switch_noise": round(float(np.sqrt(np.mean(
                                                ks_noise ** 2))), 2),
                                            "modulus_switch_drift": round(float(np.sqrt(np.mean(
                                                drift ** 2))), 2)},
                     "interval_error_rms": round(float(np.sqrt(np.mean(
                         (i_sel - i_true)[ok].astype(float) ** 2))), 2),
                     "simulated_bits_at_measured_selector_rms": round(sim, 2)})
        log(f"[precision] refine {refine} margin {margin}: {fn} [{lo}, {hi}]: "
            f"{rows[-1]['bits_vs_exact']} bits (paper {paper})")
    return rows


def main():
    ap = argparse.ArgumentParser()
    ap.add_argument("--gpus", type=int, default=1)
    ap.add_argument("--steps", type=int, default=10)
    ap.add_argument("--warmup", type=int, default=2)
    ap.add_argument("--workload", default=None)
    ap.add_argument("--cpu-seconds", type=float, default=15.0,
                    help="target CPU time of the oracle baseline sample (0 = skip)")
    ap.add_argument("--batch", type=int, default=None,
                    help="override the workload's batch (experiments only)")
    ap.add_argument("--lookup-steps", type=int, default=3,
                    help="timed steps of the lookup select (0 = skip)")
    ap.add_argument("--protocol-steps", type=int, default=1,
                    help="timed steps of the full lookup pipeline (0 = skip)")
    ap.add_argument("--protocol-batch", type=int, default=4096,
                    help="inputs of the lookup pipeline")
    ap.add_argument("--precision", type=int, default=0,
                    help="instead of the benchmark: encrypted lookup precision in bits over "
                         "this many uniform inputs per primitive of the paper's tables "
                         "(keys: --workload, default llama3_8b_lookup)")
    ap.add_argument("--precision-variants", default="5:32",
                    help="comma-separated refine:margin pairs of the precision run")
    ap.add_argument("--calibrate-copy-mib", type=int, default=0,
                    help="also run one plain device copy of this many MiB, outside the timed "
                         "region, as the reference kernel for memory-traffic counters")
    args = ap.parse_args()
    if args.gpus != 1:
        print(f"bench.py measures one GPU only (got --gpus {args.gpus}); batched PBS shards "
              "by ciphertext with no exchange, so a multi-GPU figure is not produced here",
              file=sys.stderr)
        sys.exit(2)

    import torch
    from paper_2609_16915_amd import rosetta as R
    from paper_2609_16915_amd import workloads as W

    name = args.workload or ("llama3_8b_lookup" if args.precision else W.HEADLINE)
    w = W.get(name)
    if args.batch:
        import dataclasses
        w = dataclasses.replace(w, batch=args.batch)
    p = R.Params.from_dict(w.params())
    torch.cuda.set_device(0)
    stream = torch.cuda.current_stream()

    log(f"[bench] {name}: keygen (library host helper)")
    keys = R.keygen(w.key_seed, p, w.sigma_lwe, w.sigma_glwe)
    msgs = w.messages()
    cts = R.lwe_encrypt(w.enc_seed, p, w.sigma_lwe, keys["lwe_key"], msgs)
    table = w.table()
    v = R.lut_build(p, table)

    bsk = R.bsk_prepare(R.to_device(keys["bsk"]), p)
    ksk = R.ksk_prepare(R.to_device(keys["ksk"]), p)
    if args.precision:
        variants = [tuple(int(v) for v in pair.split(":"))
                    for pair in args.precision_variants.split(",")]
        rows = lookup_precision(R, w, p, keys, bsk, ksk, stream, args.precision, variants)
        print(json.dumps({"lookup_precision": rows, "workload": name, "library": R.version()}),
              flush=True)
        return
    d_in, d_v = R.to_device(cts), R.to_device(v)
    d_out = R.empty((w.batch, w.n + 1))
    ws = R.empty(R.pbs_workspace_bytes(p, w.batch) // 8)
    big = ws.view(w.batch, w.N + 1)
    torch.cuda.synchronize()

    def step():
        R.blind_rotate_extract(d_in, bsk, d_v, p, out=big)
        R.keyswitch(big, ksk, p, out=d_out)

    if args.calibrate_copy_mib:
        words = args.calibrate_copy_mib * (1 << 20) // 8
        src = torch.zeros(words, dtype=torch.int64, device="cuda")
        dst = torch.empty_like(src)
        torch.cuda.synchronize()
        torch.add(src, 1, out=dst)  # elementwise: reads and writes `words` * 8 bytes
        torch.cuda.synchronize()
        del src, dst

    log(f"[bench] warmup {args.warmup}")
    for _ in range(args.warmup):
        step()
    torch.cuda.synchronize()

    ev = [(torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True),
           torch.cuda.Event(enable_timing=True)) for _ in range(args.steps)]
    log(f"[bench] timing {args.steps} steps")
    torch.cuda.synchronize()
    t0 = time.perf_counter()
    for e0, e1, e2 in ev:
        e0.record(stream)
        R.blind_rotate_extract(d_in, bsk, d_v, p, out=big)
        e1.record(stream)
        R.keyswitch(big, ksk, p, out=d_out)
        e2.record(stream)
    torch.cuda.synchronize()
    wall = time.perf_counter() - t0
    br_ms = float(np.mean([a.elapsed_time(b) for a, b, _ in ev]))
    ks_ms = float(np.mean([b.elapsed_time(c) for _, b, c in ev]))
    step_ms = [a.elapsed_time(c) for a, _, c in ev]
    ms_per_step = wall * 1e3 / args.steps
    value = w.batch / (wall / args.steps)

    # the same step through the single entry point gives the same bits
    ref = R.pbs_batch(d_in, bsk, ksk, d_v, p)
    torch.cuda.synchronize()
    out = R.to_host(d_out)
    same = bool(np.array_equal(out, R.to_host(ref)))
    ok_rate = float(np.mean(R.lwe_decrypt(p, keys["lwe_key"], out) == table[msgs]))

    modmul_per_launch = w.br_modmul_per_pbs() * w.batch
    achieved_t = modmul_per_launch / (br_ms * 1e-3) / 1e12
    probe_t = modmul_probe(stream)
    pieces = key_pieces(w.N, w.pbs_level, w.pbs_base_log)
    if pieces:
        # double-precision transforms take the modular products' place, so the
        # modular count is an equivalent (its frac may pass 1) and the roofline
        # counts the double-precision operations the method needs
        flops = w.batch * w.n * fft_flops(w.N, int(math.log2(w.N)) - 1, 2 * w.pbs_level,
                                          2 * pieces, 4 * w.pbs_level * pieces)
        achieved_f = flops / (br_ms * 1e-3) / 1e12
        roofline = {"bound": "alu", "kernel": "k_blind_rotate_fft", "dtype": "f64",
                    "achieved": round(achieved_f, 4), "peak": round(FP64_PEAK_T, 4),
                    "unit": "TFLOP/s", "frac": round(achieved_f / FP64_PEAK_T, 4),
                    "traffic": measured_traffic(name, w.batch),
                    "per_launch_flops": flops, "key_pieces": pieces}
    else:
        few = w.N <= 1024 and w.batch <= 2 * CU
        roofline = {"bound": "alu", "kernel": "k_blind_rotate_teams" if few else "k_blind_rotate",
                    "achieved": round(achieved_t, 4),
                    "peak": round(MODMUL_PEAK_T, 4), "unit": "Tmodmul/s",
                    "frac": round(achieved_t / MODMUL_PEAK_T, 4),
                    "traffic": measured_traffic(name, w.batch)}
    roofline.update({"launch_ms": round(br_ms, 3), "per_launch_modmul": modmul_per_launch,
                     "modmul_equivalent": round(achieved_t, 4),
                     "modmul_peak": round(MODMUL_PEAK_T, 4),
                     "modmul_equivalent_frac": round(achieved_t / MODMUL_PEAK_T, 4),
                     "multiplier_bound": round(MULTIPLIER_BOUND_T, 4),
                     "modmul_probe": round(probe_t, 4)})
    hbm_bytes = (w.bsk_words() + w.ksk_words()) * 8 + w.batch * 2 * (w.n + 1) * 8 + w.N * 8
    ks_kernel = keyswitch_kernel(w.n, w.N, w.ks_level, w.ks_base_log, w.batch)
    # (on the int8 matrix cores: 8 byte-plane products of 2 ops per digit MAC)
    ks_mfma = ks_kernel != "k_keyswitch"
    # algorithmic work: one multiply and one add per digit MAC; the kernel
    # executes 8 byte-plane products per MAC (dense_equivalent_ops)
    ks_ops = 2 * w.batch * w.N * w.ks_level * (w.n + 1)
    ks_dense = 8 * ks_ops
    roofline_ks = ({"bound": "mfma", "kernel": ks_kernel, "dtype": "i8",
                    "achieved": round(ks_ops / (ks_ms * 1e-3) / 1e15, 5),
                    "peak": INT8_PEAK_P, "unit": "POP/s",
                    "frac": round(ks_ops / (ks_ms * 1e-3) / 1e15 / INT8_PEAK_P, 5),
                    "per_launch_ops": ks_ops, "dense_equivalent_ops": ks_dense,
                    "frac_dense_equivalent": round(ks_dense / (ks_ms * 1e-3) / 1e15
                                                   / INT8_PEAK_P, 4),
                    "launch_ms": round(ks_ms, 3)}
                   if ks_mfma else None)

    result = {
        "metric": f"PBS/sec (bootstraps/s) at N={w.N} batch {w.batch}; "
                  "% of int64-VALU / HBM roofline",
        "value": round(value, 2), "unit": "PBS/s", "n_gpus": 1, "steps": args.steps,
        "warmup": args.warmup, "ms_per_step": round(ms_per_step, 3),
        "ms_per_step_events": {"median": round(float(np.median(step_ms)), 3),
                               "min": round(float(np.min(step_ms)), 3)},
        "higher_is_better": True,
        "scaling": "weak", "vs_baseline": None, "dtype": "u64 mod p (Goldilocks)",
        "data": "synthetic (seeded activations, random keys)",
        "library": R.version(),
        "config": {"workload": name, "n": w.n, "N": w.N, "pbs_level": w.pbs_level,
                   "pbs_base_log": w.pbs_base_log, "ks_level": w.ks_level,
                   "ks_base_log": w.ks_base_log, "msg_bits": w.msg_bits, "batch": w.batch,
                   "function": w.function},
        "kernels_ms": {"blind_rotate_extract": round(br_ms, 3), "keyswitch": round(ks_ms, 3)},
        "hbm_algorithmic_frac": round(hbm_bytes / (ms_per_step * 1e-3) / 1e9 / HBM_PEAK_GBS, 6),
        "checks": {"split_equals_pbs_batch": same, "decrypt_equals_table_rate": round(ok_rate, 5)},
        "roofline": roofline,
        "roofline_keyswitch": roofline_ks,
    }
    if args.lookup_steps > 0:
        log("[bench] lookup select (blind rotation of ciphertext test polynomials + trace)")
        result["lookup_select"] = lookup_select(R, W, w, p, keys, d_in, bsk, stream,
                                                args.lookup_steps)
    if args.protocol_steps > 0:
        log("[bench] lookup pipeline (Algorithm 1, Steps 1-3)")
        result["lookup_protocol"] = lookup_protocol(R, W, stream, args.protocol_steps,
                                                    args.protocol_batch)
    if args.cpu_seconds > 0:
        log("[bench] CPU oracle baseline")
        result["cpu_baseline"] = cpu_baseline(w, keys, cts, v, args.cpu_seconds)
    else:
        result["cpu_baseline"] = None
    print(json.dumps(result), flush=True)


if __name__ == "__main__":
    main()
