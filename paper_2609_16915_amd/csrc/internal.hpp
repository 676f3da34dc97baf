// Internal interface between the C ABI (abi.cpp) and the kernels
// (kernels.hip).  Not installed; the public surface is include/rosetta.h.
#pragma once

#include <hip/hip_runtime.h>

#include <cstddef>
#include <cstdint>

#include "rosetta.h"

namespace rosetta {

// Largest LWE dimension the blind-rotation kernel accepts (its rounded
// rotation amounts are staged in LDS).
constexpr uint32_t MAX_LWE_N = 2048;
constexpr size_t LDS_PER_CU = 160 * 1024;

// Shape of the transform the kernels use at N = 2^logn: E = 2^ntt_le(logn)
// elements per thread, pass 0 spanning ntt_first(logn) stages and every
// later pass ntt_le(logn) (Ntt in ntt.hpp).  The twiddle table (abi.cpp)
// is laid out for exactly this shape.
constexpr int ntt_le(int logn) { return logn == 8 ? 2 : 3; }
constexpr int ntt_first(int logn) { return logn == 11 ? 2 : ntt_le(logn); }

// Per-device, per-N transform tables (device pointers) and N^-1.
struct Tables {
  // N words: zeta[m] = psi^rev(m) (zeta[0] = 1), with the regions of the
  // twisted passes holding their block powers and the stages of a last
  // pass that is not twisted stored slot-major (see ntt.hpp)
  const uint64_t *zeta;
  // N words: psi^e for e = 0 .. N-1 (psi^N = -1 gives the rest), read by the
  // blind rotation that keeps its accumulator in the transform domain
  const uint64_t *psi;
  uint64_t ninv;
  // complex words of the double-precision transform (Fft::TABLE, fft.hpp),
  // N >= 2048; nullptr below
  const double *fft;
};

enum BrMode { BR_GLWE = 0, BR_EXTRACT = 1 };

// rosetta_pbs_batch_ws; may_allocate false keeps the whole call free of
// device allocations.
rosetta_status pbs_batch(const uint64_t *lwe_in, const uint64_t *bsk_dev, const uint64_t *ksk_dev,
                         const uint64_t *lut, uint64_t *lwe_out, size_t batch,
                         const rosetta_params *params, void *workspace, size_t workspace_bytes,
                         bool may_allocate, void *stream);

// Compute units of the current device (0 if unknown).
int device_cus();

// Record the calling thread's error message (read by rosetta_last_error).
void set_last_error(const char *msg);

hipError_t launch_bsk_prepare(const uint64_t *bsk_std, uint64_t *bsk_dev,
                              const rosetta_params &p, const Tables &tb, hipStream_t st);
hipError_t launch_ksk_prepare(const uint64_t *ksk_std, uint64_t *ksk_dev,
                              const rosetta_params &p, hipStream_t st);
// Blind rotation: with double-precision transforms where fft_pieces allows
// them and the key can be expanded into memory of the call's own (not while
// the stream is being captured, and only if the caller allows allocations),
// else with the modular ones.
hipError_t launch_blind_rotate(const uint64_t *lwe_in, const uint64_t *bsk_dev,
                               const uint64_t *lut, uint64_t *out, size_t batch,
                               const rosetta_params &p, const Tables &tb, BrMode mode,
                               int tp_glwe, bool may_allocate, hipStream_t st);
hipError_t launch_blind_rotate_ntt(const uint64_t *lwe_in, const uint64_t *bsk_dev,
                                   const uint64_t *lut, uint64_t *out, size_t batch,
                                   const rosetta_params &p, const Tables &tb, BrMode mode,
                                   int tp_glwe, hipStream_t st);
// Device memory for one call on stream st (scratch.cpp): nullptr where it is
// not to be had, the stream being captured included.  scratch_give returns it
// once the work enqueued so far is done; scratch_release waits for every
// device that has a pool and gives what the pools keep back to it.
void *scratch_take(size_t bytes, hipStream_t st);
hipError_t scratch_give(void *p, hipStream_t st);
void scratch_release();

// Pieces per key coefficient of the double-precision blind rotation and
// trace, R rows of base_log = beta bits: 3 of 22 bits, 4 of 16, or 0 where
// only the modular transforms are exact.
//
// Error bound, u = 2^-53, M = log2(N/2) stages.  A butterfly's
// sum is off by at most u(2|a| + 3|b|), its difference by u(3|a| + 4|b|)
// (inputs a, b; roundings and the twiddle's own u), in the 2-norm 4.4 u of
// the outputs, so the transforms of a digit polynomial d and of a piece k
// are off by 4.4 M u relative each; the R complex products summed by fused
// multiply-adds add 2.9 R u of sum |D||K| per point; and a coefficient of
// the inverse is off by at most (4 (M - 2) + 2 + 7) u of the mean over
// points of sum |D||K| (every path's roundings, the final twist included),
// which is at most sum ||d|| ||k|| (Cauchy-Schwarz and Parseval).  Together
// 146.4 u at N = 2048 and 159.2 u at N = 4096 for R = 6: 160 u.  With |d| <=
// 2^(beta-1) and |k| <= 2^(b-1), ||d|| ||k|| <= N 2^(beta + b - 2), hence
//   error <= R N 2^(beta + b - 2) 160 2^-53, wanted <= 1/4.
// No input can exceed it: the bound holds for every digit and key word.
inline int fft_pieces_for(unsigned N, unsigned rows, unsigned base_log) {
  if (N != 2048 && N != 4096) return 0;
  const uint64_t f = (uint64_t)rows * N * 160;  // below 2^24
  auto holds = [&](unsigned bits) {
    const unsigned e = base_log + bits - 2;
    return e < 40 && f << e <= (uint64_t)1 << 51;
  };
  return holds(22) ? 3 : holds(16) ? 4 : 0;
}
inline int fft_pieces(const rosetta_params &p) {
  if (p.pbs_level > 3) return 0;  // (no registers for eight transforms)
  const int pieces = fft_pieces_for(p.N, 2 * p.pbs_level, p.pbs_base_log);
  // the 3-piece instances keep the rounded value in 32 bits
  return pieces == 3 && p.pbs_level * p.pbs_base_log > 30 ? 4 : pieces;
}

// Pieces of the double-precision trace of a batch on a device of `cus` compute
// units, 0 for the modular one.  A single level in four pieces takes eight
// sums back for the one digit polynomial it transforms and pays only where
// that hides: N = 2048, 13 bits, up to two workgroups per CU (256 / 513 / 14336
// traces 123 / 250 / 3916 against 132 / 229 / 3620 us modular); N = 4096, 12
// bits, past one per CU (256 / 513 / 14336 traces 233 / 624 / 11301 against
// 215 / 631 / 11989).
inline int trace_pieces(unsigned N, unsigned level, unsigned base_log, size_t batch, size_t cus) {
  const int pieces = fft_pieces_for(N, level, base_log);
  if (level == 1 && pieces == 4 && (N == 2048 ? batch > 2 * cus : batch <= cus)) return 0;
  return pieces;
}

hipError_t launch_rows_prepare(const uint64_t *rows_std, uint64_t *rows_dev, size_t rows,
                               uint32_t N, const Tables &tb, hipStream_t st);
// Trace: as launch_blind_rotate, with double-precision transforms where it can.
hipError_t launch_trace(const uint64_t *in, const uint64_t *autk_dev, uint64_t *out,
                        size_t batch, uint32_t N, int level, int base_log, const Tables &tb,
                        hipStream_t st);
hipError_t launch_trace_ntt(const uint64_t *in, const uint64_t *autk_dev, uint64_t *out,
                            size_t batch, uint32_t N, int level, int base_log, const Tables &tb,
                            hipStream_t st);
hipError_t launch_glwe_mul_plain(const uint64_t *in, const uint64_t *pa_dev, const uint64_t *pb,
                                 uint64_t *out, size_t batch, int npoly, uint32_t N,
                                 const Tables &tb, hipStream_t st);
// Monomial exponents (each in [0, 2N)) passed by value to the kernels.
constexpr int MAX_MONOMIALS = 256;
struct Exponents {
  uint16_t e[MAX_MONOMIALS];
};

hipError_t launch_glwe_recombine(const uint64_t *in, uint64_t *out, size_t batch, int count,
                                 const Exponents &ex, uint32_t N, hipStream_t st);
hipError_t launch_glwe_monomial_mul(const uint64_t *in, uint64_t *out, size_t batch, int count,
                                    const Exponents &ex, uint32_t N, hipStream_t st);
hipError_t launch_sample_extract(const uint64_t *in, uint64_t *out, size_t batch, uint32_t N,
                                 hipStream_t st);

// Per-copy constants passed by value (at most MAX_MONOMIALS).
struct Consts {
  uint64_t c[MAX_MONOMIALS / 4];
};
hipError_t launch_lwe_add_consts(const uint64_t *in, uint64_t *out, size_t batch, int count,
                                int dim, const Consts &cs, hipStream_t st);
hipError_t launch_lwe_combine(const uint64_t *a, uint64_t alpha, const uint64_t *b, uint64_t beta,
                              const uint64_t *c, uint64_t gamma, uint64_t *out, size_t words,
                              hipStream_t st);
hipError_t launch_lwe_sum_groups(const uint64_t *in, uint64_t *out, size_t batch, int count,
                                 int dim, uint64_t c0, hipStream_t st);
// op as in rosetta_field_op (validated by the caller)
hipError_t launch_field_op(int op, const uint64_t *a, const uint64_t *b, const uint64_t *c,
                           uint64_t *out, size_t count, hipStream_t st);
hipError_t launch_modmul_chain(uint64_t seed, uint32_t threads, uint32_t iters, uint64_t *out,
                               hipStream_t st);
hipError_t launch_keyswitch(const uint64_t *big, const uint64_t *ksk_dev, uint64_t *out,
                            size_t batch, const rosetta_params &p, bool may_allocate,
                            hipStream_t st);

// The key switch is one integer matrix product over the batch (digits x
// key), run on the int8 matrix cores when the signed digits fit a byte
// (|d| <= 2^(beta_ks-1) <= 64), the rounded value 31 bits (l_ks beta_ks
// <= 30), N is a multiple of 32 (whole 32-deep k blocks), and no int32 sum
// of N l_ks digit x key-byte products can overflow (N l_ks 2^(beta_ks-1)
// 128 < 2^31).  Otherwise the VALU kernel runs.  The prepared key's layout
// follows the choice (launch_ksk_prepare).
inline bool ks_on_matrix_cores(const rosetta_params &p) {
  if (p.ks_base_log < 1 || p.ks_base_log > 7 || p.ks_level < 1) return false;
  if (p.ks_level * p.ks_base_log > 30 || p.N % 32 != 0) return false;
  const uint64_t bound = (uint64_t)p.N * p.ks_level * (1ull << (p.ks_base_log - 1)) * 128;
  return bound < (1ull << 31);
}
// Which kernel switches a batch on a device of `cus` compute units.  (Times in
// us with 256 CUs, calls back to back.)
enum class KsRoute { VALU, SPLIT, DIGITS, MFMA };
constexpr size_t KS_MFMA_ROWS = 128;  // ciphertexts of a workgroup of k_keyswitch_mfma
inline KsRoute ks_route(const rosetta_params &p, size_t batch, size_t cus) {
  if (!ks_on_matrix_cores(p)) return KsRoute::VALU;
  const size_t cols = (p.n + 1 + 31) / 32, K = (size_t)p.N * p.ks_level;
  // Few enough ciphertexts that every 16 of them and 32 columns have a CU
  // (a workgroup of the split kernel fills one): there the split wins, 64
  // ciphertexts 82 against 175 at the headline parameters; just past it,
  // 128, it ties (178 against 175), at 1024 it loses (510 against 184).
  if ((batch + 15) / 16 * cols <= cus) return KsRoute::SPLIT;
  // Digits made once pay by being shared among column blocks and cost a pass
  // over the batch and 28 us of host work (two launches, scratch).  Against
  // them k_keyswitch_mfma takes one round of workgroups (about as long at any
  // batch up to rows = cus), then two per CU.  Digits against that kernel:
  const size_t rows = (batch + KS_MFMA_ROWS - 1) / KS_MFMA_ROWS;
  // one or two column blocks and the chip filled: n = 50, N = 2048, 6 levels,
  // 20480 / 28672 / 131072 ciphertexts 444 / 541 / 2722 against 494 / 493 /
  // 2179; n = 20, N = 1024, 2 levels, 12288 / 16384 / 20480 ones 88 / 113 /
  // 130 against 109 / 110 / 110; n = 20, N = 512, 1 level, 9000 / 12288 ones
  // 37 / 50 against 39 / 40
  if (cols <= 2 && 16 * rows > (K <= 1024 ? 5 : K <= 2048 ? 7 : 10) * cus) return KsRoute::MFMA;
  // three, and two full workgroups per CU: n = 80, N = 512, 2 levels, 16384 /
  // 20480 / 22528 ciphertexts 66 / 80 / 95 against 72 / 70 / 118
  if (cols == 3 && K <= 1024 && 16 * rows * cols > 26 * cus && rows * cols <= 2 * cus)
    return KsRoute::MFMA;
  // the shortest contractions.  1 level, N = 256: up to 96 columns (n = 64, 1361 /
  // 32768 / 65536 ciphertexts 29 / 63 / 110 against 18 / 50 / 95), or while the
  // work is less than the host's (n = 1024, 896 / 1408 / 1920 ciphertexts, 231 /
  // 363 / 495 workgroups, 30 / 29 / 30 against 21 / 29 / 32); 2 levels: n = 1024,
  // 226 / 896 ciphertexts, 66 / 231 workgroups, 29 / 29 against 25 / 32
  if (K == 256 && (cols <= 3 || 2 * rows * cols <= 3 * cus)) return KsRoute::MFMA;
  if (p.N == 256 && p.ks_level == 2 && 2 * rows * cols <= cus) return KsRoute::MFMA;
  return KsRoute::DIGITS;
}
// Words of the byte-plane key: ceil((n+1)/32) column blocks x N l_ks / 32
// k blocks x 1024 words (16 operand fragments of 64 lanes x 8 bytes).
inline size_t ks_matrix_key_words(const rosetta_params &p) {
  return (size_t)((p.n + 1 + 31) / 32) * ((size_t)p.N * p.ks_level / 32) * 1024;
}
hipError_t launch_ntt(const uint64_t *in, uint64_t *out, size_t count, uint32_t N,
                      const Tables &tb, bool inverse, hipStream_t st);
hipError_t launch_poly_mul(const uint64_t *a, const uint64_t *b, uint64_t *c, size_t count,
                           uint32_t N, const Tables &tb, hipStream_t st);

}  // namespace rosetta
