// Blind rotation and trace with double-precision transforms (see fft.hpp),
// exact.
//
// The products of a step, digits x key row, are exact integers that
// only have to be known modulo p, so the transform need not be modular: each
// centred key coefficient is cut into P balanced pieces of PB bits, every
// digit polynomial is transformed once in double precision, multiplied with
// the transforms of the pieces, and the P sums per component come back with
// an error below 1/4 (fft_pieces has the bound), round to the exact integers
// and are put together modulo p.  Same bits as the modular transforms of
// kernels.hip for every input.
#include <hip/hip_runtime.h>

#include <type_traits>

#include "fft.hpp"
#include "gl.hpp"
#include "internal.hpp"
#include "ntt.hpp"

namespace rosetta {

extern __shared__ __align__(16) u64 fft_lds[];

// Bits per key piece.
template <int P>
constexpr int piece_bits() {
  return P == 3 ? 22 : 16;
}

// ---------------------------------------------------------------------------
// Key expansion: prepared (modular) rows -> transforms of their pieces
// ---------------------------------------------------------------------------

// Workgroups (step, y): a step is a GGSW or a round of the trace, of which
// workgroup y takes every gridDim.y-th row.  Row (r, c) of the
// prepared key, r < R, goes back to coefficients (its N^-1 scaling makes the
// plain inverse exact), each is centred and cut into P balanced pieces, and
// the pieces are transformed.  Expanded layout, in complex words:
// [step][c][p][r][slot k][thread], scaled by +-1/C (a power of two, exact), as
// the products read it.
template <class S, class F, int P>
__global__ void __launch_bounds__(S::T)
k_expand_key(const u64 *__restrict__ prepared, cd *__restrict__ out, int R, double scale,
             const u64 *__restrict__ zeta, const cd *__restrict__ fft_tab) {
  static_assert(S::T == F::T && S::E == 8, "one thread layout for both transforms");
  constexpr int N = S::N, T = S::T, C = F::C, PB = piece_bits<P>();
  cd *tab = (cd *)fft_lds;
  u64 *tw = fft_lds + F::TABLE_BYTES / 8;
  u64 *xch = tw + S::TW_WORDS;
  LdsBufs<S> lds(xch);
  const int tid = threadIdx.x;
  const FftLane<F::TABLE_BYTES + 8 * S::TW_WORDS> ln(tid);  // (the buffer is xch)
  load_twiddles<S>(tw, zeta, tid);
  for (int i = tid; i < F::TABLE; i += T) tab[i] = fft_tab[i];
  __syncthreads();
  const int rows = 2 * R;
#pragma unroll 1
  for (int row = blockIdx.y; row < rows; row += gridDim.y) {
    const u64 *src = prepared + ((size_t)blockIdx.x * rows + row) * N;
    u64 x[8];
#pragma unroll
    for (int k = 0; k < 8; ++k) x[k] = gl_canon(src[k * T + tid]);
    ntt_inverse<S>(x, lds, tid, tw);
    // centred representative, |v| <= (p - 1) / 2
    i64 v[8];
#pragma unroll
    for (int k = 0; k < 8; ++k) v[k] = x[k] > (GL_P - 1) / 2 ? (i64)(x[k] - GL_P) : (i64)x[k];
    const int c = row & 1, r = row >> 1;
#pragma unroll 1
    for (int p = 0; p < P; ++p) {
      cd z[1][4];
#pragma unroll
      for (int k = 0; k < 4; ++k) {
        i64 d[2];
#pragma unroll
        for (int h = 0; h < 2; ++h) {
          i64 &w = v[k + 4 * h];
          // balanced low PB bits, the rest carried up; the last piece is
          // what remains
          d[h] = p == P - 1 ? w : (i64)((u64)w << (64 - PB)) >> (64 - PB);
          w = (w - d[h]) >> PB;
        }
        z[0][k] = cd{(double)d[0] * scale, (double)d[1] * scale};
      }
      // the transform opens with a barrier, so the last reads of the buffer
      // are over
      fft_forward<F, 1, 0>(z, ln, NoHook{});
      cd *o = out + (((size_t)(blockIdx.x * 2 + c) * P + p) * R + r) * C + tid;
#pragma unroll
      for (int k = 0; k < 4; ++k) o[k * T] = z[0][k];
    }
    __syncthreads();
  }
}

// ---------------------------------------------------------------------------
// Blind rotation
// ---------------------------------------------------------------------------

// Rows of the expanded key through a raw buffer descriptor (as KeyRows in
// kernels.hip): wave-uniform base, the lane's offset in a vector register.
struct ExpandedRows {
  __amdgpu_buffer_rsrc_t r;
  __device__ __forceinline__ explicit ExpandedRows(const cd *base)
      : r(__builtin_amdgcn_make_buffer_rsrc((void *)base, (short)0, 0x7FFFFFFF, 0x00020000)) {}
  __device__ __forceinline__ cd load(int lane_byte, int byte) const {
    const auto v = __builtin_amdgcn_raw_buffer_load_b128(r, lane_byte, byte, 0);
    return cd{__longlong_as_double((long long)gl_mk(v[0], v[1])),
              __longlong_as_double((long long)gl_mk(v[2], v[3]))};
  }
};

// The P rounded sums of one coefficient put together and added to acc.
// t_p = y_p + M_p with M_p = 1.5 2^52 + m_p rounds y_p to an integer r_p and
// leaves bits(t_p) = 0x4338 2^48 + m_p + r_p (|r_p| < 2^44 wherever fft_pieces
// accepts; for P = 4 the last m_p keeps the sum positive).  sum 2^(PB p) bits(t_p) without the constant top
// bits of the last one (52.. for P = 3, 48.. for P = 4) is the wanted sum
// plus a constant that the m_p make 0 mod p (PieceOffsets), so nothing is
// left to subtract: lo and the word hi of 2^64 = 2^32 - 1 are added up and
// reduced once, canonical.
template <int P>
struct PieceOffsets {
  double m[P];  // M_p
};
template <int P>
constexpr PieceOffsets<P> piece_offsets() {
  constexpr int PB = piece_bits<P>();
  typedef unsigned __int128 u128;
  // the last piece's own part: 2^51 (P = 3) or 2^47 on top of zero (P = 4:
  // m_3 includes 2^47 so that the 48 kept bits stay positive)
  u64 k = 0, w = 1;  // constant so far and 2^(PB p), mod p
  for (int p = 0; p < P; ++p) {
    const u64 top = p < P - 1 ? 0x4338000000000000ull : (P == 3 ? (1ull << 51) : (1ull << 47));
    k = (u64)(((u128)w * (top % GL_P) + k) % GL_P);
    w = (u64)(((u128)w << PB) % GL_P);
  }
  const u64 target = k ? GL_P - k : 0;  // = sum 2^(PB p) m_p mod p
  i64 v = target > (GL_P - 1) / 2 ? (i64)(target - GL_P) : (i64)target;
  PieceOffsets<P> r{};
  for (int p = 0; p < P; ++p) {
    const i64 half = (i64)1 << (PB - 1);
    const i64 d = p == P - 1 ? v : (((v + half) & (((i64)1 << PB) - 1)) - half);
    v = (v - d) >> PB;
    r.m[p] = 6755399441055744.0 + (double)d +
             (P == 4 && p == P - 1 ? 140737488355328.0 : 0.0);  // 1.5 2^52 (+ 2^47)
  }
  return r;
}

// The rounded sum of piece p into (acc, top): 128-bit sums, top at 2^64.
template <int P, int p>
__device__ __forceinline__ void add_piece(u64 &acc, u32 &top, double y) {
#if defined(__HIP_DEVICE_COMPILE__)
  constexpr PieceOffsets<P> M = piece_offsets<P>();
  constexpr int sh = p * piece_bits<P>();
  const u64 B = (u64)__double_as_longlong(y + M.m[p]);
  u64 c0, c1;
  u32 lo = (u32)acc, hi = (u32)(acc >> 32);
  if constexpr (p == 0) {
    lo = isa::add_c(lo, (u32)B, c0);
    hi = isa::addc_c(hi, (u32)(B >> 32), c0, c1);
    top = isa::inc_ci(0u, c1);
  } else if constexpr (sh < 32) {
    const u64 w = B << sh;
    lo = isa::add_c(lo, (u32)w, c0);
    hi = isa::addc_c(hi, (u32)(w >> 32), c0, c1);
    top = isa::inc_ci(top + (u32)(B >> (64 - sh)), c1);
  } else {
    hi = isa::add_c(hi, (u32)B << (sh - 32), c1);
    top = isa::inc_ci(top + (u32)(B >> (64 - sh)), c1);
  }
  acc = gl_mk(lo, hi);
#endif
}
// acc + top (2^32 - 1) mod p, canonical: a wrapped sum plus 2^32 - 1 stays
// below p.
__device__ __forceinline__ u64 finish_pieces(u64 acc, u32 top) {
#if defined(__HIP_DEVICE_COMPILE__)
  u64 ca;
  const u64 R = isa::mad_eps_c(top, acc, ca);
  return isa::add_eps_if(R, ca | isa::ge_p(R));
#else
  return acc;
#endif
}

// Key groups (16 registers each) in flight ahead of their use: what the 256
// registers of two waves per SIMD leave room for.  A step asks for 590 KB of
// key per ciphertext at N = 2048, l = 3, 9.2k cycles of a CU's 64 bytes per
// cycle, so the loads have to spread over the whole step.  N = 2048, l = 3, 3
// groups (with the accumulator parked, below) against 2: one ciphertext 15.9
// against 16.8 ms, 1536 of them 64.8 against 65.7 ms; 4 spill 67 registers:
// 100.5 ms.
template <int L>
constexpr int key_ahead() {
  return L == 3 ? 3 : 2;
}
// Sums taken back side by side: two where fewer rows leave the registers
// (l = 2, 1536 GPT-2 ciphertexts: 35.8 ms, one sum and 4 groups 36.9 ms).
template <int L>
constexpr int sums_at_once() {
  return L == 3 ? 1 : 2;
}
// Complex words of the exchange buffer: the L digit polynomials of a
// component, two sums, or the two components of the rotation.
template <class F, int L>
constexpr int fft_buf_words() {
  return (L > 2 ? L : 2) * F::C;
}
template <class F, int L>
constexpr size_t br_fft_lds_bytes(int n) {
  return F::TABLE_BYTES + (size_t)fft_buf_words<F, L>() * sizeof(cd) +
         (((size_t)(n + 1) * 2 + 15) & ~(size_t)15);
}

// One workgroup per ciphertext, the coefficient-domain loop of
// k_blind_rotate.  Per CMux step: both components rotate through LDS and
// are rounded (R); the L digit polynomials of each are transformed side by
// side into D (2L transforms, 16 registers each, live to the end of the
// step); sum S = (component, piece) over the 2L rows is formed a group (one
// row of the key, 4 points per thread) at a time, taken back, rounded and put
// together into the accumulator.  Every wait of a transform for the LDS or
// for the other waves is filled (hooks) with work that is ready: component
// 1's digits during component 0's transforms, sum 0's first rows during
// component 1's, the groups of sum S + 1 during sum S's inverse.
//
// Bound: VALU issue.  N = 2048, l = 3: 3.2k VALU instructions per wave and
// step (9.3k with modular transforms), 1536 ciphertexts 62.0 ms against 96
// ms; two workgroups share a CU (77 KB of LDS, 256 registers) and the
// VALU issues 60 % of the time (21.4k clocks of a CU per step, against 34k
// for a workgroup alone); without the key loads (a build that
// computes something else) the step is 20 % shorter, with all keys in the L2
// 3 %.  The lane swaps between the (7,6) and (5,4) passes beat a third
// exchange through LDS by 3 %; two sums side by side, or products and inverse
// one after the other, were 10 % slower (spills; waits nothing fills).
template <class F, int L, int P, typename RT>
__global__ void __launch_bounds__(F::T) __attribute__((amdgpu_waves_per_eu(2, 2)))
k_blind_rotate_fft(const u64 *__restrict__ lwe_in, const cd *__restrict__ key,
                   const u64 *__restrict__ lut, u64 *__restrict__ out, int n, int beta, int mode,
                   int tp_glwe, const cd *__restrict__ fft_tab) {
  constexpr int N = F::N, C = F::C, T = F::T;
  // (table first: its words and most of the buffer's are then within the 16
  // bits of an LDS instruction's offset)
  cd *tab = (cd *)fft_lds;
  cd *buf = tab + F::TABLE_BYTES / 16;
  uint16_t *rot = (uint16_t *)(buf + fft_buf_words<F, L>());
  const int tid = threadIdx.x;
  const FftLane<F::TABLE_BYTES> ln(tid);
  const size_t ct = blockIdx.x;

  const u64 *lwe = lwe_in + (ct / (size_t)(tp_glwe > 1 ? tp_glwe : 1)) * (size_t)(n + 1);
  for (int i = tid; i <= n; i += T) rot[i] = (uint16_t)gl_modswitch(lwe[i], F::LOGN);
  for (int i = tid; i < F::TABLE; i += T) tab[i] = fft_tab[i];
  __syncthreads();

  u64 acc[2][8];
  {
    const int r = (2 * N - (int)rot[n]) & (2 * N - 1);  // X^(-b~)
    const u64 *tpA = lut + (tp_glwe ? ct * (size_t)(2 * N) : 0);
    const u64 *tpB = tp_glwe ? tpA + N : lut;
#pragma unroll
    for (int k = 0; k < 8; ++k) {
      acc[0][k] = tp_glwe ? rotated_coef<N>(tpA, tid + T * k, r) : 0;
      acc[1][k] = rotated_coef<N>(tpB, tid + T * k, r);
    }
  }

  const int s = 64 - L * beta;
  const RT half = (RT)1 << (beta - 1);
  const int dsh = (int)(8 * sizeof(RT)) - beta;
  constexpr size_t step_words = (size_t)2 * P * 2 * L * C;
  constexpr int ROWS = 2 * L, SUMS = 2 * P;
  // a multiple of the ring per step keeps its places compile-time constants
  constexpr int PD = key_ahead<L>(), NB = sums_at_once<L>();
  static_assert((SUMS * ROWS) % PD == 0, "whole turns of the ring");
  constexpr bool PARK = L == 3;
  // ring of key groups (a sum's row), loaded PD ahead of their use
  cd q[PD][4];
  {
    const ExpandedRows G(key);
#pragma unroll
    for (int g = 0; g < PD; ++g)
#pragma unroll
      for (int k = 0; k < 4; ++k) q[g][k] = G.load(tid * 16, (g * C + k * T) * 16);
  }
#pragma unroll 1
  for (int i = 0; i < n; ++i) {
    const int a = __builtin_amdgcn_readfirstlane(rot[i]);
    const int ar = a & (N - 1);
    const bool flip = a >= N;
    // a2: rotate-subtract, both components
    u64 d[2][8];
    {
      u64 *w = (u64 *)buf;
      __syncthreads();
#pragma unroll
      for (int u = 0; u < 2; ++u)
#pragma unroll
        for (int k = 0; k < 8; ++k) w[u * N + tid + T * k] = acc[u][k];
      __syncthreads();
#pragma unroll
      for (int u = 0; u < 2; ++u)
#pragma unroll
        for (int k = 0; k < 8; ++k) d[u][k] = w[u * N + ((tid + T * k - ar) & (N - 1))];
    }
    // a3: rounding of component u, its digits of level t
    RT R[2][8];
    cd D[2][L][4];
    auto round = [&](int u) {
#pragma unroll
      for (int k = 0; k < 8; ++k) {
        const bool neg = (tid + T * k < ar) != flip;
        const u64 v = gl_sub(neg ? GL_P - d[u][k] : d[u][k], acc[u][k]);
        if constexpr (sizeof(RT) == 4)
          R[u][k] = gl_round_top32(v, s);
        else
          R[u][k] = gl_round_top(v, s);
      }
    };
    auto digits = [&](int u, int t) {
#pragma unroll
      for (int k = 0; k < 4; ++k) {
        int32_t e[2];
#pragma unroll
        for (int h = 0; h < 2; ++h) {
          RT &r = R[u][k + 4 * h];
          if (t == 0) {
            e[h] = (int32_t)r;
          } else {
            e[h] = (int32_t)((RT)((std::make_unsigned_t<RT>)r << dsh) >> dsh);
            r = (r + half) >> beta;
          }
        }
        D[u][t][k] = cd{(double)e[0], (double)e[1]};
      }
    };
    // a5: group g (sum g / ROWS, row g % ROWS) into its sum
    cd Y[2][NB][4];
    const ExpandedRows G(key + (size_t)i * step_words);
    auto group = [&](auto gc) {
      constexpr int g = decltype(gc)::value;
      constexpr int r = g % ROWS, sum = g / ROWS;
      cd(&y)[4] = Y[(sum / NB) & 1][sum % NB];
#pragma unroll
      for (int k = 0; k < 4; ++k) {
        const cd w = q[g % PD][k];
        const cd x = D[r / L][r % L][k];
        if (r == 0) {
          y[k].re = __builtin_fma(-x.im, w.im, x.re * w.re);
          y[k].im = __builtin_fma(x.im, w.re, x.re * w.im);
        } else {
          y[k].re = __builtin_fma(-x.im, w.im, __builtin_fma(x.re, w.re, y[k].re));
          y[k].im = __builtin_fma(x.im, w.re, __builtin_fma(x.re, w.im, y[k].im));
        }
      }
#pragma unroll
      for (int k = 0; k < 4; ++k) q[g % PD][k] = G.load(tid * 16, ((g + PD) * C + k * T) * 16);
      __builtin_amdgcn_sched_barrier(0);
    };
    // share h of `of` of the groups [g0, g0 + cnt)
    auto groups = [&](auto g0, auto cnt, auto h, auto of) {
      constexpr int b = decltype(cnt)::value * decltype(h)::value / decltype(of)::value;
      constexpr int e = decltype(cnt)::value * (decltype(h)::value + 1) / decltype(of)::value;
      static_for<decltype(g0)::value + b, decltype(g0)::value + e>(group);
    };
    // a4; while component 0 is transformed, component 1 is cut into digits,
    // while component 1 is, the first sum takes component 0's rows
    round(0);
#pragma unroll
    for (int t = L - 1; t >= 0; --t) digits(0, t);
    fft_forward<F, L, 0>(D[0], ln, [&](auto h) {
      constexpr int H = decltype(h)::value;
      if constexpr (H == 0) round(1);
      else if constexpr (H <= L) digits(1, L - H);
    });
    fft_forward<F, L, 0>(D[1], ln, [&](auto h) {
      groups(std::integral_constant<int, 0>{}, std::integral_constant<int, L>{}, h,
             std::integral_constant<int, F::FWD_HOOKS>{});
    });
    static_for<L, NB * ROWS>(group);
    // Three levels leave no registers for both components of the accumulator
    // next to three key groups in flight: the one whose sums are not being
    // taken back waits in the wave's own block of the buffer's third part,
    // which only the forward transforms use.
    auto put = [&](int c) {
#pragma unroll
      for (int k = 0; k < 4; ++k)
        fft_put(ln.own, 16 * (2 * C + 64 * k),
                cd{__longlong_as_double((long long)acc[c][2 * k]),
                   __longlong_as_double((long long)acc[c][2 * k + 1])});
    };
    auto get = [&](int c) {
#pragma unroll
      for (int k = 0; k < 4; ++k) {
        const cd v = fft_get(ln.own, 16 * (2 * C + 64 * k));
        acc[c][2 * k] = (u64)__double_as_longlong(v.re);
        acc[c][2 * k + 1] = (u64)__double_as_longlong(v.im);
      }
    };
    if constexpr (PARK) put(1);
    // a6: NB sums go back to coefficients while the next ones' groups are
    // added up
    u32 top[8];
    static_for<0, SUMS / NB>([&](auto bc) {
      constexpr int B = decltype(bc)::value;
      cd(&y)[NB][4] = Y[B & 1];
      // The wave's own blocks first.  One sum: in odd LOGC the same words
      // again, read by the others before the barrier of the last exchange (in
      // O2); in even LOGC two sets of words in turn, the others' last reads of
      // one lie before the barrier of the other.  Two sums: one set of words,
      // which a barrier opens again.
      constexpr bool ONE = NB > 1;
      constexpr int O1 = F::ODD || ONE ? 0 : (B & 1) * C, O2 = ONE ? 0 : C;
      fft_inverse<F, NB, 0, O1, O2, ONE && (B > 0)>(y, ln, [&](auto h) {
        if constexpr (B + 1 < SUMS / NB)
          groups(std::integral_constant<int, (B + 1) * NB * ROWS>{},
                 std::integral_constant<int, NB * ROWS>{}, h,
                 std::integral_constant<int, F::INV_HOOKS>{});
      });
      static_for<0, NB>([&](auto jc) {
        constexpr int j = decltype(jc)::value, S = B * NB + j, c = S / P, p = S % P;
#pragma unroll
        for (int k = 0; k < 4; ++k) {
          add_piece<P, p>(acc[c][k], top[k], y[j][k].re);
          add_piece<P, p>(acc[c][k + 4], top[k + 4], y[j][k].im);
        }
        if constexpr (p == P - 1) {
#pragma unroll
          for (int k = 0; k < 8; ++k) acc[c][k] = finish_pieces(acc[c][k], top[k]);
          if constexpr (PARK && c == 0) {
            get(1);
            put(0);
          } else if constexpr (PARK) {
            get(0);
          }
        }
      });
    });
  }

  if (mode == BR_GLWE) {
    u64 *o = out + ct * (size_t)(2 * N);
#pragma unroll
    for (int k = 0; k < 8; ++k) {
      o[tid + T * k] = acc[0][k];
      o[N + tid + T * k] = acc[1][k];
    }
  } else {
    // a7: sample extraction  a'_0 = A_0, a'_j = -A_{N-j}, b' = B_0
    u64 *o = out + ct * (size_t)(N + 1);
#pragma unroll
    for (int k = 0; k < 8; ++k) {
      const int j = tid + T * k;
      o[(N - j) & (N - 1)] = j ? gl_neg(acc[0][k]) : acc[0][k];
      if (j == 0) o[N] = acc[1][k];
    }
  }
}

// ---------------------------------------------------------------------------
// Trace
// ---------------------------------------------------------------------------

// Digit polynomials transformed side by side: two at a time where there are
// four, so that two workgroups' buffers fit a CU's LDS.
template <int L>
constexpr int trace_batch() {
  return L == 4 ? 2 : L;
}
template <class F, int L>
constexpr size_t trace_fft_lds_bytes() {
  return F::TABLE_BYTES + (size_t)(trace_batch<L>() > 2 ? trace_batch<L>() : 2) * F::C * sizeof(cd);
}

// The rounds of k_trace (kernels.hip) with the machinery of
// k_blind_rotate_fft: the L digit polynomials of tau_d(A), the 2P sums over
// their rows (the expanded key carries the minus sign of the key switch),
// taken back one after the other while the next is added up.
// Bound as there: VALU issue, and the waits of eight inverse transforms a
// round with less to fill them (4 rows a sum).  14336 traces at N = 2048, 4 x
// 12 bits (4 pieces): 6.0 ms (6.1 with one sum at a time), 7.5 ms with modular
// transforms; 3 x 10 bits (3 pieces) 4.3 against 6.2, N = 4096 15.5 against
// 24.1 ms; one trace 167 against 258 us.
template <class F, int L, int P>
__global__ void __launch_bounds__(F::T) __attribute__((amdgpu_waves_per_eu(2, 2)))
k_trace_fft(const u64 *__restrict__ in, const cd *__restrict__ key, u64 *__restrict__ out,
            int beta, u64 ninv, const cd *__restrict__ fft_tab) {
  constexpr int N = F::N, C = F::C, T = F::T;
  cd *tab = (cd *)fft_lds;
  u64 *w = (u64 *)(tab + F::TABLE_BYTES / 16);
  const int tid = threadIdx.x;
  const FftLane<F::TABLE_BYTES> ln(tid);
  const size_t ct = blockIdx.x;
  for (int i = tid; i < F::TABLE; i += T) tab[i] = fft_tab[i];

  u64 acc[2][8];
#pragma unroll
  for (int c = 0; c < 2; ++c)
#pragma unroll
    for (int k = 0; k < 8; ++k) acc[c][k] = gl_mul(in[(ct * 2 + c) * N + tid + T * k], ninv);

  const int s = 64 - L * beta;
  const i64 half = (i64)1 << (beta - 1);
  const int dsh = 64 - beta;
  constexpr int SUMS = 2 * P, GROUPS = SUMS * L, FB = trace_batch<L>();
  constexpr int NB = 2, PD = 2;  // sums side by side, key groups in flight
  static_assert(GROUPS % PD == 0 && L % FB == 0, "whole turns of the ring, whole batches");
  constexpr size_t round_words = (size_t)GROUPS * C;
  cd q[PD][4];
  {
    const ExpandedRows G(key + (F::LOGN - 1) * round_words);
#pragma unroll
    for (int g = 0; g < PD; ++g)
#pragma unroll
      for (int k = 0; k < 4; ++k) q[g][k] = G.load(tid * 16, (g * C + k * T) * 16);
  }
#pragma unroll 1
  for (int kr = F::LOGN; kr >= 1; --kr) {
    const u32 dinv = odd_inverse_mod((1u << kr) + 1, 2 * N);
    cd D[L / FB][FB][4];
    {
      __syncthreads();
#pragma unroll
      for (int c = 0; c < 2; ++c)
#pragma unroll
        for (int k = 0; k < 8; ++k) w[c * N + tid + T * k] = acc[c][k];
      __syncthreads();
      i64 R[8];
#pragma unroll
      for (int k = 0; k < 8; ++k) R[k] = gl_round_top(automorphism_coef<N>(w, tid + T * k, dinv), s);
#pragma unroll
      for (int k = 0; k < 8; ++k)
        acc[1][k] = gl_add(acc[1][k], automorphism_coef<N>(w + N, tid + T * k, dinv));
#pragma unroll
      for (int t = L - 1; t >= 0; --t)
#pragma unroll
        for (int k = 0; k < 4; ++k) {
          int32_t e[2];
#pragma unroll
          for (int h = 0; h < 2; ++h) {
            i64 &r = R[k + 4 * h];
            if (t == 0) {
              e[h] = (int32_t)r;
            } else {
              e[h] = (int32_t)((i64)((u64)r << dsh) >> dsh);
              r = (r + half) >> beta;
            }
          }
          D[t / FB][t % FB][k] = cd{(double)e[0], (double)e[1]};
        }
    }
    cd Y[2][NB][4];
    const ExpandedRows G(key + (kr - 1) * round_words);
    // the groups loaded past this round's belong to the next one's
    const ExpandedRows Gn(key + (kr > 1 ? kr - 2 : 0) * round_words);
    auto group = [&](auto gc) {
      constexpr int g = decltype(gc)::value, r = g % L, nx = g + PD;
      cd(&y)[4] = Y[(g / L / NB) & 1][g / L % NB];
#pragma unroll
      for (int k = 0; k < 4; ++k) {
        const cd z = q[g % PD][k];
        const cd x = D[r / FB][r % FB][k];
        if (r == 0) {
          y[k].re = __builtin_fma(-x.im, z.im, x.re * z.re);
          y[k].im = __builtin_fma(x.im, z.re, x.re * z.im);
        } else {
          y[k].re = __builtin_fma(-x.im, z.im, __builtin_fma(x.re, z.re, y[k].re));
          y[k].im = __builtin_fma(x.im, z.re, __builtin_fma(x.re, z.im, y[k].im));
        }
      }
#pragma unroll
      for (int k = 0; k < 4; ++k)
        q[g % PD][k] = (nx < GROUPS ? G : Gn).load(tid * 16, ((nx % GROUPS) * C + k * T) * 16);
      __builtin_amdgcn_sched_barrier(0);
    };
    fft_forward<F, FB, 0>(D[0], ln, NoHook{});
    if constexpr (FB < L) {
      fft_forward<F, FB, 0>(D[1], ln, [&](auto h) {
        constexpr int H = decltype(h)::value, HN = F::FWD_HOOKS;
        static_for<FB * H / HN, FB * (H + 1) / HN>(group);
      });
      static_for<FB, NB * L>(group);
    } else {
      static_for<0, NB * L>(group);
    }
    u32 top[8];
    static_for<0, SUMS / NB>([&](auto bc) {
      constexpr int B = decltype(bc)::value;
      cd(&y)[NB][4] = Y[B & 1];
      // (NB sums leave room for one set of words: a barrier opens it again)
      constexpr bool ONE = NB > 1;
      constexpr int O1 = F::ODD || ONE ? 0 : (B & 1) * C, O2 = ONE ? 0 : C;
      fft_inverse<F, NB, 0, O1, O2, ONE && (B > 0)>(y, ln, [&](auto h) {
        if constexpr (B + 1 < SUMS / NB) {
          constexpr int H = decltype(h)::value, HN = F::INV_HOOKS, M = NB * L;
          static_for<(B + 1) * M + M * H / HN, (B + 1) * M + M * (H + 1) / HN>(group);
        }
      });
      static_for<0, NB>([&](auto jc) {
        constexpr int j = decltype(jc)::value, S = B * NB + j, c = S / P, p = S % P;
#pragma unroll
        for (int k = 0; k < 4; ++k) {
          add_piece<P, p>(acc[c][k], top[k], y[j][k].re);
          add_piece<P, p>(acc[c][k + 4], top[k + 4], y[j][k].im);
        }
        if constexpr (p == P - 1) {
#pragma unroll
          for (int k = 0; k < 8; ++k) acc[c][k] = finish_pieces(acc[c][k], top[k]);
        }
      });
    });
  }
#pragma unroll
  for (int c = 0; c < 2; ++c)
#pragma unroll
    for (int k = 0; k < 8; ++k) out[(ct * 2 + c) * N + tid + T * k] = acc[c][k];
}

// ---------------------------------------------------------------------------
// Launch
// ---------------------------------------------------------------------------

namespace {

template <typename K>
hipError_t allow_lds(K kernel, size_t bytes) {
  if (bytes <= 65536) return hipSuccess;
  return hipFuncSetAttribute((const void *)kernel, hipFuncAttributeMaxDynamicSharedMemorySize,
                             (int)bytes);
}

// One workgroup per step shares the tables among its 2R rows; few steps take
// one per row.
dim3 expand_grid(unsigned steps, unsigned R) {
  return dim3(steps, steps < (unsigned)device_cus() ? 2 * R : 1);
}

template <class S, class F, int L, int P, typename RT>
hipError_t launch_fft(const uint64_t *lwe_in, const uint64_t *bsk_dev, const uint64_t *lut,
                      uint64_t *out, size_t batch, const rosetta_params &p, const Tables &tb,
                      int mode, int tp_glwe, cd *key, hipStream_t st) {
  const size_t xlds = F::TABLE_BYTES + (size_t)(S::TW_WORDS + S::XCHG_WORDS) * 8;
  static_assert(br_fft_lds_bytes<F, L>(MAX_LWE_N) <= LDS_PER_CU, "room at every n");
  const size_t lds = br_fft_lds_bytes<F, L>((int)p.n);
  hipError_t e;
  if ((e = allow_lds(k_expand_key<S, F, P>, xlds)) != hipSuccess) return e;
  hipLaunchKernelGGL((k_expand_key<S, F, P>), expand_grid(p.n, 2 * L), dim3(S::T), xlds, st, bsk_dev, key,
                     2 * L, 1.0 / F::C, tb.zeta, (const cd *)tb.fft);
  if ((e = allow_lds(k_blind_rotate_fft<F, L, P, RT>, lds)) != hipSuccess) return e;
  hipLaunchKernelGGL((k_blind_rotate_fft<F, L, P, RT>), dim3(batch), dim3(F::T), lds, st, lwe_in,
                     key, lut, out, (int)p.n, (int)p.pbs_base_log, mode, tp_glwe,
                     (const cd *)tb.fft);
  return hipGetLastError();
}

template <class S, class F, int L>
hipError_t launch_fft_pieces(const uint64_t *lwe_in, const uint64_t *bsk_dev, const uint64_t *lut,
                             uint64_t *out, size_t batch, const rosetta_params &p,
                             const Tables &tb, int mode, int tp_glwe, cd *key, hipStream_t st) {
  if (fft_pieces(p) == 3)
    return launch_fft<S, F, L, 3, int32_t>(lwe_in, bsk_dev, lut, out, batch, p, tb, mode, tp_glwe,
                                           key, st);
  return launch_fft<S, F, L, 4, int64_t>(lwe_in, bsk_dev, lut, out, batch, p, tb, mode, tp_glwe,
                                         key, st);
}

template <int LOGN>
hipError_t launch_fft_levels(const uint64_t *lwe_in, const uint64_t *bsk_dev, const uint64_t *lut,
                             uint64_t *out, size_t batch, const rosetta_params &p,
                             const Tables &tb, int mode, int tp_glwe, cd *key, hipStream_t st) {
  using S = Ntt<LOGN, ntt_le(LOGN), ntt_first(LOGN)>;
  using F = Fft<LOGN>;
  switch (p.pbs_level) {
    case 1: return launch_fft_pieces<S, F, 1>(lwe_in, bsk_dev, lut, out, batch, p, tb, mode, tp_glwe, key, st);
    case 2: return launch_fft_pieces<S, F, 2>(lwe_in, bsk_dev, lut, out, batch, p, tb, mode, tp_glwe, key, st);
    default: return launch_fft_pieces<S, F, 3>(lwe_in, bsk_dev, lut, out, batch, p, tb, mode, tp_glwe, key, st);
  }
}

template <int LOGN, int L, int P>
hipError_t launch_trace_fft(const uint64_t *in, const uint64_t *autk_dev, uint64_t *out,
                            size_t batch, int base_log, const Tables &tb, cd *key,
                            hipStream_t st) {
  using S = Ntt<LOGN, ntt_le(LOGN), ntt_first(LOGN)>;
  using F = Fft<LOGN>;
  const size_t xlds = F::TABLE_BYTES + (size_t)(S::TW_WORDS + S::XCHG_WORDS) * 8;
  const size_t lds = trace_fft_lds_bytes<F, L>();
  hipError_t e;
  if ((e = allow_lds(k_expand_key<S, F, P>, xlds)) != hipSuccess) return e;
  if ((e = allow_lds(k_trace_fft<F, L, P>, lds)) != hipSuccess) return e;
  hipLaunchKernelGGL((k_expand_key<S, F, P>), expand_grid(LOGN, L), dim3(S::T), xlds, st, autk_dev, key, L,
                     -1.0 / F::C, tb.zeta, (const cd *)tb.fft);
  hipLaunchKernelGGL((k_trace_fft<F, L, P>), dim3(batch), dim3(F::T), lds, st, in, key, out,
                     base_log, tb.ninv, (const cd *)tb.fft);
  return hipGetLastError();
}

template <int LOGN, int L>
hipError_t launch_trace_pieces(const uint64_t *in, const uint64_t *autk_dev, uint64_t *out,
                               size_t batch, int base_log, int pieces, const Tables &tb, cd *key,
                               hipStream_t st) {
  return pieces == 3 ? launch_trace_fft<LOGN, L, 3>(in, autk_dev, out, batch, base_log, tb, key, st)
                     : launch_trace_fft<LOGN, L, 4>(in, autk_dev, out, batch, base_log, tb, key, st);
}

template <int LOGN>
hipError_t launch_trace_levels(const uint64_t *in, const uint64_t *autk_dev, uint64_t *out,
                               size_t batch, int level, int base_log, int pieces,
                               const Tables &tb, cd *key, hipStream_t st) {
  switch (level) {
    case 1: return launch_trace_pieces<LOGN, 1>(in, autk_dev, out, batch, base_log, pieces, tb, key, st);
    case 2: return launch_trace_pieces<LOGN, 2>(in, autk_dev, out, batch, base_log, pieces, tb, key, st);
    case 3: return launch_trace_pieces<LOGN, 3>(in, autk_dev, out, batch, base_log, pieces, tb, key, st);
    default: return launch_trace_pieces<LOGN, 4>(in, autk_dev, out, batch, base_log, pieces, tb, key, st);
  }
}

}  // namespace

hipError_t launch_blind_rotate(const uint64_t *lwe_in, const uint64_t *bsk_dev,
                               const uint64_t *lut, uint64_t *out, size_t batch,
                               const rosetta_params &p, const Tables &tb, BrMode mode,
                               int tp_glwe, bool may_allocate, hipStream_t st) {
  const int pieces = may_allocate ? fft_pieces(p) : 0;
  if (pieces) {
    // (one step more: the key stream is loaded ahead of its use)
    const size_t bytes =
        ((size_t)p.n + 1) * 2 * pieces * 2 * p.pbs_level * (p.N / 2) * sizeof(cd);
    if (void *key = scratch_take(bytes, st)) {
      const hipError_t e = p.N == 2048
                               ? launch_fft_levels<11>(lwe_in, bsk_dev, lut, out, batch, p, tb,
                                                       (int)mode, tp_glwe, (cd *)key, st)
                               : launch_fft_levels<12>(lwe_in, bsk_dev, lut, out, batch, p, tb,
                                                       (int)mode, tp_glwe, (cd *)key, st);
      const hipError_t f = scratch_give(key, st);
      return e != hipSuccess ? e : f;
    }
    // the modular transforms need no expanded key
  }
  return launch_blind_rotate_ntt(lwe_in, bsk_dev, lut, out, batch, p, tb, mode, tp_glwe, st);
}

hipError_t launch_trace(const uint64_t *in, const uint64_t *autk_dev, uint64_t *out,
                        size_t batch, uint32_t N, int level, int base_log, const Tables &tb,
                        hipStream_t st) {
  const int pieces =
      trace_pieces(N, (unsigned)level, (unsigned)base_log, batch, (size_t)device_cus());
  if (pieces) {
    const size_t rounds = N == 2048 ? 11 : 12;
    if (void *key = scratch_take(rounds * 2 * pieces * level * (N / 2) * sizeof(cd), st)) {
      const hipError_t e = N == 2048 ? launch_trace_levels<11>(in, autk_dev, out, batch, level,
                                                               base_log, pieces, tb, (cd *)key, st)
                                     : launch_trace_levels<12>(in, autk_dev, out, batch, level,
                                                               base_log, pieces, tb, (cd *)key, st);
      const hipError_t f = scratch_give(key, st);
      return e != hipSuccess ? e : f;
    }
  }
  return launch_trace_ntt(in, autk_dev, out, batch, N, level, base_log, tb, st);
}

}  // namespace rosetta
