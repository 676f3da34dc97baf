// Negacyclic transform of real polynomials in double precision, held in
// registers by one workgroup.
//
// A real polynomial y of N coefficients modulo X^N + 1 folds into the complex
// polynomial z_j = y_j + i y_(j+N/2) of C = N/2 coefficients modulo X^C - i
// (X^C = i satisfies X^N = -1), and products carry over.  T = C / 4 threads
// hold 4 complex coefficients each; natural layout: slot k of thread t holds
// z_(t + T k), i.e. y_(t + T k) and y_(t + T (k + 4)), which is the natural
// layout of the modular transforms (ntt.hpp) with 8 coefficients per thread.
//
// Forward: stage s splits each block modulo X^(2m) - theta into X^m -+ sqrt
// theta by butterflies (u + w v, u - w v), w = sqrt theta.  With angles in
// turns, block b of stage s (b's bits are the choices so far, the first one
// on top) has theta = e(phi), phi(s, b) = 2^-(s+2) + rev_s(b) / 2^s, so the
// twiddle depends on the block alone.  Two stages make a radix-4 pass with
// the twiddles a = e(phi / 2) and b = e(phi / 4) (the second block's second
// twiddle is i b).  The sum costs two fused multiply-adds per component and
// the difference one, 2u - (u + w v): 6 instructions per butterfly and no
// separate products.
//
// Inverse: position j holds the value at e(2^-(LOGC+2) + rev(j) / C), so
//   z_n = e(-n / 4C) (1/C) sum_r value_(rev r) e(-n r / C):
// the textbook decimation in time from bit-reversed order (twiddles that
// depend on the position inside the block, in the same 6-instruction
// butterfly; the first stage pair needs none) and one product per point by
// e(-n / 4C) at the end.  1/C is folded into the key's transform.
//
// Index bits of a pass: F (first) covers the top bit (odd LOGC) or two bits;
// the others two bits each down to (1, 0).  From pass (7, 6) on, wave w holds
// the 256 indices w 2^8 .. w 2^8 + 255, so the exchanges between those passes
// stay inside the wave: (7,6) to (5,4) trades the slot bits with lane bits 5
// and 4 by lane swaps (v_permlane32_swap, v_permlane16_swap: no LDS), the
// other two go through the wave's own block of the LDS buffer in an order
// that keeps the 16-byte words of any 16 consecutive lanes on distinct banks.
#pragma once

#include "gl.hpp"
#include "ntt.hpp"

namespace rosetta {

struct alignas(16) cd {
  double re, im;
};

template <int LOGN_>
struct Fft {
  static constexpr int LOGN = LOGN_;
  static constexpr int N = 1 << LOGN;
  static constexpr int LOGC = LOGN - 1;
  static constexpr int C = 1 << LOGC;
  static constexpr int T = C / 4;
  static constexpr bool ODD = (LOGC & 1) != 0;
  static_assert(LOGC >= 10, "at least two passes across waves");
  // Table (cd words): forward pass s (its first stage) holds a, then b, of
  // its 2^s blocks; inverse pass q (its lower index bit) v^2, then v =
  // e(-k / 2^(q+2)), of its 2^q positions; then, for odd LOGC, the last
  // inverse stage's e(-t / C) for t < T, and e(-t / 4C) for t < T.
  // Forward passes with tables start at stage 1, 3, .. (odd) or 2, 4, ..
  static constexpr int S0 = ODD ? 1 : 2;
  __host__ __device__ static constexpr int fwd_at(int s) {
    int o = 0;
    for (int i = S0; i < s; i += 2) o += 2 << i;
    return o;
  }
  __host__ __device__ static constexpr int inv_at(int q) {
    int o = fwd_at(LOGC);
    for (int i = 2; i < q; i += 2) o += 2 << i;
    return o;
  }
  static constexpr int Q_END = ODD ? LOGC - 1 : LOGC;  // inverse radix-4 passes: q < Q_END
  static constexpr int LAST_AT = inv_at(Q_END);
  static constexpr int TWIST_AT = LAST_AT + (ODD ? T : 0);
  static constexpr int TABLE = TWIST_AT + T;
  static constexpr int TABLE_BYTES = (TABLE * 16 + 255) / 256 * 256;  // (XORs below bit 8)
  // places where a forward / inverse transform calls its hook
  static constexpr int FWD_HOOKS = ODD ? 6 : 4, INV_HOOKS = ODD ? 6 : 4;
};

// (u, v) -> (u + w v, u - w v)
__device__ __forceinline__ void fft_bfly(cd &u, cd &v, double wr, double wi) {
  const double sr = __builtin_fma(wr, v.re, __builtin_fma(-wi, v.im, u.re));
  const double si = __builtin_fma(wr, v.im, __builtin_fma(wi, v.re, u.im));
  v.re = __builtin_fma(2.0, u.re, -sr);
  v.im = __builtin_fma(2.0, u.im, -si);
  u.re = sr;
  u.im = si;
}
__device__ __forceinline__ cd fft_mul(cd x, cd w) {
  return cd{__builtin_fma(x.re, w.re, -(x.im * w.im)), __builtin_fma(x.re, w.im, x.im * w.re)};
}

__device__ __forceinline__ void fft_fwd4(cd (&x)[4], cd a, cd b) {
  fft_bfly(x[0], x[2], a.re, a.im);
  fft_bfly(x[1], x[3], a.re, a.im);
  fft_bfly(x[0], x[1], b.re, b.im);
  fft_bfly(x[2], x[3], -b.im, b.re);
}
// slot bit 0 is the lower index bit: pairs (0,1), (2,3) first
__device__ __forceinline__ void fft_inv4(cd (&x)[4], cd a, cd v) {
  fft_bfly(x[0], x[1], a.re, a.im);
  fft_bfly(x[2], x[3], a.re, a.im);
  fft_bfly(x[0], x[2], v.re, v.im);
  fft_bfly(x[1], x[3], v.im, -v.re);
}
// fft_inv4 with both twiddles 1
__device__ __forceinline__ void fft_inv4_first(cd (&x)[4]) {
  const cd p = {x[0].re + x[1].re, x[0].im + x[1].im}, m = {x[0].re - x[1].re, x[0].im - x[1].im};
  const cd q = {x[2].re + x[3].re, x[2].im + x[3].im}, r = {x[2].re - x[3].re, x[2].im - x[3].im};
  x[0] = cd{p.re + q.re, p.im + q.im};
  x[2] = cd{p.re - q.re, p.im - q.im};
  x[1] = cd{m.re + r.im, m.im - r.re};  // m - i r
  x[3] = cd{m.re - r.im, m.im + r.re};
}

// Trade slot bit 1 with lane bit 5 and slot bit 0 with lane bit 4.
__device__ __forceinline__ void swap32(double &a, double &b) {
  u64 x = (u64)__double_as_longlong(a), y = (u64)__double_as_longlong(b);
  const auto lo = __builtin_amdgcn_permlane32_swap((u32)x, (u32)y, false, false);
  const auto hi = __builtin_amdgcn_permlane32_swap((u32)(x >> 32), (u32)(y >> 32), false, false);
  a = __longlong_as_double((long long)gl_mk(lo[0], hi[0]));
  b = __longlong_as_double((long long)gl_mk(lo[1], hi[1]));
}
__device__ __forceinline__ void swap16(double &a, double &b) {
  u64 x = (u64)__double_as_longlong(a), y = (u64)__double_as_longlong(b);
  const auto lo = __builtin_amdgcn_permlane16_swap((u32)x, (u32)y, false, false);
  const auto hi = __builtin_amdgcn_permlane16_swap((u32)(x >> 32), (u32)(y >> 32), false, false);
  a = __longlong_as_double((long long)gl_mk(lo[0], hi[0]));
  b = __longlong_as_double((long long)gl_mk(lo[1], hi[1]));
}
__device__ __forceinline__ void fft_lane_swap(cd (&x)[4]) {
  swap32(x[0].re, x[2].re);
  swap32(x[0].im, x[2].im);
  swap32(x[1].re, x[3].re);
  swap32(x[1].im, x[3].im);
  swap16(x[0].re, x[1].re);
  swap16(x[0].im, x[1].im);
  swap16(x[2].re, x[3].re);
  swap16(x[2].im, x[3].im);
}

// Exchanges inside the wave's own 256-word block.  The lane holds, in its
// lane bits (5,4), (3,2), (1,0), index bits (5,4),(3,2),(1,0) in the layout
// with slot bits (7,6), and (7,6),(3,2),(1,0) / (7,6),(5,4),(1,0) /
// (7,6),(5,4),(3,2) in those with slot bits (5,4) / (3,2) / (1,0).  Index e
// goes to word e between the first two; to e76 64 + e54 16 + (e32 ^ e54) 4 +
// e10 between the next two; to e76 64 + e32 16 + e54 4 + (e32 ^ e10) between
// the last two: any 16 consecutive lanes touch 16 distinct words modulo 16 on
// both sides.  With lane bits (g, h, w) that is word g 64 + 4 h + w, that + 16
// h, or that + 16 w, XOR a constant of the slot and plus another.  FftLane
// keeps the three as byte offsets (own block included).
template <int BUF>
struct FftLane {
  int t16, nat, own, base, plus_h, plus_w;
  __device__ __forceinline__ explicit FftLane(int tid) {
    const int l = tid & 63, h = (l >> 2) & 3, w = l & 3, blk = (tid >> 6) * 256;
    t16 = tid * 16;
    nat = BUF + t16;
    own = BUF + (blk + l) * 16;
    base = BUF + (blk + (l >> 4) * 64 + 4 * h + w) * 16;
    plus_h = base + 16 * 16 * h;
    plus_w = base + 16 * 16 * w;
  }
};
// LDS by byte address.  The kernels that use these have dynamic LDS only, so
// it starts at address 0 (test_code_objects_cpu.py holds the built library to
// that).  (Through pointers the base is added once per address, at run time.)
typedef double fft_v2 __attribute__((ext_vector_type(2)));
__device__ __forceinline__ cd fft_get(int at, int off) {
#if defined(__HIP_DEVICE_COMPILE__)
  typedef const fft_v2 __attribute__((address_space(3))) lds_v2;
  const fft_v2 v = *(lds_v2 *)(unsigned)(at + off);
  return cd{v.x, v.y};
#else
  return cd{0, 0};
#endif
}
__device__ __forceinline__ void fft_put(int at, int off, cd x) {
#if defined(__HIP_DEVICE_COMPILE__)
  typedef fft_v2 __attribute__((address_space(3))) lds_v2;
  *(lds_v2 *)(unsigned)(at + off) = fft_v2{x.re, x.im};
#endif
}
// v ^ c, v & c and v >> c as asm: out of reach of loop-invariant motion (what
// they would keep in registers all along is worth more than the instruction).
__device__ __forceinline__ int fft_xor(int v, int c) {
#if defined(__HIP_DEVICE_COMPILE__)
  int r;
  asm volatile("v_xor_b32 %0, %1, %2" : "=v"(r) : "s"(c), "v"(v));
  return r;
#else
  return v ^ c;
#endif
}
__device__ __forceinline__ int fft_and(int v, int c) {
#if defined(__HIP_DEVICE_COMPILE__)
  int r;
  asm volatile("v_and_b32 %0, %1, %2" : "=v"(r) : "s"(c), "v"(v));
  return r;
#else
  return v & c;
#endif
}
__device__ __forceinline__ int fft_shr(int v, int c) {
#if defined(__HIP_DEVICE_COMPILE__)
  int r;
  asm volatile("v_lshrrev_b32 %0, %1, %2" : "=v"(r) : "s"(c), "v"(v));
  return r;
#else
  return v >> c;
#endif
}
struct NoHook {
  template <class I>
  __device__ __forceinline__ void operator()(I) const {}
};
// Slot k's word in exchange X (1: (5,4)/(3,2), 2: (3,2)/(1,0)), on the side
// of the upper slot bits (UP) or the lower ones.
template <int X, bool UP, class Lane>
__device__ __forceinline__ int fft_word(const Lane &ln, int k) {
  const int o = UP ? ln.base : X == 1 ? ln.plus_h : ln.plus_w;
  return k > 0 ? fft_xor(o, 16 * (X == 1 ? 4 * k : k)) : o;
}
// The four slots' words on one side of an exchange, and one transform's data
// to and from there (words off .. of the buffer).
template <int X, bool UP>
struct FftWords {
  int w[4];
  template <class Lane>
  __device__ __forceinline__ explicit FftWords(const Lane &ln) {
#pragma unroll
    for (int k = 0; k < 4; ++k) w[k] = fft_word<X, UP>(ln, k);
  }
  __device__ __forceinline__ void put(const cd (&x)[4], int off) const {
#pragma unroll
    for (int k = 0; k < 4; ++k) fft_put(w[k], 16 * (off + (UP ? 16 * k : 0)), x[k]);
  }
  __device__ __forceinline__ void get(cd (&x)[4], int off) const {
#pragma unroll
    for (int k = 0; k < 4; ++k) x[k] = fft_get(w[k], 16 * (off + (UP ? 16 * k : 0)));
  }
};

// Layouts across waves: 0 the natural one (j = t + T k); 1 (odd LOGC) slot
// bits (9,8); 2 slot bits (7,6), the wave's own block.
template <class F, int LY, class Lane>
__device__ __forceinline__ int fft_at(const Lane &ln) {
  if (LY == 0) return ln.nat;
  if (LY == 1) return ln.nat + 16 * 768 * (ln.t16 >> 12);  // (t >> 8) 1024 + (t & 255)
  return ln.own;
}
template <class F, int LY>
constexpr int fft_step() {
  return LY == 0 ? F::T : LY == 1 ? 256 : 64;
}
template <class F, int LY, class Lane>
__device__ __forceinline__ void fft_put_cross(const cd (&x)[4], int off, const Lane &ln) {
#pragma unroll
  for (int k = 0; k < 4; ++k) fft_put(fft_at<F, LY>(ln), 16 * (off + k * fft_step<F, LY>()), x[k]);
}
template <class F, int LY, class Lane>
__device__ __forceinline__ void fft_get_cross(cd (&x)[4], int off, const Lane &ln) {
#pragma unroll
  for (int k = 0; k < 4; ++k) x[k] = fft_get(fft_at<F, LY>(ln), 16 * (off + k * fft_step<F, LY>()));
}

// cos, sin of 1/8 and 1/16 of a turn
constexpr double FFT_C8 = 0.70710678118654752440, FFT_C16 = 0.92387953251128675613,
                 FFT_S16 = 0.38268343236508977173;

// NB forward transforms side by side: natural layout in, slot bits (1,0) out.
// The table starts at byte TAB of the LDS, the buffer where ln says; the
// transforms use words [0, NB C) of it and start with a barrier.
// hook(0 .. HOOKS - 1) runs where the wave waits for the LDS or the others.
// Each transform is written as soon as its pass is done and the next one's
// pass follows, so that the LDS works while the VALU does.
template <class F, int NB, int TAB, class Lane, class Hook>
__device__ __forceinline__ void fft_forward(cd (&x)[NB][4], const Lane &ln, const Hook &hook) {
  constexpr int H0 = F::ODD ? 2 : 0, C = F::C;
  struct Tw {
    cd a, b;
  };
  auto twiddles = [&](int at, int stages, int block16) {
    return Tw{fft_get(block16, TAB + 16 * at), fft_get(block16, TAB + 16 * (at + (1 << stages)))};
  };
  auto first = [&](cd (&z)[4]) {
    if constexpr (F::ODD) {
      fft_bfly(z[0], z[2], FFT_C8, FFT_C8);
      fft_bfly(z[1], z[3], FFT_C8, FFT_C8);
    } else {
      fft_fwd4(z, cd{FFT_C8, FFT_C8}, cd{FFT_C16, FFT_S16});
    }
  };
  first(x[0]);
  __syncthreads();
  static_for<0, NB>([&](auto bc) {
    constexpr int b = decltype(bc)::value;
    if constexpr (b > 0) first(x[b]);
    fft_put_cross<F, 0>(x[b], b * C, ln);
  });
  hook(std::integral_constant<int, 0>{});
  __syncthreads();
  if constexpr (F::ODD) {
    const Tw w = twiddles(F::fwd_at(1), 1, fft_and(fft_shr(ln.t16, 8), ~15));
#pragma unroll
    for (int b = 0; b < NB; ++b) fft_get_cross<F, 1>(x[b], b * C, ln);
    hook(std::integral_constant<int, 1>{});
    fft_fwd4(x[0], w.a, w.b);
    __syncthreads();
    static_for<0, NB>([&](auto bc) {
      constexpr int b = decltype(bc)::value;
      if constexpr (b > 0) fft_fwd4(x[b], w.a, w.b);
      fft_put_cross<F, 1>(x[b], b * C, ln);
    });
    hook(std::integral_constant<int, 2>{});
    __syncthreads();
  }
  {
    const Tw w = twiddles(F::fwd_at(F::LOGC - 8), F::LOGC - 8, fft_and(fft_shr(ln.t16, 6), ~15));
    const Tw v = twiddles(F::fwd_at(F::LOGC - 6), F::LOGC - 6, fft_and(fft_shr(ln.t16, 4), ~15));
#pragma unroll
    for (int b = 0; b < NB; ++b) fft_get_cross<F, 2>(x[b], b * C, ln);
    hook(std::integral_constant<int, H0 + 1>{});
    const FftWords<1, true> up(ln);
#pragma unroll
    for (int b = 0; b < NB; ++b) {
      fft_fwd4(x[b], w.a, w.b);
      fft_lane_swap(x[b]);
      fft_fwd4(x[b], v.a, v.b);
      up.put(x[b], b * C);
    }
  }
  {
    const Tw w = twiddles(F::fwd_at(F::LOGC - 4), F::LOGC - 4, fft_and(fft_shr(ln.t16, 2), ~15));
    const FftWords<1, false> lo(ln);
    const FftWords<2, true> up(ln);
    wave_sync();
#pragma unroll
    for (int b = 0; b < NB; ++b) lo.get(x[b], b * C);
    hook(std::integral_constant<int, H0 + 2>{});
#pragma unroll
    for (int b = 0; b < NB; ++b) {
      fft_fwd4(x[b], w.a, w.b);
      up.put(x[b], b * C);
    }
  }
  const Tw w = twiddles(F::fwd_at(F::LOGC - 2), F::LOGC - 2, ln.t16);
  const FftWords<2, false> lo(ln);
  wave_sync();
#pragma unroll
  for (int b = 0; b < NB; ++b) lo.get(x[b], b * C);
  hook(std::integral_constant<int, H0 + 3>{});
#pragma unroll
  for (int b = 0; b < NB; ++b) fft_fwd4(x[b], w.a, w.b);
}

// NB inverse transforms (times C) side by side: slot bits (1,0) in, natural
// layout out.  They work in the wave's own blocks of words [O1, O1 + NB C) of
// the buffer, which nobody else may read any more (OPEN: a barrier first sees
// to that), write those once more, and read all of them after a barrier; for
// odd LOGC a second exchange goes through words [O2, O2 + NB C), which, unless
// they are the same, have to be free once that barrier is passed.
template <class F, int NB, int TAB, int O1, int O2, bool OPEN, class Lane, class Hook>
__device__ __forceinline__ void fft_inverse(cd (&x)[NB][4], const Lane &ln, const Hook &hook) {
  constexpr int H0 = F::ODD ? 6 : 4, C = F::C;
  struct Tw {
    cd a, v;
  };
  auto twiddles = [&](int at, int bits, int pos16) {
    return Tw{fft_get(pos16, TAB + 16 * at), fft_get(pos16, TAB + 16 * (at + (1 << bits)))};
  };
  fft_inv4_first(x[0]);
  if constexpr (OPEN) __syncthreads();
  {
    const FftWords<2, false> lo(ln);
    const FftWords<2, true> up(ln);
    static_for<0, NB>([&](auto bc) {
      constexpr int b = decltype(bc)::value;
      if constexpr (b > 0) fft_inv4_first(x[b]);
      lo.put(x[b], O1 + b * C);
    });
    const Tw w = twiddles(F::inv_at(2), 2, fft_and(ln.t16, 48));
    wave_sync();
#pragma unroll
    for (int b = 0; b < NB; ++b) up.get(x[b], O1 + b * C);
    hook(std::integral_constant<int, 0>{});
    const FftWords<1, false> lo1(ln);
#pragma unroll
    for (int b = 0; b < NB; ++b) {
      fft_inv4(x[b], w.a, w.v);
      lo1.put(x[b], O1 + b * C);
    }
  }
  {
    const FftWords<1, true> up(ln);
    const Tw w = twiddles(F::inv_at(4), 4, fft_and(ln.t16, 240));
    wave_sync();
#pragma unroll
    for (int b = 0; b < NB; ++b) up.get(x[b], O1 + b * C);
    hook(std::integral_constant<int, 1>{});
    const Tw v = twiddles(F::inv_at(6), 6, fft_and(ln.t16, 1008));
#pragma unroll
    for (int b = 0; b < NB; ++b) {
      fft_inv4(x[b], w.a, w.v);
      fft_lane_swap(x[b]);
      fft_inv4(x[b], v.a, v.v);
      fft_put_cross<F, 2>(x[b], O1 + b * C, ln);
    }
  }
  hook(std::integral_constant<int, 2>{});
  __syncthreads();
  if constexpr (F::ODD) {
    const Tw w = twiddles(F::inv_at(8), 8, fft_and(ln.t16, 4080));
#pragma unroll
    for (int b = 0; b < NB; ++b) fft_get_cross<F, 1>(x[b], O1 + b * C, ln);
    hook(std::integral_constant<int, 3>{});
    fft_inv4(x[0], w.a, w.v);
    if constexpr (O1 == O2) __syncthreads();
    static_for<0, NB>([&](auto bc) {
      constexpr int b = decltype(bc)::value;
      if constexpr (b > 0) fft_inv4(x[b], w.a, w.v);
      fft_put_cross<F, 1>(x[b], O2 + b * C, ln);
    });
    hook(std::integral_constant<int, 4>{});
    __syncthreads();
#pragma unroll
    for (int b = 0; b < NB; ++b) fft_get_cross<F, 0>(x[b], O2 + b * C, ln);
  } else {
#pragma unroll
    for (int b = 0; b < NB; ++b) fft_get_cross<F, 0>(x[b], O1 + b * C, ln);
  }
  hook(std::integral_constant<int, H0 - 1>{});
  if constexpr (F::ODD) {
    const cd w = fft_get(ln.t16, TAB + 16 * F::LAST_AT);
#pragma unroll
    for (int b = 0; b < NB; ++b) {
      fft_bfly(x[b][0], x[b][2], w.re, w.im);
      fft_bfly(x[b][1], x[b][3], w.im, -w.re);
    }
  } else {
    const Tw w = twiddles(F::inv_at(8), 8, ln.t16);
#pragma unroll
    for (int b = 0; b < NB; ++b) fft_inv4(x[b], w.a, w.v);
  }
  // e(-(t + T k) / 4C) = e(-t / 4C) e(-k / 16)
  const cd w0 = fft_get(ln.t16, TAB + 16 * F::TWIST_AT);
  const cd w1 = fft_mul(w0, cd{FFT_C16, -FFT_S16}), w2 = fft_mul(w0, cd{FFT_C8, -FFT_C8}),
           w3 = fft_mul(w0, cd{FFT_S16, -FFT_C16});
#pragma unroll
  for (int b = 0; b < NB; ++b) {
    x[b][0] = fft_mul(x[b][0], w0);
    x[b][1] = fft_mul(x[b][1], w1);
    x[b][2] = fft_mul(x[b][2], w2);
    x[b][3] = fft_mul(x[b][3], w3);
  }
}

}  // namespace rosetta
