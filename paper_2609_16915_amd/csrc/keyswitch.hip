// Key switching kernels (step a8) and the preparation of their key: the
// int8 matrix-core kernel for parameter sets whose digits fit a signed byte
// (ks_on_matrix_cores), the VALU kernel for the others.
//
// Kept apart from kernels.hip because they are compiled with the compiler's
// default instruction scheduling: both are streams of independent
// multiply-accumulates (matrix products, or 32x32-bit products into 64-bit
// accumulators), which the default occupancy-first schedule already
// interleaves, while the transform kernels are built with the ILP-first one.
#include <hip/hip_runtime.h>

#include "gl.hpp"
#include "internal.hpp"

namespace rosetta {

// Prepared key-switching key: the standard [N*l_ks][n+1] words followed by
// h * (sum over rows of column c), h = 2^(beta_ks - 1), for the offset-digit
// accumulation of k_keyswitch.
__global__ void k_ksk_colsum(const u64 *__restrict__ ksk, u64 *__restrict__ out, size_t rows,
                             int cols, u64 half) {
  const int c = blockIdx.x * blockDim.x + threadIdx.x;
  if (c >= cols) return;
  u64 s = 0;
  for (size_t r = 0; r < rows; ++r) s = gl_add(s, ksk[r * cols + c]);
  out[c] = gl_mul(s, half);
}

// ---------------------------------------------------------------------------
// Key switching
// ---------------------------------------------------------------------------

// out[b][c] = (c == n ? b'_b : 0) - sum_{j,t} d_{b,j,t} KSK[j][t][c].
// A workgroup covers KS_BT ciphertexts x 256 output columns.  Digits are
// produced in LDS per chunk of KS_JC input coefficients in offset form
// d + h in [0, 2h] (h = 2^(beta_ks-1)); the offset is removed at the end
// with the column sums stored after the key (k_ksk_colsum).  Sums of
// offset digit x 32-bit half-word products stay below N l_ks 2^beta_ks
// 2^32 < 2^64, so the two 64-bit accumulators per output never wrap.
constexpr int KS_BT = 16;
constexpr int KS_JC = 32;
constexpr int KS_TPB = 256;

template <int LKS>
__global__ void __launch_bounds__(KS_TPB)
k_keyswitch(const u64 *__restrict__ big, const u64 *__restrict__ ksk, u64 *__restrict__ out,
            size_t batch, int n, int N, int beta) {
  __shared__ u32 dig[KS_JC][LKS][KS_BT];
  __shared__ u64 body[KS_BT];
  const int tid = threadIdx.x;
  const int c = blockIdx.y * KS_TPB + tid;
  const size_t b0 = (size_t)blockIdx.x * KS_BT;
  const int cols = n + 1;
  const int s = 64 - LKS * beta;
  const i64 h = (i64)1 << (beta - 1);
  const i64 mask = ((i64)1 << beta) - 1;

  u64 acc_lo[KS_BT], acc_hi[KS_BT];
#pragma unroll
  for (int b = 0; b < KS_BT; ++b) acc_lo[b] = acc_hi[b] = 0;
  if (tid < KS_BT) body[tid] = (b0 + tid < batch) ? big[(b0 + tid) * (size_t)(N + 1) + N] : 0;

  for (int j0 = 0; j0 < N; j0 += KS_JC) {
    __syncthreads();
    for (int e = tid; e < KS_BT * KS_JC; e += KS_TPB) {
      const int bb = e / KS_JC, jj = e % KS_JC;
      const size_t q = b0 + bb;
      const u64 a = q < batch ? big[q * (size_t)(N + 1) + j0 + jj] : 0;
      i64 r = gl_round_top(a, s);
#pragma unroll
      for (int t = LKS - 1; t >= 1; --t) {
        const i64 d = ((r + h) & mask) - h;
        r = (r - d) >> beta;
        dig[jj][t][bb] = (u32)(d + h);
      }
      dig[jj][0][bb] = (u32)(r + h);
    }
    __syncthreads();
    if (c < cols) {
      const u64 *kp = ksk + (size_t)j0 * LKS * cols + c;
#pragma unroll 4
      for (int jj = 0; jj < KS_JC; ++jj) {
#pragma unroll
        for (int t = 0; t < LKS; ++t) {
          const u64 w = kp[(size_t)(jj * LKS + t) * cols];
          const u32 wl = (u32)w, wh = (u32)(w >> 32);
#pragma unroll
          for (int b = 0; b < KS_BT; ++b) {
            const u32 d = dig[jj][t][b];
            acc_lo[b] += (u64)d * wl;
            acc_hi[b] += (u64)d * wh;
          }
        }
      }
    }
  }
  if (c < cols) {
    const u64 hc = ksk[(size_t)N * LKS * cols + c];
#pragma unroll
    for (int b = 0; b < KS_BT; ++b) {
      const size_t q = b0 + b;
      if (q >= batch) break;
      u64 lo = acc_lo[b] + (acc_hi[b] << 32);
      const u64 hi = (acc_hi[b] >> 32) + (lo < acc_lo[b] ? 1 : 0);
      const u64 sum = gl_reduce128(lo, hi);
      u64 r = gl_sub(c == n ? body[b] : 0, sum);
      out[q * (size_t)cols + c] = gl_add(r, hc);
    }
  }
}

// ---------------------------------------------------------------------------
// Key switching on the int8 matrix cores
// ---------------------------------------------------------------------------

// Over a batch the key switch is one integer matrix product: digits
// D[b][kappa] (batch x N l_ks) times key K[kappa][c] ((N l_ks) x (n+1)),
// kappa = t N + j for digit level t of input coefficient j (any order of
// the contraction index gives the same sum).  Each key word K in [0, p) is
// replaced by V = K or K - p, whichever lies in the range of 8 balanced
// base-256 digits [-128 S, 127 S], S = (2^64 - 1) / 255; V = sum_m 256^m k_m
// with k_m in [-128, 127], so D K = sum_m 256^m (D k_m) (mod p) with eight
// exact int8 x int8 -> int32 products.  X = V + 128 S lies in [0, 2^64) and
// its plain base-256 digits are k_m + 128, so byte m of X with its top bit
// flipped is k_m as a signed byte; X is K + 128 S, plus 2^32 - 1 (= -p mod
// 2^64) when V = K - p.
//
// Byte-plane layout, in 8-byte words: word ((cb KB + kb) 8 + m) 128
// + 2 lane + cc holds, in byte i, k_m[kappa][c] with kappa = 32 kb +
// 8 (lane / 16) + i and c = 32 cb + 16 cc + lane % 16 (0 past the last
// column): the B operand of a 16 x 16 x 32 int8 product (lane l supplies
// rows 8 (l / 16) .. + 7 of column l % 16) for column tile cc of column
// block cb, plane m, k block kb (KB = N l_ks / 32 of them).  The 1024
// words of one (cb, kb) are contiguous, and a lane's two column tiles are
// adjacent.
constexpr u64 KS_S128 = 0x8080808080808080ull;   // 128 S
constexpr u64 KS_S127 = 0x7F7F7F7F7F7F7F7Full;   // 127 S

__global__ void k_ksk_planes(const u64 *__restrict__ ksk, u64 *__restrict__ planes, int N,
                             int lks, int cols, size_t words) {
  const size_t w = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (w >= words) return;
  const int cc = (int)(w & 1), lane = (int)((w >> 1) & 63), m = (int)((w >> 7) & 7);
  const size_t blk = w >> 10;              // cb KB + kb
  const size_t KB = (size_t)N * lks / 32;
  const int kb = (int)(blk % KB), cb = (int)(blk / KB);
  const int c = 32 * cb + 16 * cc + lane % 16;
  u64 word = 0;
  for (int i = 0; i < 8; ++i) {
    const int kappa = 32 * kb + 8 * (lane / 16) + i;
    const int t = kappa / N, j = kappa % N;
    const u64 K = c < cols ? ksk[((size_t)j * lks + t) * cols + c] : 0;
    const u64 X = K + KS_S128 + (K <= KS_S127 ? 0 : GL_EPS);
    word |= (((X >> (8 * m)) & 0xFF) ^ 0x80) << (8 * i);
  }
  planes[w] = word;
}

typedef int32_t ks_v4i __attribute__((ext_vector_type(4)));

// out[b][c] = (c == n ? b'_b : 0) - sum_kappa D[b][kappa] K[kappa][c].
// (The kernel for batches too large to be split where digits made once do not
// pay (ks_route) or no scratch is to be had: captured streams, the
// allocation-free entry point.)
// Workgroup = 4 waves on one 32-column block, each wave on its own 32
// ciphertexts: two 16-ciphertext row tiles x two 16-column tiles x 8 byte
// planes of int32 accumulators.  The contraction runs over k blocks in the
// order (32-coefficient chunk, level from the bottom); the workgroup
// stages each k block's 8 KB of key fragments in LDS (double-buffered, one
// barrier per k block, the next block's global loads in flight during the
// current one's products), so the key is fetched once per 128 ciphertexts.
// At a chunk's first level a lane rounds its 8 coefficients of each row
// tile (loaded one chunk ahead) and issues the next chunk's loads; every
// level peels one balanced digit from the bottom (the A operand of level
// t: row l % 16, coefficients 8 (l / 16) .. + 7) and issues 32 products.
// The planes are recombined exactly: with |acc| < 2^31, lo = sum_{m<4}
// 256^m acc_m and hi = sum_{m>=4} 256^(m-4) acc_m are below 2^56 in
// magnitude, and the sum is lo + 2^32 hi mod p.  A wave with no
// ciphertexts still takes part in the staging and the barriers.
//
// Two waves per SIMD: the register cap of 256 holds the 128 accumulators,
// the key fragments and the prefetched coefficients without spills (left
// to itself the compiler takes 256 + 128 registers and one wave).
constexpr int KSM_WAVES = 4;
static_assert(32 * KSM_WAVES == KS_MFMA_ROWS, "ks_route counts these workgroups");

template <int LKS>
__global__ void __launch_bounds__(64 * KSM_WAVES) __attribute__((amdgpu_waves_per_eu(2, 2)))
k_keyswitch_mfma(const u64 *__restrict__ big, const u64 *__restrict__ planes,
                 u64 *__restrict__ out, size_t batch, int n, int N, int beta) {
  __shared__ __attribute__((aligned(16))) u64 kbuf[2][1024];
  const int tid = threadIdx.x;
  const int wv = tid >> 6, l = tid & 63;
  const int cb = blockIdx.y;
  const int cols = n + 1;
  const size_t b0 = ((size_t)blockIdx.x * KSM_WAVES + wv) * 32;
  const bool active = b0 < batch;
  const int s = 64 - LKS * beta;
  const int32_t h = 1 << (beta - 1), mask = (1 << beta) - 1;
  const int NB = N / 32, KB = NB * LKS;
  // this thread's 32 bytes of each k block's 8 KB
  const ulonglong2 *gsrc = (const ulonglong2 *)(planes + (size_t)cb * KB * 1024) + 2 * tid;

  const u64 *arow[2];
  bool aok[2];
#pragma unroll
  for (int bt = 0; bt < 2; ++bt) {
    const size_t q = b0 + 16 * bt + (l & 15);
    aok[bt] = q < batch;
    arow[bt] = big + (aok[bt] ? q : 0) * (size_t)(N + 1) + 8 * (l >> 4);
  }
  ks_v4i acc[2][2][8];
#pragma unroll
  for (int bt = 0; bt < 2; ++bt)
#pragma unroll
    for (int cc = 0; cc < 2; ++cc)
#pragma unroll
      for (int m = 0; m < 8; ++m) acc[bt][cc][m] = ks_v4i{0, 0, 0, 0};

  {
    const ulonglong2 g0 = gsrc[(size_t)(LKS - 1) * NB * 512], g1 = gsrc[(size_t)(LKS - 1) * NB * 512 + 1];
    ((ulonglong2 *)kbuf[0])[2 * tid] = g0;
    ((ulonglong2 *)kbuf[0])[2 * tid + 1] = g1;
  }
  __syncthreads();

  // raw coefficients of the next chunk, loaded a whole chunk (l_ks k
  // blocks) before they are rounded
  u64 cn[2][8];
#pragma unroll
  for (int bt = 0; bt < 2; ++bt)
#pragma unroll
    for (int i = 0; i < 8; ++i) cn[bt][i] = (active && aok[bt]) ? arow[bt][i] : 0;
  int32_t r[2][8];
  const int total = NB * LKS;
#pragma unroll 1
  for (int it = 0; it < total; ++it) {
    const int jb = it / LKS, t = LKS - 1 - (it - jb * LKS);
    // next k block: (jb, t - 1), or (jb + 1, LKS - 1)
    ulonglong2 p0, p1;
    const bool more = it + 1 < total;
    if (more) {
      const int kn = t > 0 ? (t - 1) * NB + jb : (LKS - 1) * NB + jb + 1;
      p0 = gsrc[(size_t)kn * 512];
      p1 = gsrc[(size_t)kn * 512 + 1];
    }
    if (active) {
      if (t == LKS - 1) {
#pragma unroll
        for (int bt = 0; bt < 2; ++bt)
#pragma unroll
          for (int i = 0; i < 8; ++i) r[bt][i] = gl_round_top32(cn[bt][i], s);
        if (jb + 1 < NB) {
#pragma unroll
          for (int bt = 0; bt < 2; ++bt)
#pragma unroll
            for (int i = 0; i < 8; ++i) cn[bt][i] = aok[bt] ? arow[bt][32 * (jb + 1) + i] : 0;
        }
      }
      long a[2];
#pragma unroll
      for (int bt = 0; bt < 2; ++bt) {
        u32 w0 = 0, w1 = 0;
#pragma unroll
        for (int i = 0; i < 8; ++i) {
          int32_t d = r[bt][i];
          if (t > 0) {
            d = ((d + h) & mask) - h;
            r[bt][i] = (r[bt][i] - d) >> beta;
          }
          const u32 byte = (u32)d & 0xFFu;
          if (i < 4) w0 |= byte << (8 * i);
          else w1 |= byte << (8 * (i - 4));
        }
        a[bt] = (long)gl_mk(w0, w1);
      }
      const ulonglong2 *kb2 = (const ulonglong2 *)kbuf[it & 1] + l;
#pragma unroll
      for (int m = 0; m < 8; ++m) {
        const ulonglong2 f = kb2[64 * m];
#pragma unroll
        for (int bt = 0; bt < 2; ++bt) {
          acc[bt][0][m] = __builtin_amdgcn_mfma_i32_16x16x32_i8(a[bt], (long)f.x, acc[bt][0][m], 0, 0, 0);
          acc[bt][1][m] = __builtin_amdgcn_mfma_i32_16x16x32_i8(a[bt], (long)f.y, acc[bt][1][m], 0, 0, 0);
        }
      }
    }
    if (more) {
      ((ulonglong2 *)kbuf[(it + 1) & 1])[2 * tid] = p0;
      ((ulonglong2 *)kbuf[(it + 1) & 1])[2 * tid + 1] = p1;
    }
    __syncthreads();
  }
  if (!active) return;

#pragma unroll
  for (int bt = 0; bt < 2; ++bt)
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const size_t q = b0 + 16 * bt + 4 * (l >> 4) + i;
      if (q >= batch) continue;
      const u64 body = big[q * (size_t)(N + 1) + N];
#pragma unroll
      for (int cc = 0; cc < 2; ++cc) {
        const int c = 32 * cb + 16 * cc + (l & 15);
        if (c >= cols) continue;
        int64_t lo = 0, hi = 0;
#pragma unroll
        for (int m = 3; m >= 0; --m) {
          lo = lo * 256 + acc[bt][cc][m][i];
          hi = hi * 256 + acc[bt][cc][m + 4][i];
        }
        const u64 lop = (u64)lo + (lo < 0 ? GL_P : 0);
        const u64 hi_p = (u64)hi + (hi < 0 ? GL_P : 0);
        const u64 sum = gl_add(lop, gl_mul_pow2<32>(hi_p));
        out[q * (size_t)cols + c] = gl_sub(c == n ? body : 0, sum);
      }
    }
}

// ---------------------------------------------------------------------------
// Key switching on the int8 matrix cores: digits made once (large batches)
// ---------------------------------------------------------------------------

// The digits of a whole batch as the matrix product's A operand.  16 x 16 x
// 64 products take 16 bytes per lane: lane l holds row l % 16 and, of each
// 64-deep block of the contraction, the indices 8 g .. + 7 and 32 + 8 g .. + 7
// (g = l / 16), two 32-deep blocks of the key's layout side by side (the
// order inside a block is free as long as both operands share it).  Words:
// [row tile][block][lane] x 16 bytes, block = t (N / 64) + j / 64; rows past
// the batch are 0.
template <int LKS>
__global__ void __launch_bounds__(256)
k_ks_digits(const u64 *__restrict__ big, uint4 *__restrict__ dig, size_t batch, int N, int beta) {
  const int l = threadIdx.x & 63;
  const int NB = N / 64;
  const size_t tile = ((size_t)blockIdx.x * 256 + threadIdx.x) / 64;  // row tile NB + chunk
  const size_t rt = tile / NB;
  const int jb = (int)(tile % NB);
  if (rt >= (batch + 15) / 16) return;
  const size_t q = 16 * rt + (l & 15);
  const u64 *src = big + q * (size_t)(N + 1) + 64 * jb + 8 * (l >> 4);
  const int s = 64 - LKS * beta;
  const int32_t h = 1 << (beta - 1), mask = (1 << beta) - 1;
  int32_t r[16];
#pragma unroll
  for (int i = 0; i < 16; ++i)
    r[i] = q < batch ? gl_round_top32(src[(i & 7) + 32 * (i >> 3)], s) : 0;
#pragma unroll
  for (int t = LKS - 1; t >= 0; --t) {
    u32 w[4] = {0, 0, 0, 0};
#pragma unroll
    for (int i = 0; i < 16; ++i) {
      int32_t d = r[i];
      if (t > 0) {
        d = ((d + h) & mask) - h;
        r[i] = (r[i] - d) >> beta;
      }
      w[i >> 2] |= ((u32)d & 0xFFu) << (8 * (i & 3));
    }
    dig[((rt * LKS + t) * NB + jb) * 64 + l] = uint4{w[0], w[1], w[2], w[3]};
  }
}

typedef int32_t ks_v16b __attribute__((ext_vector_type(4)));  // 16 bytes of an operand

// The planes' sums of one output put together: sum mod p of lo + 2^32 hi (see
// k_keyswitch_mfma), subtracted from the body in the last column.
__device__ __forceinline__ u64 ks_combine(const int32_t (&a)[8], u64 body) {
  int64_t lo = 0, hi = 0;
#pragma unroll
  for (int m = 3; m >= 0; --m) {
    lo = lo * 256 + a[m];
    hi = hi * 256 + a[m + 4];
  }
  const u64 lop = (u64)lo + (lo < 0 ? GL_P : 0);
  const u64 hi_p = (u64)hi + (hi < 0 ? GL_P : 0);
  return gl_sub(body, gl_add(lop, gl_mul_pow2<32>(hi_p)));
}

// Workgroup = 4 waves on 16 columns and 256 ciphertexts, a wave on 64 of them:
// 4 row tiles x 8 byte planes of 16 x 16 x 64 products (128 accumulator
// registers, 32 products per 64-deep block for 12 operand loads).  The key's
// 8 KB of a block are staged in LDS for the four waves (double-buffered);
// key and digits are loaded two blocks ahead (one block ahead: 1821 against
// 1624 us).  Tiles go to the XCDs in squares of 8 x 8 workgroups, what an XCD
// holds at once, which then share both operands in its L2.
//
// Bound: the matrix pipe needs 0.6 ms for 14336 ciphertexts at the headline
// parameters (16 cycles per product); measured 1.62 ms with the digits,
// against 3.55 ms for k_keyswitch_mfma, whose 33 column blocks each round
// and cut every coefficient again and whose 32-deep products run at half
// the rate.  What is left is the wait for the loads at one barrier per block
// and two waves per SIMD.
constexpr int KSG_ROWS = 256;

__global__ void __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(2, 2)))
k_keyswitch_gemm(const u64 *__restrict__ big, const uint4 *__restrict__ dig,
                 const u64 *__restrict__ planes, u64 *__restrict__ out, size_t batch, int n, int N,
                 int KC, int row_blocks, int col_blocks) {
  __shared__ __attribute__((aligned(16))) u64 kbuf[2][8 * 128];  // [plane][lane][half]
  // workgroup -> tile: XCD x (the hardware deals workgroups out in turn) takes
  // a run of the squares' order
  const int tiles = row_blocks * col_blocks, per = (tiles + 7) / 8;
  const int id = (int)(blockIdx.x & 7) * per + (int)(blockIdx.x >> 3);
  if (id >= tiles || (int)(blockIdx.x >> 3) >= per) return;
  // bands of 8 columns of tiles, in each band squares of 8 x 8 in turn
  const int band = id / (8 * row_blocks), in_band = id - band * 8 * row_blocks;
  const int bw = col_blocks - 8 * band < 8 ? col_blocks - 8 * band : 8;
  const int rb = in_band / bw, c16 = 8 * band + in_band % bw;
  const int tid = threadIdx.x, wv = tid >> 6, l = tid & 63;
  const int cols = n + 1;
  // this thread's part of a block: plane tid / 32, lanes 2 (tid % 32) and + 1,
  // both halves (the key's 32-deep blocks 2 kc and 2 kc + 1); column tile
  // c16 % 2 of the key's 32-column block c16 / 2
  const u64 *gsrc = planes + (size_t)(c16 >> 1) * (2 * KC) * 1024 + (tid >> 5) * 128 +
                    4 * (tid & 31) + (c16 & 1);
  const size_t row_tiles = (batch + 15) / 16;
  const uint4 *asrc[4];
#pragma unroll
  for (int rt = 0; rt < 4; ++rt) {
    size_t tl = (size_t)rb * (KSG_ROWS / 16) + 4 * wv + rt;
    if (tl >= row_tiles) tl = row_tiles - 1;  // (results not stored)
    asrc[rt] = dig + tl * KC * 64 + l;
  }
  ks_v4i acc[4][8];
#pragma unroll
  for (int rt = 0; rt < 4; ++rt)
#pragma unroll
    for (int m = 0; m < 8; ++m) acc[rt][m] = ks_v4i{0, 0, 0, 0};
  // operands of the block after next, loaded two blocks ahead
  u64 g[4];
  uint4 a0[4], a1[4], a2[4];
  auto fetch = [&](int kc, uint4 (&a)[4]) {
    const int k = kc < KC ? kc : KC - 1;
    const u64 *p = gsrc + (size_t)k * 2048;
    g[0] = p[0];
    g[1] = p[1024];
    g[2] = p[2];
    g[3] = p[1024 + 2];
#pragma unroll
    for (int rt = 0; rt < 4; ++rt) a[rt] = asrc[rt][(size_t)k * 64];
  };
  auto stage = [&](int b) {
    ulonglong2 *d = (ulonglong2 *)(kbuf[b] + (tid >> 5) * 128) + 2 * (tid & 31);
    d[0] = ulonglong2{g[0], g[1]};
    d[1] = ulonglong2{g[2], g[3]};
  };
  fetch(0, a0);
  stage(0);
  fetch(1, a1);
  __syncthreads();
#pragma unroll 1
  for (int kc = 0; kc < KC; ++kc) {
    // block kc + 1 goes to the buffer whose readers passed the last barrier
    stage((kc + 1) & 1);
    fetch(kc + 2, a2);
    const ks_v16b *kb = (const ks_v16b *)kbuf[kc & 1] + l;
#pragma unroll
    for (int m = 0; m < 8; ++m) {
      const ks_v16b f = kb[64 * m];
#pragma unroll
      for (int rt = 0; rt < 4; ++rt)
        acc[rt][m] = __builtin_amdgcn_mfma_i32_16x16x64_i8(
            ks_v16b{(int)a0[rt].x, (int)a0[rt].y, (int)a0[rt].z, (int)a0[rt].w}, f, acc[rt][m], 0,
            0, 0);
    }
#pragma unroll
    for (int rt = 0; rt < 4; ++rt) {
      a0[rt] = a1[rt];
      a1[rt] = a2[rt];
    }
    __syncthreads();
  }
  const int c = 16 * c16 + (l & 15);
#pragma unroll
  for (int rt = 0; rt < 4; ++rt)
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const size_t q = (size_t)rb * KSG_ROWS + 64 * wv + 16 * rt + 4 * (l >> 4) + i;
      if (q >= batch || c >= cols) continue;
      int32_t v[8];
#pragma unroll
      for (int m = 0; m < 8; ++m) v[m] = acc[rt][m][i];
      out[q * (size_t)cols + c] = ks_combine(v, c == n ? big[q * (size_t)(N + 1) + N] : 0);
    }
}

// ---------------------------------------------------------------------------
// Key switching on the int8 matrix cores: small batches
// ---------------------------------------------------------------------------

// A batch of a few ciphertexts leaves no rows to fill the chip with, so the
// contraction is split: workgroup = 16 waves on one 16-ciphertext tile and one
// 32-column block of the key, wave w on every 16th 64-coefficient chunk, all
// levels of it (a lane rounds its 16 coefficients and peels a digit per
// level).  The key goes from memory to the operands directly: nobody else in
// the workgroup reads it.  The waves' int32 sums (exact in any order, their
// total below 2^31) meet in LDS.  One ciphertext at the headline parameters
// 47 us against 336 us for k_keyswitch_mfma, 32 at N = 4096 107 against 679.
constexpr int KSS_WAVES = 16;

template <int LKS>
__global__ void __launch_bounds__(64 * KSS_WAVES) __attribute__((amdgpu_waves_per_eu(4, 4)))
k_keyswitch_small(const u64 *__restrict__ big, const u64 *__restrict__ planes,
                  u64 *__restrict__ out, size_t batch, int n, int N, int beta) {
  __shared__ int32_t sums[64 * 64];  // [value][lane]
  const int tid = threadIdx.x, wv = tid >> 6, l = tid & 63;
  const int cb = blockIdx.y, cols = n + 1;
  const int s = 64 - LKS * beta;
  const int32_t h = 1 << (beta - 1), mask = (1 << beta) - 1;
  const int NB = N / 64;
  const size_t q = (size_t)blockIdx.x * 16 + (l & 15);
  const u64 *src = big + (q < batch ? q : 0) * (size_t)(N + 1) + 8 * (l >> 4);
  const ulonglong2 *key = (const ulonglong2 *)planes + (size_t)cb * (2 * NB * LKS) * 512 + l;
  ks_v4i acc[2][8];
#pragma unroll
  for (int cc = 0; cc < 2; ++cc)
#pragma unroll
    for (int m = 0; m < 8; ++m) acc[cc][m] = ks_v4i{0, 0, 0, 0};
  for (int e = tid; e < 64 * 64; e += 64 * KSS_WAVES) sums[e] = 0;
#pragma unroll 1
  for (int jb = wv; jb < NB; jb += KSS_WAVES) {
    int32_t r[16];
#pragma unroll
    for (int i = 0; i < 16; ++i) {
      const u64 v = src[64 * jb + (i & 7) + 32 * (i >> 3)];
      r[i] = q < batch ? gl_round_top32(v, s) : 0;
    }
#pragma unroll 1
    for (int t = LKS - 1; t >= 0; --t) {
      u32 w[4] = {0, 0, 0, 0};
#pragma unroll
      for (int i = 0; i < 16; ++i) {
        int32_t d = r[i];
        if (t > 0) {
          d = ((d + h) & mask) - h;
          r[i] = (r[i] - d) >> beta;
        }
        w[i >> 2] |= ((u32)d & 0xFFu) << (8 * (i & 3));
      }
      const ks_v16b a = {(int)w[0], (int)w[1], (int)w[2], (int)w[3]};
      const ulonglong2 *k0 = key + (size_t)(2 * (t * NB + jb)) * 512;
#pragma unroll
      for (int m = 0; m < 8; ++m) {
        const ulonglong2 f0 = k0[64 * m], f1 = k0[512 + 64 * m];
        acc[0][m] = __builtin_amdgcn_mfma_i32_16x16x64_i8(
            a, ks_v16b{(int)f0.x, (int)(f0.x >> 32), (int)f1.x, (int)(f1.x >> 32)}, acc[0][m], 0, 0, 0);
        acc[1][m] = __builtin_amdgcn_mfma_i32_16x16x64_i8(
            a, ks_v16b{(int)f0.y, (int)(f0.y >> 32), (int)f1.y, (int)(f1.y >> 32)}, acc[1][m], 0, 0, 0);
      }
    }
  }
  __syncthreads();
#pragma unroll
  for (int cc = 0; cc < 2; ++cc)
#pragma unroll
    for (int m = 0; m < 8; ++m)
#pragma unroll
      for (int i = 0; i < 4; ++i) atomicAdd(&sums[(i * 16 + cc * 8 + m) * 64 + l], acc[cc][m][i]);
  __syncthreads();
  // output i (0..3) of column tile cc for lane l: one of the first 8 waves
  if (wv < 8) {
    const int i = wv & 3, cc = wv >> 2;
    const size_t row = (size_t)blockIdx.x * 16 + 4 * (l >> 4) + i;
    const int c = 32 * cb + 16 * cc + (l & 15);
    if (row < batch && c < cols) {
      int32_t v[8];
#pragma unroll
      for (int m = 0; m < 8; ++m) v[m] = sums[(i * 16 + cc * 8 + m) * 64 + l];
      out[row * (size_t)cols + c] = ks_combine(v, c == n ? big[row * (size_t)(N + 1) + N] : 0);
    }
  }
}

// ---------------------------------------------------------------------------
// Launchers
// ---------------------------------------------------------------------------

hipError_t launch_ksk_prepare(const uint64_t *ksk_std, uint64_t *ksk_dev,
                              const rosetta_params &p, hipStream_t st) {
  const size_t rows = (size_t)p.N * p.ks_level;
  const int cols = (int)p.n + 1;
  if (ks_on_matrix_cores(p)) {
    const size_t words = ks_matrix_key_words(p);
    hipLaunchKernelGGL(k_ksk_planes, dim3((unsigned)((words + 255) / 256)), dim3(256), 0, st,
                       ksk_std, ksk_dev, (int)p.N, (int)p.ks_level, cols, words);
    return hipGetLastError();
  }
  hipError_t e = hipMemcpyAsync(ksk_dev, ksk_std, rows * cols * sizeof(u64),
                                hipMemcpyDeviceToDevice, st);
  if (e != hipSuccess) return e;
  const u64 half = 1ull << (p.ks_base_log - 1);
  hipLaunchKernelGGL(k_ksk_colsum, dim3((cols + 255) / 256), dim3(256), 0, st, ksk_std,
                     ksk_dev + rows * cols, rows, cols, half);
  return hipGetLastError();
}

#define ROSETTA_KS_LEVELS(CASE) \
  CASE(1) CASE(2) CASE(3) CASE(4) CASE(5) CASE(6) CASE(7) CASE(8)

static hipError_t launch_ks_small(const uint64_t *big, const uint64_t *ksk_dev, uint64_t *out,
                                  size_t batch, const rosetta_params &p, hipStream_t st) {
  const dim3 grid((unsigned)((batch + 15) / 16), (p.n + 1 + 31) / 32);
#define ROSETTA_CASE(LK)                                                                        \
  case LK:                                                                                      \
    hipLaunchKernelGGL(k_keyswitch_small<LK>, grid, dim3(64 * KSS_WAVES), 0, st, big, ksk_dev,  \
                       out, batch, (int)p.n, (int)p.N, (int)p.ks_base_log);                     \
    break;
  switch (p.ks_level) {
    ROSETTA_KS_LEVELS(ROSETTA_CASE)
    default: return hipErrorInvalidValue;
  }
#undef ROSETTA_CASE
  return hipGetLastError();
}

// done: whether the scratch was to be had.  Batches are cut so that it stays
// below KSG_SCRATCH bytes.
constexpr size_t KSG_SCRATCH = (size_t)512 << 20;

static hipError_t launch_ks_gemm(const uint64_t *big, const uint64_t *ksk_dev, uint64_t *out,
                                 size_t batch, const rosetta_params &p, hipStream_t st,
                                 bool &done) {
  const size_t K = (size_t)p.N * p.ks_level;
  size_t rows = KSG_SCRATCH / K / KSG_ROWS * KSG_ROWS;  // per cut
  if (rows > batch) rows = batch;
  void *dig = scratch_take((rows + 15) / 16 * 16 * K, st);
  if (!dig) return hipSuccess;
  done = true;
  const int N = (int)p.N, n = (int)p.n;
  for (size_t q = 0; q < batch; q += rows) {
    const size_t cnt = batch - q < rows ? batch - q : rows;
    const uint64_t *src = big + q * (size_t)(N + 1);
    const unsigned tiles = (unsigned)((cnt + 15) / 16 * (N / 64));
    const dim3 dgrid((tiles + 3) / 4);
#define ROSETTA_CASE(LK)                                                                    \
  case LK:                                                                                  \
    hipLaunchKernelGGL(k_ks_digits<LK>, dgrid, dim3(256), 0, st, src, (uint4 *)dig, cnt, N, \
                       (int)p.ks_base_log);                                                 \
    break;
    switch (p.ks_level) {
      ROSETTA_KS_LEVELS(ROSETTA_CASE)
      default: break;
    }
#undef ROSETTA_CASE
    const int rb = (int)((cnt + KSG_ROWS - 1) / KSG_ROWS), cb = (n + 1 + 15) / 16;
    const unsigned grid = 8 * (unsigned)((rb * cb + 7) / 8);
    hipLaunchKernelGGL(k_keyswitch_gemm, dim3(grid), dim3(256), 0, st, src, (const uint4 *)dig,
                       ksk_dev, out + q * (size_t)(n + 1), cnt, n, N, (int)(K / 64), rb, cb);
  }
  const hipError_t e = hipGetLastError();
  const hipError_t f = scratch_give(dig, st);
  return e != hipSuccess ? e : f;
}

hipError_t launch_keyswitch(const uint64_t *big, const uint64_t *ksk_dev, uint64_t *out,
                            size_t batch, const rosetta_params &p, bool may_allocate,
                            hipStream_t st) {
  const KsRoute route = ks_route(p, batch, (size_t)device_cus());
  if (route == KsRoute::SPLIT) return launch_ks_small(big, ksk_dev, out, batch, p, st);
  if (route == KsRoute::DIGITS && may_allocate) {
    bool done = false;
    const hipError_t e = launch_ks_gemm(big, ksk_dev, out, batch, p, st, done);
    if (done) return e;
  }
  if (route != KsRoute::VALU) {
    const dim3 grid((unsigned)((batch + 32 * KSM_WAVES - 1) / (32 * KSM_WAVES)),
                    (p.n + 1 + 31) / 32);
    const int n = (int)p.n, N = (int)p.N, beta = (int)p.ks_base_log;
#define ROSETTA_KSM_CASE(LK)                                                               \
  case LK:                                                                                 \
    hipLaunchKernelGGL(k_keyswitch_mfma<LK>, grid, dim3(64 * KSM_WAVES), 0, st, big, ksk_dev, \
                       out, batch, n, N, beta);                                            \
    break;
    switch (p.ks_level) {
      ROSETTA_KSM_CASE(1)
      ROSETTA_KSM_CASE(2)
      ROSETTA_KSM_CASE(3)
      ROSETTA_KSM_CASE(4)
      ROSETTA_KSM_CASE(5)
      ROSETTA_KSM_CASE(6)
      ROSETTA_KSM_CASE(7)
      ROSETTA_KSM_CASE(8)
      default:
        return hipErrorInvalidValue;
    }
#undef ROSETTA_KSM_CASE
    return hipGetLastError();
  }
  const dim3 grid((unsigned)((batch + KS_BT - 1) / KS_BT), (p.n + 1 + KS_TPB - 1) / KS_TPB);
  const int n = (int)p.n, N = (int)p.N, beta = (int)p.ks_base_log;
#define ROSETTA_KS_CASE(LK)                                                                 \
  case LK:                                                                                  \
    hipLaunchKernelGGL(k_keyswitch<LK>, grid, dim3(KS_TPB), 0, st, big, ksk_dev, out, batch, \
                       n, N, beta);                                                         \
    break;
  switch (p.ks_level) {
    ROSETTA_KS_CASE(1)
    ROSETTA_KS_CASE(2)
    ROSETTA_KS_CASE(3)
    ROSETTA_KS_CASE(4)
    ROSETTA_KS_CASE(5)
    ROSETTA_KS_CASE(6)
    ROSETTA_KS_CASE(7)
    ROSETTA_KS_CASE(8)
    default:
      return hipErrorInvalidValue;
  }
#undef ROSETTA_KS_CASE
  return hipGetLastError();
}

}  // namespace rosetta
