// Chunk gradients at many evaluation points on the bf16 matrix cores.
//
// With b evaluation points W [b][d] the per-chunk gradient (Sec. 1) is two
// dense contractions per chunk i:
//   Z_i = X_i W^T          [n][b]   (K = d)
//   U_i = loss'(Z_i) - y_i [n][b]   (residuals, broadcast over the points)
//   G_i = U_i^T X_i        [b][d]   (K = n),   stored as G[q][i][:]
//
// Arithmetic: every fp32 operand v is split into three bf16 parts v = v1 + v2 + v3 (X by
// rounding to nearest, W and U by truncation) and the six products of parts i + j <= 4 are
// kept; those dropped stay below 2^-22 of the term, with random signs.  Products of two
// bf16 values are exact in fp32 and v_mfma_f32_32x32x16_bf16 accumulates them in fp32, the
// products v1 w1 in one accumulator and the five small ones in another, so only one addition
// per 16 terms rounds at the sum's own size (fp32 matrix instructions: one per 2 terms).
// The matrix cores round worse than to nearest, so long sums drift: calls whose sums were short before
// (see gc_chunk_grads) add them up in segments, of 512 columns and of 128 rows or more.
// A sum in a tile that is not finite (an infinity's or a NaN's parts, or values near the largest
// float that round up) makes its wave compute the tile again with the fp32 matrix instructions,
// which treat infinities as the vector units do.
//
// Magnitudes: parts below 2^-126 are lost, so values below about 2^-108 keep less than 24 bits.  U is
// scaled up by 2^40 for its parts, since whole chunks can have residuals that small (logistic loss of
// separated data); X and W are taken as they are.
//
//   zw_kernel     Z partials over a split of K = d, for 128 of the N n sample rows and up to
//                 128 points per block.  A wave loads its 32 rows of X from memory in the
//                 matrix operand's layout (32 neighbouring bytes of a row per instruction, four
//                 instructions a cache line), two stages of 32 k ahead; W's parts are shared
//                 through LDS by the block's four waves.
//   resid_kernel  U = loss'(sum of the partials, in split order) - y.
//   utx_kernel    G tiles: a wave loads 32 PW positions of the rows of X straight in the
//                 operand's layout (contiguous across the lanes), U is split on its way to LDS.
//                 Chunks are taken in descending order: the last ones read by zw_kernel are
//                 still in the memory-side cache.
//
// X of 50 x 512 x 16384 (1.7 GB), both GEMMs on the fp32 matrix instructions before: 20 points
// 1.11 -> 0.73 ms (the two reads of X take 0.6), 64 points 1.22 -> 1.01, 128 points 2.03 -> 1.65.
// At 64 points the matrix cores and the vector units (splits) are busy a third of the time each and
// the clock falls under both; registers allow three or two waves per SIMD (four spill).
#include <algorithm>
#include <cfloat>
#include <type_traits>

#include "common.h"

namespace gcx {
namespace {

typedef __bf16 v8bf __attribute__((ext_vector_type(8)));
typedef __bf16 v2bf __attribute__((ext_vector_type(2)));
typedef float v16f __attribute__((ext_vector_type(16)));
typedef float v2f __attribute__((ext_vector_type(2)));
typedef unsigned int v4u __attribute__((ext_vector_type(4)));
// rows of X, W and G start on any float
typedef float v4fu __attribute__((ext_vector_type(4), aligned(4)));
template <int N>
struct Floats;
template <>
struct Floats<1> { typedef float T __attribute__((ext_vector_type(1), aligned(4))); };
template <>
struct Floats<2> { typedef float T __attribute__((ext_vector_type(2), aligned(4))); };
template <>
struct Floats<4> { typedef float T __attribute__((ext_vector_type(4), aligned(4))); };

constexpr int kZThreads = 256;                    // zw_kernel
constexpr int kZRows = 32 * (kZThreads / kWave);  // sample rows per block
constexpr int kMThreads = 256;                    // utx_kernel
constexpr int kMWaves = kMThreads / kWave;
constexpr int kZK = 32;               // k per stage of zw_kernel
constexpr float kUp = 0x1p40f, kDown = 0x1p-40f;  // what U is scaled by, and its sums back
constexpr int kZSeg = 16;             // stages per segment
constexpr int kChainRows = 1024;      // rows of a chunk from which a few blocks make a long chain

__device__ __forceinline__ v16f mfma16(v8bf a, v8bf b, v16f c) {
  return __builtin_amdgcn_mfma_f32_32x32x16_bf16(a, b, c, 0, 0, 0);
}
__device__ __forceinline__ v16f mfma2(float a, float b, v16f c) {
  return __builtin_amdgcn_mfma_f32_32x32x2f32(a, b, c, 0, 0, 0);
}

// Eight values in three bf16 parts, each the rounding of what the earlier ones leave; the
// subtractions (one dot product each: v - 1 part + 0 other) are exact and what the third part
// leaves is below 2^-25 of the value.
__device__ __forceinline__ void split3_rne(const float (&v)[8], v8bf (&g)[3]) {
  // (-1, 0) and (0, -1), kept in registers: as an instruction's inline constant the first is read
  // otherwise
  uint32_t l = 0x0000bf80u, h = 0xbf800000u;
  asm("" : "+s"(l), "+s"(h));
  const v2bf lo = __builtin_bit_cast(v2bf, l), hi = __builtin_bit_cast(v2bf, h);
  v4u p[3];
#pragma unroll
  for (int j = 0; j < 4; ++j) {
    float a = v[2 * j], b = v[2 * j + 1];
#pragma unroll
    for (int s = 0; s < 3; ++s) {
      const v2bf u = __builtin_convertvector(v2f{a, b}, v2bf);
      p[s][j] = __builtin_bit_cast(uint32_t, u);
      a = __builtin_amdgcn_fdot2_f32_bf16(u, lo, a, false);
      b = __builtin_amdgcn_fdot2_f32_bf16(u, hi, b, false);
    }
  }
#pragma unroll
  for (int s = 0; s < 3; ++s) g[s] = __builtin_bit_cast(v8bf, p[s]);
}

// Two values in three parts by truncation: v = v1 + v2 + v3 exactly (|v| >= 2^-100), packed.
__device__ __forceinline__ void split3_trunc(float a, float b, uint32_t (&p)[3]) {
#pragma unroll
  for (int s = 0; s < 3; ++s) {
    const uint32_t ua = __float_as_uint(a), ub = __float_as_uint(b);
    p[s] = __builtin_amdgcn_perm(ub, ua, 0x07060302u);
    a -= __uint_as_float(ua & 0xffff0000u);
    b -= __uint_as_float(ub & 0xffff0000u);
  }
}

// big += a1 b1; small += the other products kept, the smallest first
__device__ __forceinline__ void products(const v8bf (&a)[3], const v8bf (&b)[3], v16f &big, v16f &small) {
  small = mfma16(a[2], b[0], small);
  small = mfma16(a[1], b[1], small);
  small = mfma16(a[0], b[2], small);
  small = mfma16(a[1], b[0], small);
  small = mfma16(a[0], b[1], small);
  big = mfma16(a[0], b[0], big);
}

// waves per SIMD of zw_kernel, as its registers allow
constexpr int z_waves(int qt, bool seg) { return qt == 1 ? (seg ? 3 : 4) : (qt == 2 && !seg ? 3 : 2); }

// Zp[s][r][q] = sum_{k in split s} X[r][k] * W[q][k] for the rows r of all chunks.
//   A (32 rows x 16 k): lane (h, li) holds row li at k = 4h .. 4h + 3 and 8 + 4h .. 8 + 4h + 3
//   of each 16; B (W) the same k of point li, its parts in LDS as the lanes read them:
//   Ws[buffer][16-step][part][point tile][lane] of 16 bytes.
//   SEG: the split in segments of kZSeg stages, each summed by itself and added to Zp.
template <int QT, bool SEG>  // point tiles of 32 per block
__global__ __launch_bounds__(kZThreads) __attribute__((amdgpu_waves_per_eu(z_waves(QT, SEG)))) void zw_kernel(const float *__restrict__ X, const float *__restrict__ W,
                                                          int64_t R, int64_t d, int b, int splits, int64_t kper,
                                                          int qblocks, float *__restrict__ Zp) {
  __shared__ __align__(16) uint2 Ws[2][2][3][QT][kWave][2];
  int64_t bid = blockIdx.x;
  const int q0 = int(bid % qblocks) * 32 * QT;
  bid /= qblocks;
  const int s = int(bid % splits);
  const int64_t r0 = bid / splits * kZRows;
  const int t = threadIdx.x, lane = t % kWave, wave = t / kWave, h = lane >> 5, li = lane & 31;
  const int64_t ks0 = int64_t(s) * kper;
  const int64_t ks1 = ks0 + kper < d ? ks0 + kper : d;
  const int64_t row = r0 + 32 * wave + li;
  const float *xr = X + (row < R ? row : R - 1) * d;  // rows past the last repeat it, not stored

  float rx[16];  // a stage of X: 4 times 4 neighbouring k
  auto xload = [&](int64_t kb) {
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      const v4fu v = *reinterpret_cast<const v4fu *>(xr + kb + 8 * u + 4 * h);
#pragma unroll
      for (int e = 0; e < 4; ++e) rx[4 * u + e] = v[e];
    }
  };
  // unit c = t + 256 i of a stage of W: point c / 8, k = 4 (c % 8) .. + 3
  float rw[QT][4];
  auto wload = [&](int64_t kb) {
#pragma unroll
    for (int i = 0; i < QT; ++i) {
      const int q = q0 + t / 8 + 32 * i;
      const v4fu v = *reinterpret_cast<const v4fu *>(W + int64_t(q < b ? q : b - 1) * d + kb + 4 * (t % 8));
#pragma unroll
      for (int e = 0; e < 4; ++e) rw[i][e] = v[e];
    }
  };
  auto wstore = [&](int buf) {
    const int kq = t % 8, l = 32 * (kq & 1) + t / 8;  // the lane that holds these k
#pragma unroll
    for (int i = 0; i < QT; ++i) {
      uint32_t lo[3], hi[3];
      split3_trunc(rw[i][0], rw[i][1], lo);
      split3_trunc(rw[i][2], rw[i][3], hi);
#pragma unroll
      for (int p = 0; p < 3; ++p) Ws[buf][kq >> 2][p][i][l][(kq >> 1) & 1] = make_uint2(lo[p], hi[p]);
    }
  };

  v16f big[QT], small[QT];
  // the products of the stage in rx, its W in LDS buffer buf; next(): what to issue once rx is free
  auto stage = [&](int buf, auto next) {
    v8bf a[2][3];
#pragma unroll
    for (int m = 0; m < 2; ++m) {
      float v[8];
#pragma unroll
      for (int e = 0; e < 8; ++e) v[e] = rx[8 * m + e];
      split3_rne(v, a[m]);
    }
    next();
#pragma unroll
    for (int m = 0; m < 2; ++m)
#pragma unroll
      for (int i = 0; i < QT; ++i) {
        v8bf w[3];
#pragma unroll
        for (int p = 0; p < 3; ++p) w[p] = *reinterpret_cast<const v8bf *>(&Ws[buf][m][p][i][lane][0]);
        products(a[m], w, big[i], small[i]);
      }
  };
  // the columns k0 .. k1 - 1 of the split, whose first are ks0, ..
  auto segment = [&](int64_t k0, int64_t k1) {
#pragma unroll
    for (int i = 0; i < QT; ++i) big[i] = small[i] = v16f{};
    const int64_t nst = (k1 - k0) / kZK;  // whole stages
    if (nst > 0) {
      wload(k0);
      xload(k0);
      wstore(0);
      if (nst > 1) wload(k0 + kZK);
      __syncthreads();
    }
    // stage st: its X in rx, its W in LDS buffer st & 1, the next W in rw
    for (int64_t st = 0; st < nst; ++st) {
      stage(int(st & 1), [&] {
        if (st + 1 < nst) xload(k0 + (st + 1) * kZK);
      });
      if (st + 1 < nst) {
        wstore(int(st & 1) ^ 1);
        if (st + 2 < nst) wload(k0 + (st + 2) * kZK);
      }
      __syncthreads();
    }
    if (const int left = int(k1 - k0 - nst * kZK); left > 0) {  // the last k: zeros past them
      const int64_t kb = k0 + nst * kZK;
#pragma unroll
      for (int e = 0; e < 16; ++e) {
        const int k = 8 * (e / 4) + 4 * h + e % 4;
        const float v = xr[kb + (k < left ? k : 0)];
        rx[e] = k < left ? v : 0.f;
      }
#pragma unroll
      for (int i = 0; i < QT; ++i) {
        const int q = q0 + t / 8 + 32 * i;
        const float *src = W + int64_t(q < b ? q : b - 1) * d + kb;
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          const int k = 4 * (t % 8) + e;
          const float v = src[k < left ? k : 0];
          rw[i][e] = k < left ? v : 0.f;
        }
      }
      wstore(0);
      __syncthreads();
      stage(0, [] {});
    }

    bool bad = false;
#pragma unroll
    for (int i = 0; i < QT; ++i)
#pragma unroll
      for (int v = 0; v < 16; ++v) {
        big[i][v] += small[i][v];
        bad = bad || !(fabsf(big[i][v]) <= FLT_MAX);
      }
    if (__any(bad)) {  // the tile on the fp32 matrix instructions
#pragma unroll
      for (int i = 0; i < QT; ++i) {
        const int q = q0 + 32 * i + li;
        const float *wr = W + int64_t(q < b ? q : b - 1) * d;
        big[i] = v16f{};
        for (int64_t k = k0 + h; k - h < k1; k += 2) {
          const float x = xr[k < k1 ? k : k1 - 1], w = wr[k < k1 ? k : k1 - 1];
          big[i] = mfma2(k < k1 ? x : 0.f, k < k1 ? w : 0.f, big[i]);
        }
      }
    }
    float *Zs = Zp + (int64_t(s) * R + r0 + 32 * wave) * b + q0;
#pragma unroll
    for (int i = 0; i < QT; ++i)
#pragma unroll
      for (int v = 0; v < 16; ++v) {
        const int r = 8 * (v >> 2) + 4 * h + (v & 3);
        if (r0 + 32 * wave + r < R && q0 + 32 * i + li < b) {
          float *dst = Zs + int64_t(r) * b + 32 * i + li;
          *dst = k0 == ks0 ? big[i][v] : *dst + big[i][v];
        }
      }
  };
  if constexpr (SEG) {
    for (int64_t k0 = ks0; k0 < ks1; k0 += kZSeg * kZK) segment(k0, k0 + kZSeg * kZK < ks1 ? k0 + kZSeg * kZK : ks1);
  } else {
    segment(ks0, ks1);
  }
}

// U[r][q] = loss'(sum_s Zp[s][r][q]) - y[r] for the rows r of all chunks, the splits summed in eight
// runs (one long run of 128 splits was off by 1.3e-7 in all, four by 1.2e-7); in place where there is one.
__global__ __launch_bounds__(256) void resid_kernel(const float *Zp, const float *__restrict__ y, int64_t total,
                                                    int b, int splits, int loss, float *U) {
  const int64_t e = int64_t(blockIdx.x) * blockDim.x + threadIdx.x;
  if (e >= total) return;
  float zs[8] = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
  int s = 0;
#pragma unroll 2
  for (; s + 8 <= splits; s += 8)
#pragma unroll
    for (int u = 0; u < 8; ++u) zs[u] += Zp[int64_t(s + u) * total + e];
  if (s < splits) {
#pragma unroll
    for (int u = 0; u < 8; ++u) {
      const float v = Zp[int64_t(s + u < splits ? s + u : s) * total + e];
      zs[u] += s + u < splits ? v : 0.f;
    }
  }
  const float z = ((zs[0] + zs[1]) + (zs[2] + zs[3])) + ((zs[4] + zs[5]) + (zs[6] + zs[7]));
  const float yv = y[e / b];
  U[e] = loss == GC_LOSS_LOGISTIC ? 1.0f / (1.0f + expf(-z)) - yv : z - yv;
}

// G[q][i][x] = sum_r U[i][r][q] * X[i][r][x] for QT point tiles and 4 x 32 PW positions per block.
//   B (16 rows x 32 positions): lane (h, li) holds rows h, h + 2, .. h + 14 of each 16 at positions
//   PW li .. + PW - 1, PW separate 32-wide tiles
//   SEG: the rows in segments of kseg steps of 16, each summed by itself and added to G
template <int QT, int PW, bool SEG>
__global__ __launch_bounds__(kMThreads, 2) void utx_kernel(const float *__restrict__ U, const float *__restrict__ X,
                                                           int N, int n, int64_t d, int b, int kseg, int qblocks,
                                                            int64_t tiles, float *__restrict__ G) {
  using VT = typename Floats<PW>::T;
  __shared__ __align__(16) uint32_t Us[2][QT * 3 * kWave][4];  // U's parts of a stage as the lanes read them
  // the point blocks of one tile of X: eight apart, so on one XCD (round-robin dispatch)
  const int64_t bid = blockIdx.x;
  const int qb = int(bid / 8 % qblocks);
  const int64_t item = bid / 8 / qblocks * 8 + bid % 8;
  if (item >= tiles * N) return;  // the whole block
  const int64_t i = N - 1 - item / tiles;
  const int t = threadIdx.x, lane = t % kWave, h = lane >> 5, li = lane & 31;
  const int wave = __builtin_amdgcn_readfirstlane(t / kWave);
  const int64_t x0 = (item % tiles * kMWaves + wave) * 32 * PW;
  const int64_t x = x0 + PW * li;
  const bool inside = x0 + 32 * PW <= d;
  const float *Xi = X + i * int64_t(n) * d;
  const float *Ui = U + i * int64_t(n) * b;

  const uint32_t loff = uint32_t(h) * uint32_t(d) * 4u + uint32_t(PW * li) * 4u;  // d <= 2^28
  float rx[2][PW][8];
  auto xload = [&](auto setc, int ks) {
    constexpr int SET = decltype(setc)::value;
    if (inside && 16 * ks + 16 <= n) {
#pragma unroll
      for (int j = 0; j < 8; ++j) {
        const char *src = reinterpret_cast<const char *>(Xi + int64_t(16 * ks + 2 * j) * d + x0);  // the same for all lanes
        const VT v = *reinterpret_cast<const VT *>(src + loff);
#pragma unroll
        for (int w = 0; w < PW; ++w) rx[SET][w][j] = v[w];
      }
    } else {
#pragma unroll
      for (int j = 0; j < 8; ++j) {
        const int r = 16 * ks + 2 * j + h;  // past the last row: that row again, times zero
        const float *src = Xi + int64_t(r < n ? r : n - 1) * d;
#pragma unroll
        for (int w = 0; w < PW; ++w) rx[SET][w][j] = src[x + w < d ? x + w : d - 1];
      }
    }
  };
  // each thread two rows of QT points, zero past the rows and the points
  const int uh = t / 32 % 2, uj = t / 64;
  float ru[QT][2];
  // the thread's first row of the first stage (addresses formed anew per stage cost 12% at 64 points)
  const float *up[QT];
#pragma unroll
  for (int c = 0; c < QT; ++c) {
    const int q = (qb * QT + c) * 32 + t % 32;
    up[c] = Ui + int64_t(4 * uj + uh) * b + (q < b ? q : b - 1);
  }
  auto uload = [&](int ks) {
    if (16 * ks + 16 <= n) {
#pragma unroll
      for (int c = 0; c < QT; ++c) {
        const float *src = up[c] + int64_t(16 * ks) * b;
        const bool in = (qb * QT + c) * 32 + t % 32 < b;
        const float v0 = src[0], v1 = src[2 * int64_t(b)];
        ru[c][0] = in ? v0 : 0.f;
        ru[c][1] = in ? v1 : 0.f;
      }
      return;
    }
#pragma unroll
    for (int c = 0; c < QT; ++c)
#pragma unroll
      for (int e = 0; e < 2; ++e) {
        const int r = 16 * ks + 2 * (2 * uj + e) + uh, q = (qb * QT + c) * 32 + t % 32;
        const float v = Ui[int64_t(r < n ? r : n - 1) * b + (q < b ? q : b - 1)];
        ru[c][e] = r < n && q < b ? v : 0.f;
      }
  };
  auto ustore = [&](int buf) {
#pragma unroll
    for (int c = 0; c < QT; ++c) {
      uint32_t p[3];
      split3_trunc(ru[c][0] * kUp, ru[c][1] * kUp, p);
#pragma unroll
      for (int v = 0; v < 3; ++v) Us[buf][(c * 3 + v) * kWave + 32 * uh + t % 32][uj] = p[v];
    }
  };

  v16f big[QT][PW], small[QT][PW];
  using Zero = std::integral_constant<int, 0>;
  using One = std::integral_constant<int, 1>;
  // stage ks: its X in register set ks & 1, its U in LDS buffer ks & 1, the next U in ru
  auto stage = [&](int ks, int ksteps, auto setc) {
    constexpr int SET = decltype(setc)::value;
    v8bf xs[PW][3];
#pragma unroll
    for (int w = 0; w < PW; ++w) split3_rne(rx[SET][w], xs[w]);
    if (ks + 2 < ksteps) xload(setc, ks + 2);
#pragma unroll
    for (int q = 0; q < QT; ++q) {
      v8bf u[3];
#pragma unroll
      for (int p = 0; p < 3; ++p) u[p] = *reinterpret_cast<const v8bf *>(&Us[SET][(q * 3 + p) * kWave + lane][0]);
#pragma unroll
      for (int w = 0; w < PW; ++w) products(u, xs[w], big[q][w], small[q][w]);
    }
    if (ks + 1 < ksteps) {
      ustore(SET ^ 1);
      if (ks + 2 < ksteps) uload(ks + 2);
    }
    __syncthreads();
  };
  // the steps ks0 .. ks1 - 1 of 16 rows, ks0 even
  auto segment = [&](int ks0, int ks1) {
#pragma unroll
    for (int q = 0; q < QT; ++q)
#pragma unroll
      for (int w = 0; w < PW; ++w) big[q][w] = small[q][w] = v16f{};
    uload(ks0);
    xload(Zero{}, ks0);
    if (ks0 + 1 < ks1) xload(One{}, ks0 + 1);
    ustore(0);
    if (ks0 + 1 < ks1) uload(ks0 + 1);
    __syncthreads();
    for (int ks = ks0; ks < ks1; ks += 2) {
      stage(ks, ks1, Zero{});
      if (ks + 1 < ks1) stage(ks + 1, ks1, One{});
    }

    bool bad = false;
#pragma unroll
    for (int q = 0; q < QT; ++q)
#pragma unroll
      for (int w = 0; w < PW; ++w)
#pragma unroll
        for (int v = 0; v < 16; ++v) {
          big[q][w][v] += small[q][w][v];
          bad = bad || !(fabsf(big[q][w][v]) <= FLT_MAX);
          big[q][w][v] *= kDown;
        }
    if (__any(bad)) {  // the tile on the fp32 matrix instructions
#pragma unroll
      for (int q = 0; q < QT; ++q) {
#pragma unroll
        for (int w = 0; w < PW; ++w) big[q][w] = v16f{};
        const int qq = (qb * QT + q) * 32 + li;
        const int r1 = SEG && 16 * ks1 < n ? 16 * ks1 : n;
        for (int r = 16 * ks0 + h; r - h < r1; r += 2) {
          const bool in = r < r1;
          const float uv = Ui[int64_t(in ? r : n - 1) * b + (qq < b ? qq : b - 1)];
          const float u = in && qq < b ? uv : 0.f;
          const float *src = Xi + int64_t(in ? r : n - 1) * d;
#pragma unroll
          for (int w = 0; w < PW; ++w) {
            const float v = src[x + w < d ? x + w : d - 1];
            big[q][w] = mfma2(u, in ? v : 0.f, big[q][w]);
          }
        }
      }
    }
#pragma unroll
    for (int q = 0; q < QT; ++q)
#pragma unroll
      for (int v = 0; v < 16; ++v) {
        const int qq = (qb * QT + q) * 32 + 8 * (v >> 2) + 4 * h + (v & 3);
        if (qq >= b) continue;
        float *dst = G + (int64_t(qq) * N + i) * d + x;
        if (inside) {
          VT o;
#pragma unroll
          for (int w = 0; w < PW; ++w) o[w] = big[q][w][v];
          if (ks0 > 0) o += *reinterpret_cast<const VT *>(dst);
          *reinterpret_cast<VT *>(dst) = o;
        } else {
#pragma unroll
          for (int w = 0; w < PW; ++w)
            if (x + w < d) dst[w] = ks0 > 0 ? dst[w] + big[q][w][v] : big[q][w][v];
        }
      }
  };
  const int ksteps = (n + 15) / 16;  // n <= 2^30
  if constexpr (SEG) {
    for (int ks = 0; ks < ksteps; ks += kseg) segment(ks, ks + kseg < ksteps ? ks + kseg : ksteps);
  } else {
    segment(0, ksteps);
  }
}

// Launch plan shared by the workspace-size query and the launch.
struct MfmaPlan {
  int zqt, uqt, upw;          // point tiles per block of each kernel, positions per lane
  int zqblocks, uqblocks;
  int splits;
  int64_t kper, rblocks;
  int useg, qtiles;           // steps of 16 rows per segment, tiles of 32 points
  int64_t blocks1, tiles, blocks2;
};

MfmaPlan mfma_plan(int N, int n, int64_t d, int b, bool seg, int64_t room) {
  MfmaPlan pl{};
  pl.qtiles = int(ceil_div(b, 32));
  const int64_t R = int64_t(N) * n;
  const int64_t stages = ceil_div(d, kZK);
  pl.rblocks = ceil_div(R, kZRows);
  // partials of more than one split go to G, which is written after they have been read, or to the
  // workspace where that has room for more of them (chunks of about as many rows as columns; G
  // alone against both: X of 10 x 512 x 1000 at 64 points 82 us / 46, 1 x 8192 x 8192 at 16 points 726 / 388)
  const int64_t most = std::max<int64_t>(1, std::min(std::max(d / n, room), stages));
  pl.zqt = pl.qtiles <= 2 ? pl.qtiles : (seg ? 2 : 4);
  // fewer point tiles per block where a few blocks are all there is
  while (pl.zqt > 1 && pl.rblocks * ceil_div(pl.qtiles, pl.zqt) * std::min(ceil_div(stages, 4), most) < 256) pl.zqt /= 2;
  // two positions per lane and two point tiles, but for calls short of a block per CU (us, one
  // position per lane against two: X of 8 x 8192 x 2048 at 8 points 588 / 750, 4 x 2000 x 2001 at 16
  // points 146 / 195)
  pl.upw = 2;
  pl.tiles = ceil_div(d, int64_t(32) * pl.upw * kMWaves);
  pl.uqt = pl.qtiles == 1 || pl.tiles * N * ceil_div(pl.qtiles, 2) < 256 ? 1 : 2;
  if (pl.tiles * N * ceil_div(pl.qtiles, pl.uqt) < 256) {
    pl.upw = 1;
    pl.tiles = ceil_div(d, int64_t(32) * kMWaves);
  }
  pl.zqblocks = int(ceil_div(pl.qtiles, pl.zqt));
  pl.uqblocks = int(ceil_div(pl.qtiles, pl.uqt));
  // K = d split so that the blocks fill whole rounds of the resident ones (two to four per CU
  // by point tiles, on 256 CUs); a block costs about 8 stages beyond its own (its prologue,
  // its Z partials written and summed again), and the sums about one per split.  At most 64
  // stages per block (128 additions at a partial's own size), 16 where sums were short before,
  // as far as there is room for so many splits; without it those sums run in segments (50 x 512 x 16384, 4
  // points: 750 us, with splits of 16 stages 700) and others stay below the error of one
  // point at a time (4 x 2000 x 2001, 16 points: 3.1e-7 against 7.5e-7).
  const int64_t resident = 256 * z_waves(pl.zqt, false);
  constexpr int64_t kExtra = 8;
  const int64_t max_stages = seg ? kZSeg : 64;
  const int64_t tiles = pl.rblocks * pl.zqblocks;
  const int64_t least = std::min(ceil_div(stages, max_stages), most);
  int64_t best = -1;
  for (int64_t sp = least; sp <= std::min(std::max<int64_t>(least + 8, 64), most); ++sp) {
    const int64_t nst = ceil_div(stages, sp);
    const int64_t splits = ceil_div(stages, nst);
    const int64_t cost = ceil_div(tiles * splits, resident) * (nst + kExtra) + splits;
    if (best < 0 || cost < best) {
      best = cost;
      pl.splits = int(splits);
      pl.kper = nst * kZK;
    }
  }
  pl.blocks1 = tiles * pl.splits;
  pl.useg = 8;  // about as many segments as two steps of one
  while (2 * int64_t(pl.useg) * pl.useg < ceil_div(n, 16)) pl.useg *= 2;
  pl.blocks2 = ceil_div(pl.tiles * N, 8) * 8 * pl.uqblocks;
  return pl;
}

}  // namespace

// Two passes over X whatever b is, against one (fused) or two per point: from 4 or 2 points on,
// but for small calls, where its third launch costs more than the passes saved (X of 111 x 1001
// at 20 points 13 us against 19, of 256 x 4096 at 4 points 36 against 23), and for four points of
// short rows, whose four passes are as fast (us, fused against matrix cores at 4 points: X of 20 x 512 x
// 1024 51 / 62, 16 x 2048 x 4096 226 / 321, 8 x 8192 x 2048 344 / 749, 100 x 16 x 4096 24 / 32; but 20 x
// 64 x 4096 31 / 28, 20 x 512 x 8192 224 / 177, 20 x 16 x 16384 42 / 32; at 5 points 20 x 512 x 1024 64 / 61).
bool mfma_eligible(int N, int n, int64_t d, int b, bool fused, bool seg, int64_t room) {
  if (b < (fused ? 4 : 2) || d > int64_t(1) << 28 || n > 1 << 30) return false;
  if (fused && b == 4 && d < 8192 && (n < 32 || n > 128)) return false;
  const double volume = double(N) * double(n) * double(d) * double(b);
  if (fused && volume < 3e6) return false;
  const MfmaPlan pl = mfma_plan(N, n, d, b, seg, room);
  // Against two passes per point the third launch, the chain of n rows and that of a split's stages have
  // to pay: both times in us, measured at 1 to 60 chunks of 17 x 815 to 12 x 100001 and 1 to 64 points.
  // One point at a time reads X from a cache the more the points (us, vector units / matrix cores: 1 x 1000
  // x 333 at 17 points 21 / 64, 5 x 200 x 1001 at 8 15 / 26, 2 x 12 x 100001 at 4 20 / 61; above the line 12
  // x 500 x 8193 at 2 133 / 91, 23 x 131 x 4099 at 8 122 / 36, 12 x 60 x 2101 at 64 57 / 25).
  const double vector_us = 13 + 0.014 * n + 1.15e-6 * volume / (1 + std::min(b, 128) / 64.0);
  const double matrix_us = 17 + 0.04 * n + 0.6 * double(pl.kper / kZK) + 0.9e-6 * volume / b;
  if (!fused && vector_us < matrix_us) return false;
  // Few blocks in the second product make a chain of n rows of about 0.07 us each; the fused kernel
  // takes 1 ns per row and point, more past 2000 columns (us, fused / matrix cores: 4 x 8192 x 4096 at 6
  // points 400 / 558, 4 x 2048 x 1024 at 9 116 / 129; 8 x 8192 x 2048 at 8 652 / 573, 10 x 8192 x 1024 at 8
  // 657 / 550, 20 x 2048 x 512 at 8 284 / 135).
  if (fused && pl.upw == 1 && n > kChainRows && int64_t(b) * N * std::max<int64_t>(1000, d / 2) < 60000) return false;
  // few points keep the vector units where more than 64 stages per block would cost precision
  if (b < 16 && pl.kper > 64 * kZK) return false;
  return grid_ok(pl.blocks1, kZThreads) && grid_ok(pl.blocks2, kMThreads) &&
         grid_ok(ceil_div(int64_t(N) * n * b, 256), 256);
}

// workspace: the residuals [N n][b], and room partial sums of them
void launch_mfma_grads(const float *X, const float *y, const float *W, int N, int n, int64_t d, int b,
                       int loss, bool seg, int64_t room, float *G, void *workspace, hipStream_t st) {
  const MfmaPlan pl = mfma_plan(N, n, d, b, seg, room);
  const int64_t R = int64_t(N) * n;
  float *U = static_cast<float *>(workspace);
  float *Zp = pl.splits == 1 ? U : (pl.splits <= d / n ? G : U + R * b);
  const int64_t total = R * b;
#define GC_ZW(QT, SEG)                                                                                    \
  hipLaunchKernelGGL((zw_kernel<QT, SEG>), dim3(unsigned(pl.blocks1)), dim3(kZThreads), 0, st, X, W, R,   \
                     d, b, pl.splits, pl.kper, pl.zqblocks, Zp)
  const bool zseg = seg && pl.kper > kZSeg * kZK;  // segments within the splits as well
  if (pl.zqt == 1 && zseg) GC_ZW(1, true);
  else if (zseg) GC_ZW(2, true);
  else if (pl.zqt == 1) GC_ZW(1, false);
  else if (pl.zqt == 2) GC_ZW(2, false);
  else GC_ZW(4, false);
#undef GC_ZW
  hipLaunchKernelGGL(resid_kernel, dim3(unsigned(ceil_div(total, 256))), dim3(256), 0, st, Zp, y, total, b,
                     pl.splits, loss, U);
#define GC_UTX(QT, PW)                                                                                     \
  hipLaunchKernelGGL((seg ? utx_kernel<QT, PW, true> : utx_kernel<QT, PW, false>),                        \
                     dim3(unsigned(pl.blocks2)), dim3(kMThreads), 0, st, U, X, N, n, d, b, pl.useg,        \
                     pl.uqblocks, pl.tiles, G)
  if (pl.upw == 1) GC_UTX(1, 1);
  else if (pl.uqt == 1) GC_UTX(1, 2);
  else GC_UTX(2, 2);
#undef GC_UTX
}

}  // namespace gcx
