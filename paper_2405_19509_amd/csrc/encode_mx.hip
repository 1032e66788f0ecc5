// gc_encode on the bf16 matrix cores (Sec. 2, worker encode):
//   T[p][j][x] = sum_{t < psi[p][j]} sum_{k < ell} Bc[p][j][t][k] * g_{order[j][t]}[k*L + x]
//
// Per window of (pattern, worker) rows the encode is a dense contraction
//   T[row][x] = sum_kk A[row][kk] * B[kk][x]
// over kk = (chunk slot s of the window's workers, block k): A the coefficients of the
// transmitting rows (zero where the worker does not hold the chunk or has not processed it),
// B the chunk gradients.  The vector units cannot sustain its 2 psi ell flops per 4 bytes of T
// at the HBM write rate past a few terms per output; the bf16 matrix cores can.
//
// Arithmetic: each fp32 coefficient a is split into three bf16 parts a = a1 + a2 + a3 + r
// with |r| <= 2^-24 |a| (each part the bf16 rounding of what the previous ones leave).
// bf16 chunk gradients enter as they are: three products per term.  An fp32 chunk gradient
// g is split into three such parts as well, and the six products a_i g_j with i + j <= 4 are kept:
// the dropped ones stay below 2^-25 |a g|.  Every product of two bf16 values is exact in fp32;
// v_mfma_f32_32x32x16_bf16 accumulates them in fp32, rounding worse than to nearest, so that sums of
// few terms (one K step) keep the small products apart and add them at the end on the vector
// units.  Relative error against 64 bits, with the vector units' (1e-8): rows of one term 2.6 (2.5; 3.9
// with truncated parts and one sum), of up to three terms 2.6 (3.3;
// 3.9), at two steps of up to 21 terms 3.5 (7.1; 3.9).
// A zero coefficient times a non-finite gradient is not zero, so tiles whose gradients are
// not all finite are computed term by term over each row's processed prefix instead.
//
// Layout: a window is up to CW candidate rows, PB patterns x J workers, its transmitting rows
// compacted into 32-row tiles; their coefficient planes are built in LDS once per block.  A
// wave then walks tiles of W = 32 PW positions: it loads B straight into registers in the
// matrix operand's layout (lane (h, li): positions x0 + PW li .. + PW - 1 of the rows kk
// with kk % 2 = h; PW positions per lane are PW separate 32-wide tiles, so loads and stores
// stay contiguous across the lanes), splits it once, multiplies every row tile by it and
// stores each.  The gradients are thus read and split once per window instead of passing
// through LDS, no barrier separates the phases, and nothing orders one wave's stores with
// another's loads.  Measured against LDS slices with barriers between staging, products and
// stores (time per call, MI355X): m = 100, d = 2^20 fp32, ell = 2, 64 patterns 3.2 -> 2.5
// ms (vector path before), ell = 8, 256 patterns 6.3 -> 3.8 ms; m = 200 bf16, d = 2^22, ell =
// 4, half the workers lost 2.8 -> 2.05 ms, d = 2^24, ell = 2, one pattern 3.8 -> 2.6 ms.
// What bounds it: the T stores alone take 1.85 / 2.1 / 1.2 ms of the first three, the products
// 0.6 / 1.6 / 0.7 ms, and the two barely overlap (the clock falls to 1.7 GHz under both); the
// last runs at the rate of a plain copy of its 6.7 GB in and 6 GB out.
//
// Rows of workers that transmit nothing (psi = 0) are not written.  The blocks of a position
// range run back to back on one XCD (round-robin dispatch), so its L2 serves the windows'
// overlapping chunks; those of the ranges past whole eights are spread over all XCDs.  If a window's workers hold more distinct chunks than its slots (orders
// other than the cyclic one), the block takes as many of its workers at a time as fit.
#include <algorithm>
#include <type_traits>

#include "common.h"
#include "encode_mx.h"

namespace gcx {
namespace {

constexpr int kMxThreads = 512;         // threads per block, at most
constexpr int kMxMaxCW = 256;           // candidate rows per window, at most
// K steps of 16 rows of B, as the registers allow
constexpr int kMxMaxKSF32 = 11, kMxMaxKSBF16 = 12;
constexpr int kMxApartTerms = 3;        // terms per output up to which one K step is taken for its smaller error
constexpr int kMxMapChunks = 4096;      // chunks up to which groups of workers are formed
constexpr size_t kMxLds = 144 * 1024;   // dynamic LDS of a block, at most

typedef __bf16 v8bf __attribute__((ext_vector_type(8)));
typedef __bf16 v2bf __attribute__((ext_vector_type(2)));
typedef float v16f __attribute__((ext_vector_type(16)));
typedef float v2f __attribute__((ext_vector_type(2)));
typedef unsigned int v4u __attribute__((ext_vector_type(4)));
// PW neighbouring positions of a gradient or of T, at element alignment: rows start anywhere
template <int N>
struct __attribute__((packed, aligned(2))) HalfPairs {
  uint32_t v[N];
};
template <int N>
struct Floats;
template <>
struct Floats<1> { typedef float T; };
template <>
struct Floats<2> { typedef float T __attribute__((ext_vector_type(2), aligned(4))); };
template <>
struct Floats<4> { typedef float T __attribute__((ext_vector_type(4), aligned(4))); };

// A coefficient in three bf16 parts, each the rounding of what the earlier ones leave, all exact
// steps; the first part is at most the largest bf16, so that what would round past it stays finite.
// An infinity leaves a NaN, as a NaN does.  Two instructions for the limits: v_med3_f32's constant
// stays in a register over the tile loop, one too many for three waves at 11 steps of bf16.
__device__ __forceinline__ void split_coef(float v, uint16_t (&b)[3]) {
  constexpr float most = 0x1.fep127f;
  const __bf16 b1 = __bf16(fmaxf(fminf(v, most), -most));
  const float r1 = v - float(b1);
  const __bf16 b2 = __bf16(r1), b3 = __bf16(r1 - float(b2));
  b[0] = __builtin_bit_cast(uint16_t, b1);
  b[1] = __builtin_bit_cast(uint16_t, b2);
  b[2] = __builtin_bit_cast(uint16_t, b3);
}

// chk + 0 * (either bf16 half of pair): a NaN once a half is infinite or a NaN
__device__ __forceinline__ float times_zero(uint32_t pair, float chk) {
  return __builtin_amdgcn_fdot2_f32_bf16(__builtin_bit_cast(v2bf, pair), __builtin_bit_cast(v2bf, 0u), chk, false);
}

// Eight finite fp32 values in three bf16 parts, each the rounding of what the earlier ones leave
// (|g2| <= 2^-9 |g|, |g3| <= 2^-18 |g|); the subtractions (one dot product each: v - 1 part + 0
// other) are exact for |g| >= 2^-108 and what the third part leaves is below 2^-26 |g|.  A value that is
// not finite, or rounds past the largest bf16, leaves a first part that is not finite.
__device__ __forceinline__ void split3(const float (&v)[8], v8bf (&g)[3]) {
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

struct MxArgs {
  const void *G;
  int N;
  int64_t d, L;
  int64_t lmin;  // positions valid in every block: max(0, d - (ell - 1) L)
  const int32_t *psi;
  const int32_t *order;
  const float *Bc;
  int64_t P;
  int m, delta, ell;
  float *T;
  bool nt;       // rows of T on 64-byte boundaries
  int J, PB;     // workers and patterns per window
  int CW;        // candidate rows J * PB, rounded up to 32
  int ngroups;
  int64_t ntp;   // pattern windows
  int slots;     // chunk slots (rows of B / ell)
  int64_t ntiles, tpb, nsr;  // position tiles, per block, ranges
  // grid: (group, pattern window) units; blocks of the ranges in whole eights; (range, unit) pairs of
  // the ranges left, and an eighth of them
  uint32_t units, whole, left, eighth;
};

// dynamic LDS of a block, as laid out at the kernel
size_t mx_lds(const MxArgs &a, int KS) {
  const size_t Kp = 16 * size_t(KS);
  return size_t(a.CW) * 3 * (Kp + 8) * 2 + 2 * sizeof(int64_t) * Kp + sizeof(int64_t) * a.CW +
         sizeof(int32_t) * (size_t(a.J) * a.delta + a.slots + (a.J > 1 ? a.N : 0)) + 2 * sizeof(int16_t) * a.CW;
}

template <typename GT, int KS, int PW>
struct MxLayout {
  static constexpr bool F32 = sizeof(GT) == 4;
  static constexpr int NP = F32 ? 3 : 1;  // parts of a gradient value
  static constexpr int Kp = 16 * KS;
  static constexpr int AP = Kp + 8;       // plane row stride (bf16): 16-byte rows, staggered banks
  static constexpr int W = 32 * PW;       // positions per tile
  static constexpr bool APART = KS == 1;  // small products in sums of their own
  // Nothing that only the tables' construction needs kept in registers over the tile loop, and one
  // position's sums formed at a time: at one fp32 step and four positions 168 registers, three waves per
  // SIMD, instead of 214 (m = 37, delta = 8, d = 3261045, 2 patterns 399 -> 307 us, m = 90, delta = 7, d =
  // 349517, 3 patterns 99 -> 88).  Elsewhere the waves stay as many and calls lost up to 7% by it.
  static constexpr bool LEAN = F32 && APART;
  // registers: B (4 NP PW KS; fp32 splits take some more), accumulators (16 PW), one K step
  // of A (12), addresses
  static constexpr int REGS = (F32 ? 15 : 4) * PW * KS + 16 * PW + 12 + 40;
  // waves per SIMD asked for: the most that the compiler fits without scratch, which costs a call 18 us
  static constexpr int WPE =
      APART ? 3 : (REGS <= 128 || (F32 && KS == 2 && PW == 2) ? 4 : (REGS <= 168 ? 3 : 2));
};

// The window's rows at the positions of one tile, term by term over the processed prefix in
// order, on the vector units: what a row has not processed does not enter it.  For tiles whose
// gradients are not all finite only.
template <typename GT>
__device__ __forceinline__ void mx_tile_terms(const MxArgs &a, int64_t p0, int j0, int nsend,
                                              const int16_t *crow, const int16_t *cnp, int64_t x0, int64_t x1) {
  const GT *G = static_cast<const GT *>(a.G);
  for (int c = 0; c < nsend; ++c) {
    const int r = __builtin_amdgcn_readfirstlane(crow[c]), np = __builtin_amdgcn_readfirstlane(cnp[c]);
    const int pb = r / a.J, j = j0 + r - pb * a.J;
    const int64_t row = (p0 + pb) * a.m + j;
    const int32_t *ord = a.order + int64_t(j) * a.delta;
    const float *coef = a.Bc + row * a.delta * a.ell;
    for (int64_t x = x0 + threadIdx.x % kWave; x < x1; x += kWave) {
      float acc = 0.f;
      for (int k = 0; k < a.ell; ++k) {  // block k of a gradient, zero from d on
        const int64_t col = int64_t(k) * a.L + x;
        const bool in = col < a.d;
        const GT *gx = G + (in ? col : 0);
#pragma unroll 4
        for (int t = 0; t < np; ++t) {  // loads unconditional, so that several are in flight
          const int ch = ord[t];
          const bool ok = ch >= 0 && ch < a.N;
          const GT v = gx[int64_t(ok ? ch : 0) * a.d];
          float g;
          if constexpr (sizeof(GT) == 4) g = v;
          else g = bf16_to_f32(v);
          const float w = coef[t * a.ell + k];
          acc = fmaf(ok ? w : 0.f, ok && in ? g : 0.f, acc);
        }
      }
      a.T[row * a.L + x] = acc;
    }
  }
}

// LDS: [ planes: CW/32 tiles x 3 x 32 rows x AP bf16 ][ base, lim: Kp int64 each ]
//      [ rowoff: CW int64 ][ code: J*delta int32 ][ slotc: slots int32 ][ map: N int32 (J > 1) ]
//      [ crow, cnp: CW int16 each ]
template <typename GT, int KS, int PW>
__global__ __launch_bounds__(kMxThreads) __attribute__((amdgpu_waves_per_eu(MxLayout<GT, KS, PW>::WPE))) void
encode_mx_kernel(MxArgs a) {
  using Lay = MxLayout<GT, KS, PW>;
  constexpr bool F32 = Lay::F32;
  constexpr int NP = Lay::NP, Kp = Lay::Kp, AP = Lay::AP, W = Lay::W;
  using VT = typename Floats<PW>::T;
  extern __shared__ __align__(16) unsigned char lds[];
  uint16_t *Ap = reinterpret_cast<uint16_t *>(lds);
  int64_t *base = reinterpret_cast<int64_t *>(lds + size_t(a.CW) * 3 * AP * 2);  // [2][Kp / 2]
  int64_t *lim = base + Kp;
  int64_t *rowoff = lim + Kp;
  int32_t *code = reinterpret_cast<int32_t *>(rowoff + a.CW);
  int32_t *slotc = code + a.J * a.delta;
  int32_t *map = slotc + a.slots;
  int16_t *crow = reinterpret_cast<int16_t *>(map + (a.J > 1 ? a.N : 0));
  int16_t *cnp = crow + a.CW;
  __shared__ int wcnt[kMxThreads / kWave];
  __shared__ int nuni_s, jn_s;

  // block -> (position range, unit = (group, pattern window)); XCD x takes ranges x, x + 8, ...
  // of whole eights, and an eighth of the (range, unit) pairs of the ranges left: all of them on
  // short rows, where whole ranges would leave XCDs idle (m = 37, d = 1001, ell = 3, 5000 patterns,
  // one range: 540 us on one XCD, 83 on eight; m = 50, d = 2047, ell = 2, two: 549, 209)
  const int nth = blockDim.x;
  uint32_t b = blockIdx.x, sr, unit;
  if (b < a.whole) {
    sr = (b & 7) + 8 * ((b >> 3) / a.units);
    unit = (b >> 3) % a.units;
  } else {
    b -= a.whole;
    const uint32_t e = (b & 7) * a.eighth + (b >> 3);
    if (e >= a.left) return;  // the whole block
    sr = uint32_t(a.nsr & ~int64_t(7)) + e / a.units;
    unit = e % a.units;
  }
  const int64_t t_begin = int64_t(sr) * a.tpb;
  const int64_t t_end = t_begin + a.tpb < a.ntiles ? t_begin + a.tpb : a.ntiles;
  const int64_t p0 = int64_t(unit / uint32_t(a.ngroups)) * a.PB;
  const int j0 = int(unit % uint32_t(a.ngroups)) * a.J;
  const int nj = a.m - j0 < a.J ? a.m - j0 : a.J;
  const int ell = a.ell;
  float *const Tw = a.T + (p0 * a.m + j0) * a.L;  // row (pattern p0, worker j0) of T
  // a block's value in a scalar register
  auto uniform = [](int v) { return Lay::LEAN ? __builtin_amdgcn_readfirstlane(v) : v; };
  const int tid = threadIdx.x;
  const int wave = __builtin_amdgcn_readfirstlane(tid / kWave), nw = nth / kWave;
  const int lane = tid % kWave, h = lane >> 5, li = lane & 31;

  // every load that waits for nothing: the chunks at each (worker, position), and the counts of
  // the candidates (pattern p0 + r / J, worker j0 + r % J)
  for (int e = tid; e < nj * a.delta; e += nth) {
    const int c = a.order[int64_t(j0) * a.delta + e];
    code[e] = c >= 0 && c < a.N ? c : -1;
  }
  const int rpb = tid / a.J, rjb = tid - rpb * a.J;
  int npr = 0;
  if (tid < a.CW && rpb < a.PB && p0 + rpb < a.P && rjb < nj) npr = a.psi[(p0 + rpb) * a.m + j0 + rjb];
  npr = npr < 0 ? 0 : (npr > a.delta ? a.delta : npr);

  // Passes over the group's workers, each with the slots of its workers' distinct chunks.  One
  // worker: slot t = position t.  Else one pass where every worker's chunks together fit the
  // slots (slots in ascending chunk order; the cyclic order always does), and as many
  // consecutive workers per pass as fit elsewhere.
  int nuni = a.slots + 1;
  if (a.J > 1) {
    for (int c = tid; c < a.N; c += nth) map[c] = -1;
    __syncthreads();
    for (int e = tid; e < nj * a.delta; e += nth)
      if (code[e] >= 0) map[code[e]] = 0;
    __syncthreads();
    if (tid < kWave) {
      int cnt = 0;
      for (int c0 = 0; c0 < a.N; c0 += kWave) {
        const int c = c0 + tid;
        const bool on = c < a.N && map[c] == 0;
        const unsigned long long mk = __ballot(on);
        const int s = cnt + __popcll(mk & ((1ull << tid) - 1));
        if (on) {
          map[c] = s;
          if (s < a.slots) slotc[s] = c;
        }
        cnt += __popcll(mk);
      }
      if (tid == 0) nuni_s = cnt;
    }
    __syncthreads();
    nuni = uniform(nuni_s);
  }
  for (int ja = 0, jn = nj; ja < nj; ja = jn) {  // workers ja .. jn - 1 of the group
    int tp = tid;
    if constexpr (Lay::LEAN) asm volatile("" : "+v"(tp));  // opaque: formed anew in each pass
    int nslot = nuni;
    __syncthreads();  // the previous pass is done with every table
    if (a.J == 1) {
      nslot = a.delta;
      for (int t = tp; t < a.delta; t += nth) slotc[t] = code[t] >= 0 ? code[t] : 0;
    } else if (nuni > a.slots) {
      for (int c = tp; c < a.N; c += nth) map[c] = -1;
      __syncthreads();
      if (tp < kWave) {
        int cnt = 0, j = ja;
        for (; j < nj; ++j) {
          const int c = lane < a.delta ? code[j * a.delta + lane] : -1;  // delta <= 64
          const bool fresh = c >= 0 && map[c] < 0;
          const unsigned long long mk = __ballot(fresh);
          if (cnt + __popcll(mk) > a.slots) break;  // never at j = ja: delta <= slots
          const int s = cnt + __popcll(mk & ((1ull << lane) - 1));
          if (fresh) {
            map[c] = s;
            slotc[s] = c;
          }
          cnt += __popcll(mk);
          __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
          __builtin_amdgcn_wave_barrier();
          __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
        }
        if (tp == 0) {
          nuni_s = cnt;
          jn_s = j;
        }
      }
      __syncthreads();
      nslot = uniform(nuni_s);
      jn = uniform(jn_s);
    }
    const int K = nslot * ell;  // rows of B
    for (int e = tp; e < (a.CW / 32) * (3 * 32 * AP / 8); e += nth)
      reinterpret_cast<uint4 *>(Ap)[e] = make_uint4(0u, 0u, 0u, 0u);
    // the transmitting candidates, compacted in order
    const int rpb = tp / a.J, rjb = tp - rpb * a.J;
    const bool on = npr > 0 && rjb >= ja && rjb < jn;
    const unsigned long long mk = __ballot(on);
    if (lane == 0) wcnt[wave] = __popcll(mk);
    __syncthreads();
    int c0 = 0, nsend = 0;
    for (int w = 0; w < nw; ++w) {
      if (w < wave) c0 += wcnt[w];
      nsend += wcnt[w];
    }
    nsend = uniform(nsend);
    if (on) {
      const int c = c0 + __popcll(mk & ((1ull << lane) - 1));
      crow[c] = int16_t(tp);
      cnp[c] = int16_t(npr);
      rowoff[c] = (int64_t(rpb) * a.m + rjb) * a.L;
    }
    const int ntile = (nsend + 31) / 32;
    // row kk of B: half kk % 2, place kk / 2 (a place past K repeats row 0, with zero
    // coefficients): its element offset in G and the end of its valid positions
    for (int e = tp; e < Kp; e += nth) {
      const int kk = e < K ? e : 0;
      const int s = kk / ell, k = kk - s * ell;
      const int64_t rem = a.d - int64_t(k) * a.L;
      const int q = (e & 1) * (Kp / 2) + (e >> 1);
      base[q] = int64_t(K > 0 ? slotc[s] : 0) * a.d + (rem > 0 ? int64_t(k) * a.L : 0);
      lim[q] = rem < a.L ? rem : a.L;
    }
    __syncthreads();
    // three bf16 planes per row tile, one for each part of the coefficients; row kk at column
    // 16 (kk / 16) + 8 (kk % 2) + (kk % 16) / 2
    for (int e = tp; e < nsend * a.delta; e += nth) {
      const int c = e / a.delta, t = e - c * a.delta;
      if (t >= cnp[c]) continue;
      const int pb = crow[c] / a.J, jb = crow[c] - pb * a.J;
      const int ch = code[jb * a.delta + t];
      if (ch < 0) continue;
      const int s = a.J == 1 ? t : map[ch];
      const float *src = a.Bc + (((p0 + pb) * a.m + j0 + jb) * a.delta + t) * ell;
      uint16_t *row = Ap + (c / 32) * (3 * 32 * AP) + (c % 32) * AP;
      for (int k = 0; k < ell; ++k) {
        const int kk = s * ell + k;
        const int col = (kk & ~15) + 8 * (kk & 1) + ((kk & 15) >> 1);
        uint16_t part[3];
        split_coef(src[k], part);
#pragma unroll
        for (int i = 0; i < 3; ++i) row[32 * i * AP + col] = part[i];
      }
    }
    __syncthreads();

    const int64_t *bh = base + h * (Kp / 2), *lh = lim + h * (Kp / 2);
    unsigned long long terms = 0;  // this wave's tiles left to the term-by-term sums (the last bit: and all after)
    int step = 0;
    for (int64_t tl = t_begin + wave; tl < t_end; tl += nw, ++step) {
      const int64_t x0 = tl * W, x = x0 + li * PW;  // this lane's positions x .. x + PW - 1
      v8bf bf[KS][PW][NP];
      // every load of the tile in flight before the first is used; past a row's valid
      // positions (EDGE: the last tiles) zeros, loaded from the row's start
      auto load = [&](auto edge_c) {
        constexpr bool EDGE = decltype(edge_c)::value;
        if constexpr (F32) {
          const float *G = static_cast<const float *>(a.G);
          float raw[KS][PW][8];
#pragma unroll
          for (int q = 0; q < KS; ++q)
#pragma unroll
            for (int i = 0; i < 8; ++i) {
              const float *src = G + bh[8 * q + i];
              if constexpr (EDGE) {
                const int64_t lm = lh[8 * q + i];
#pragma unroll
                for (int w = 0; w < PW; ++w) {
                  const float v = src[x + w < lm ? x + w : 0];
                  raw[q][w][i] = x + w < lm ? v : 0.f;
                }
              } else {
                const VT v = *reinterpret_cast<const VT *>(src + x);
                if constexpr (PW == 1) {
                  raw[q][0][i] = v;
                } else {
#pragma unroll
                  for (int w = 0; w < PW; ++w) raw[q][w][i] = v[w];
                }
              }
            }
#pragma unroll
          for (int q = 0; q < KS; ++q)
#pragma unroll
            for (int w = 0; w < PW; ++w) split3(raw[q][w], bf[q][w]);
        } else {
          static_assert(F32 || PW % 2 == 0, "bf16: pairs of positions");
          constexpr int PP = F32 ? 1 : PW / 2;
          const uint16_t *G = static_cast<const uint16_t *>(a.G);
          uint32_t raw[KS][8][PP];
#pragma unroll
          for (int q = 0; q < KS; ++q)
#pragma unroll
            for (int i = 0; i < 8; ++i) {
              const uint16_t *src = G + bh[8 * q + i];
              if constexpr (EDGE) {
                const int64_t lm = lh[8 * q + i];
#pragma unroll
                for (int w = 0; w < PP; ++w) {
                  const int64_t y = x + 2 * w;
                  const uint32_t lo = src[y < lm ? y : 0], hi = src[y + 1 < lm ? y + 1 : 0];
                  raw[q][i][w] = (y < lm ? lo : 0u) | (y + 1 < lm ? hi << 16 : 0u);
                }
              } else {
                const auto v = *reinterpret_cast<const HalfPairs<PP> *>(src + x);
#pragma unroll
                for (int w = 0; w < PP; ++w) raw[q][i][w] = v.v[w];
              }
            }
#pragma unroll
          for (int q = 0; q < KS; ++q)
#pragma unroll
            for (int w = 0; w < PP; ++w) {
              v4u e, o;  // the pair's even and odd position
#pragma unroll
              for (int j = 0; j < 4; ++j) {
                e[j] = __builtin_amdgcn_perm(raw[q][2 * j + 1][w], raw[q][2 * j][w], 0x05040100u);
                o[j] = __builtin_amdgcn_perm(raw[q][2 * j + 1][w], raw[q][2 * j][w], 0x07060302u);
              }
              bf[q][2 * w][0] = __builtin_bit_cast(v8bf, e);
              bf[q][2 * w + 1][0] = __builtin_bit_cast(v8bf, o);
            }
        }
      };
      if (x0 + W <= a.lmin) load(std::false_type{});
      else load(std::true_type{});
      // a sum that is a NaN once a value loaded is not finite
      float chk[4] = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
      for (int q = 0; q < KS; ++q)
#pragma unroll
        for (int w = 0; w < PW; ++w) {
          const v4u top = __builtin_bit_cast(v4u, bf[q][w][0]);
#pragma unroll
          for (int j = 0; j < 4; ++j) chk[j] = times_zero(top[j], chk[j]);
        }
      const float nan_if_bad = (chk[0] + chk[1]) + (chk[2] + chk[3]);
      if (__any(nan_if_bad != nan_if_bad)) {
        terms |= 1ull << (step < 63 ? step : 63);
        continue;
      }
      const bool inside = x0 + W <= a.L;
      float *Tx = Tw + x;
#pragma unroll 1
      for (int rt = 0; rt < ntile; ++rt) {
        const uint16_t *At = Ap + rt * (3 * 32 * AP) + li * AP + 8 * h;
        v16f acc[PW];
        auto mm = [&](v16f &sum, const uint16_t *plane, int q, int w, int part) {
          const v8bf av = *reinterpret_cast<const v8bf *>(plane + 16 * q);
          sum = __builtin_amdgcn_mfma_f32_32x32x16_bf16(av, bf[q][w][part], sum, 0, 0, 0);
        };
        // the products of parts above 2^-24 relative; those below 2^-7 of the whole first, over
        // all of K, so that only the last KS sums round at the result's own size
        if constexpr (Lay::APART) {
#pragma unroll
          for (int w = 0; w < PW; ++w) {
            v16f sum = v16f{};
            mm(sum, At + 64 * AP, 0, w, 0);
            if constexpr (F32) {
              mm(sum, At + 32 * AP, 0, w, 1);
              mm(sum, At, 0, w, 2);
            }
            mm(sum, At + 32 * AP, 0, w, 0);
            if constexpr (F32) mm(sum, At, 0, w, 1);
            acc[w] = sum;
            if constexpr (Lay::LEAN) __builtin_amdgcn_sched_barrier(0);
            v16f big = v16f{};
            mm(big, At, 0, w, 0);
            acc[w] = acc[w] + big;
            if constexpr (Lay::LEAN) __builtin_amdgcn_sched_barrier(0);
          }
        } else {
#pragma unroll
          for (int w = 0; w < PW; ++w) acc[w] = v16f{};
          auto each = [&](const uint16_t *plane, int q, int part) {
#pragma unroll
            for (int w = 0; w < PW; ++w) mm(acc[w], plane, q, w, part);
          };
#pragma unroll
          for (int q = 0; q < KS; ++q) {
            each(At + 64 * AP, q, 0);
            if constexpr (F32) {
              each(At + 32 * AP, q, 1);
              each(At, q, 2);
            }
            each(At + 32 * AP, q, 0);
            if constexpr (F32) each(At, q, 1);
          }
#pragma unroll
          for (int q = 0; q < KS; ++q) each(At, q, 0);
        }
        // lane (h, li) holds D[8(v/4) + 4h + v%4][li] of each 32-wide tile: rows 32 rt + 8g + 4h
        // + i, PW neighbouring positions each.  Non-temporal where rows start on 64-byte
        // boundaries; elsewhere the pieces of a row meet inside a memory line, which plain
        // stores let L2 put together (m = 37, L = 33335: 0.62 ms against 0.70)
        auto value = [&](int v) {
          VT o;
          if constexpr (PW == 1) {
            o = acc[0][v];
          } else {
#pragma unroll
            for (int w = 0; w < PW; ++w) o[w] = acc[w][v];
          }
          return o;
        };
        const int64_t *ro = rowoff + 32 * rt + 4 * h;
        auto full = [&](auto nt_c) {
#pragma unroll
          for (int g = 0; g < 4; ++g) {
            const longlong2 o0 = *reinterpret_cast<const longlong2 *>(ro + 8 * g);
            const longlong2 o1 = *reinterpret_cast<const longlong2 *>(ro + 8 * g + 2);
            const int64_t off[4] = {o0.x, o0.y, o1.x, o1.y};
#pragma unroll
            for (int i = 0; i < 4; ++i) {
              VT *dst = reinterpret_cast<VT *>(Tx + off[i]);
              if constexpr (decltype(nt_c)::value) __builtin_nontemporal_store(value(4 * g + i), dst);
              else *dst = value(4 * g + i);
            }
          }
        };
        if (inside && 32 * rt + 32 <= nsend) {
          if (a.nt) full(std::true_type{});
          else full(std::false_type{});
        } else {
#pragma unroll
          for (int v = 0; v < 16; ++v) {
            const int c = 8 * (v >> 2) + (v & 3);
            if (32 * rt + 4 * h + c >= nsend) continue;
            float *dst = Tx + ro[c];
            if (inside) {
              *reinterpret_cast<VT *>(dst) = value(v);
            } else {
#pragma unroll
              for (int w = 0; w < PW; ++w)
                if (x + w < a.L) dst[w] = acc[w][v];
            }
          }
        }
      }
    }
    for (int s = 0; terms >> (s < 63 ? s : 63); ++s) {
      const int64_t x0 = (t_begin + wave + int64_t(s) * nw) * W;
      if (x0 >= a.L || t_begin + wave + int64_t(s) * nw >= t_end) break;
      if ((terms >> (s < 63 ? s : 63)) & 1)
        mx_tile_terms<GT>(a, p0, j0, nsend, crow, cnp, x0, x0 + W < a.L ? x0 + W : a.L);
    }
  }
}

// The grid of a launch and its blocks: every (range, unit) pair, those of the ranges past whole eights
// in eight equal parts.  False past the launch limits.
bool mx_grid(MxArgs &a, int threads, int64_t *blocks) {
  const int64_t units = int64_t(a.ngroups) * a.ntp, eights = a.nsr & ~int64_t(7);
  const int64_t left = (a.nsr - eights) * units;
  *blocks = eights * units + 8 * ceil_div(left, 8);
  if (!grid_ok(*blocks, threads)) return false;
  a.units = uint32_t(units);
  a.whole = uint32_t(eights * units);
  a.left = uint32_t(left);
  a.eighth = uint32_t(ceil_div(left, 8));
  return true;
}

template <typename GT, int KS, int PW>
int launch_mx(const MxArgs &a, int64_t blocks, int threads, hipStream_t st) {
  const size_t lds = mx_lds(a, KS);
  if (hipFuncSetAttribute(reinterpret_cast<const void *>(&encode_mx_kernel<GT, KS, PW>),
                          hipFuncAttributeMaxDynamicSharedMemorySize, int(lds)) != hipSuccess)
    return GC_ELAUNCH;
  hipLaunchKernelGGL((encode_mx_kernel<GT, KS, PW>), dim3(unsigned(blocks)), dim3(threads), lds, st, a);
  return GC_OK;
}

}  // namespace

int encode_mx(const void *G, bool f32, int32_t N, int64_t d, const int32_t *psi, const int32_t *order,
              const float *Bc, int64_t P, int32_t m, int32_t delta, int32_t ell, float *T, hipStream_t stream) {
  MxArgs a{};
  a.G = G;
  a.N = N;
  a.d = d;
  a.L = ceil_div(d, ell);
  a.lmin = std::max<int64_t>(0, d - int64_t(ell - 1) * a.L);
  a.psi = psi;
  a.order = order;
  a.Bc = Bc;
  a.P = P;
  a.m = m;
  a.delta = delta;
  a.ell = ell;
  a.T = T;
  a.nt = a.L % 16 == 0 && (reinterpret_cast<uintptr_t>(T) & 63) == 0;
  auto steps = [&](int64_t slots) { return ceil_div(slots * ell, 16); };
  const int64_t max_steps = f32 ? kMxMaxKSF32 : kMxMaxKSBF16;
  if (steps(delta) > max_steps) return kEncodeMxNotApplicable;
  // Candidate rows per window: as many as the LDS allows, so that B is loaded and split
  // for more rows (fp32, ell = 8: 64 / 128 / 256 rows 4.5 / 4.1 / 3.8 ms; bf16, ell = 4: 64 /
  // 128 / 192 rows 2.4 / 2.1 / 2.05 ms).  With few K steps on rows that start anywhere 128 rows
  // and four positions per lane (0.62 ms against 0.65 with 256 rows, 0.68 with two positions).
  const bool small_odd = f32 && !a.nt && steps(delta) <= 2;
  // The same on rows at 64 bytes with many patterns: at most 32 patterns per K step and window, so
  // that a window takes several workers, and four positions per lane.  Windows of 256 patterns of one
  // worker wrote 256-byte pieces m rows apart, below the worker groups' rate (ms, one worker / this /
  // worker groups: m = 100, delta = 10, d = 2^20, ell = 1, 256 patterns 21.4 / 16.1 / 15.8, ell = 2, 512
  // patterns 24.3 / 17.7 / 22.8; m = 200, delta = 20, d = 2^18, 512 patterns 27.6 / 19.2 / 22.9; 64 patterns
  // per step / 32 / worker groups: m = 50, delta = 5, d = 2^14, ell = 2, 1000 patterns 0.276 / 0.251 / 0.417,
  // 10,000 2.39 / 2.32 / 2.19).
  const bool many = f32 && a.nt && steps(delta) <= 2 && P > 64;
  int KS = 0;
  for (int cw = small_odd ? 128 : (f32 ? kMxMaxCW : 192);; cw -= 32) {
    // one pattern window where P allows, else balanced ones; then workers while there is
    // room.  J workers share J + delta - 1 chunks under the cyclic order, so for each count of
    // K steps the most workers it holds, and of these the one with the least work per row: KS
    // products per row tile, and for each K step loads and splits that cost about as much as
    // 2.5 row tiles' products
    a.PB = int(ceil_div(P, ceil_div(P, many ? std::min<int64_t>(cw, 32 * steps(delta)) : cw)));
    a.ntp = ceil_div(P, a.PB);
    const int64_t most = N <= kMxMapChunks ? std::min<int64_t>(cw / a.PB, m) : 1;
    double best = 0;
    for (int64_t k = steps(delta); k <= (delta * ell <= kMxApartTerms ? 1 : max_steps); ++k) {
      int64_t J = std::max<int64_t>(1, std::min<int64_t>(16 * k / ell - delta + 1, most));
      const int64_t groups = ceil_div(m, J);
      J = ceil_div(m, groups);  // balanced groups
      const int64_t ks = std::min<int64_t>(k, steps(std::min<int64_t>(J + delta - 1, std::max(N, delta))));
      const double cost = double(ks) * double(2 * ceil_div(J * a.PB, 32) + 5) / double(J * a.PB);
      if (best == 0 || cost < best) {
        best = cost;
        a.J = int(J);
        a.ngroups = int(groups);
        KS = int(ks);
      }
      if (J >= most || J >= m) break;
    }
    a.slots = a.J == 1 ? delta : std::min<int>(16 * KS / ell, std::max(N, delta));
    a.CW = (a.J * a.PB + 31) & ~31;
    if (mx_lds(a, KS) <= kMxLds || cw == 32) break;  // 32 rows always fit
  }
  // positions per lane, as registers allow (fp32: 12 PW per K step, bf16 4 PW; 16 PW sums)
  const int64_t units = int64_t(a.ngroups) * a.ntp;
  const int pw = f32 ? (KS <= 2 ? (small_odd || many ? 4 : 2) : (KS <= 5 ? 2 : 1)) : (KS <= 8 ? 4 : 2);
  const int threads = KS <= (f32 ? 2 : 3) ? 256 : 512;
  const int nw = threads / kWave;
  a.ntiles = ceil_div(a.L, int64_t(32) * pw);
  // tiles per wave: the planes cost more to build with more K steps (2 up to 3 steps, else 8;
  // m = 200 bf16 at ell = 1 2.67 ms against 2.77 with 4, at ell = 4 2.05 against 2.31 with 2; 4 for
  // bf16 at two steps and many patterns: m = 200, delta = 20, d = 2^18, 128 patterns 3.94 against 4.40,
  // m = 100, delta = 16, ell = 2, 256 patterns 2.11 against 2.22, 64 patterns of m = 200 2.47 against 2.43),
  // fewer while the grid is short of four blocks per CU
  a.tpb = int64_t(nw) * (!f32 && KS == 2 && P > 64 ? 4 : (KS <= 3 ? 2 : 8));
  while (a.tpb > nw && ceil_div(a.ntiles, a.tpb) * units < 4 * int64_t(cu_count())) a.tpb -= nw;
  a.nsr = ceil_div(a.ntiles, a.tpb);
  int64_t blocks = 0;
  while (!mx_grid(a, threads, &blocks) && a.nsr > 1) {
    a.tpb *= 2;
    a.nsr = ceil_div(a.ntiles, a.tpb);
  }
  if (!mx_grid(a, threads, &blocks)) {  // so many windows: half of the patterns at a time
    const int64_t half = P / 2;
    const int st = encode_mx(G, f32, N, d, psi, order, Bc, half, m, delta, ell, T, stream);
    if (st != GC_OK) return st;
    return encode_mx(G, f32, N, d, psi + half * m, order, Bc + half * m * delta * ell, P - half, m, delta, ell,
                     T + half * m * a.L, stream);
  }
#define GC_BF16_CASE(K, PWN) \
  case K: return launch_mx<uint16_t, K, PWN>(a, blocks, threads, stream);
#define GC_F32_CASE(K, PWN) \
  case K: return launch_mx<float, K, PWN>(a, blocks, threads, stream);
  if (!f32) {
    switch (KS) {
      GC_BF16_CASE(1, 4) GC_BF16_CASE(2, 4) GC_BF16_CASE(3, 4) GC_BF16_CASE(4, 4) GC_BF16_CASE(5, 4)
      GC_BF16_CASE(6, 4) GC_BF16_CASE(7, 4) GC_BF16_CASE(8, 4) GC_BF16_CASE(9, 2) GC_BF16_CASE(10, 2)
      GC_BF16_CASE(11, 2) GC_BF16_CASE(12, 2)
    }
  } else if (pw == 4) {
    switch (KS) { GC_F32_CASE(1, 4) GC_F32_CASE(2, 4) }
  } else {
    switch (KS) {
      GC_F32_CASE(1, 2) GC_F32_CASE(2, 2) GC_F32_CASE(3, 2) GC_F32_CASE(4, 2) GC_F32_CASE(5, 2)
      GC_F32_CASE(6, 1) GC_F32_CASE(7, 1) GC_F32_CASE(8, 1) GC_F32_CASE(9, 1) GC_F32_CASE(10, 1)
      GC_F32_CASE(11, 1)
    }
  }
#undef GC_BF16_CASE
#undef GC_F32_CASE
  return kEncodeMxNotApplicable;
}

}  // namespace gcx
