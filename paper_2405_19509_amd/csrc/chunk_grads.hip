// gc_chunk_grads: per-chunk gradients g_{D_i} = X_i^T r_i (Sec. 1), with
// r_i = X_i w - y_i (linear) or sigmoid(X_i w) - y_i (logistic), at b
// evaluation points.
//
// For one evaluation point this is two matrix-vector products per chunk at
// about 1 flop per byte of X: HBM-bound, and X is the only large operand, so
// the goal is to read it exactly once.
//
// Fused path (d <= 16384, d % 4 == 0): fused_grad_kernel gives each block a
// contiguous range of sample rows (at most n, so it touches at most two
// chunks).  A 512-thread block holds a whole row in registers (8 float4 per
// thread at d = 16384) together with w and its running partial gradient:
// load the row once, reduce x.w across the block, form the residual, and add
// r * x into the partial.  Partials go to the workspace (two slots per
// block) and reduce_partials_kernel sums, for every chunk, the partials of
// the blocks that touched it, in block order: one read of X, deterministic.
//
// Many points (from 4 on, from 2 where the fused path does not apply): two matrix-core GEMMs
// per chunk (chunk_grads_mfma.hip), two reads of X in all.
//
// General path (any d, any alignment: and the fused one's d off 16-byte boundaries, where the
// workspace holds the residuals): two streaming kernels
//   dot_kernel   x.w of 4 rows (few rows: 1) over a segment of the columns by one wave, 16-byte
//                loads from any float on, w loaded once for the rows; several segments' sums
//                go to G and seg_residual_kernel adds them -> workspace residuals [b][N][n]
//   xtr_kernel   one block per (point, chunk, 1024 or 256 columns): the chunk's residuals
//                in LDS, then the columns down all n rows, 8 loads in flight; fixed summation
//                order -> deterministic.
// Both read X at the rate of the memory (X of 20 x 100 x 250001, 2 GB: 0.36 ms each, 5.5
// TB/s; scalar loads and one wave per row took 2.1 ms in all).
#include <algorithm>

#include "common.h"

namespace gcx {

// multi-point path on the matrix cores (chunk_grads_mfma.hip)
bool mfma_eligible(int N, int n, int64_t d, int b, bool fused, bool seg, int64_t room);
void launch_mfma_grads(const float *X, const float *y, const float *W, int N, int n, int64_t d, int b,
                      int loss, bool seg, int64_t room, float *G, void *workspace, hipStream_t st);

namespace {

constexpr int kGradThreads = 256;
constexpr int kGradWaves = kGradThreads / kWave;
constexpr int kResidStage = 2048;  // residuals staged in LDS per step

// rows of X and W start on any float
typedef float v4fu __attribute__((ext_vector_type(4), aligned(4)));

__device__ __forceinline__ float loss_residual(float z, float yv, int loss) {
  return loss == GC_LOSS_LOGISTIC ? 1.0f / (1.0f + expf(-z)) - yv : z - yv;
}

// out[row][seg] = sum over the columns of segment seg of x * w, for ROWS rows by one wave: w is
// read once for all of them.  One segment: the row's residual instead.
template <int ROWS>
__global__ __launch_bounds__(kGradThreads) void dot_kernel(const float *__restrict__ X, const float *__restrict__ W,
                                                           int64_t Nn, int64_t d, int64_t groups, int segs,
                                                           int64_t seglen, int64_t units, const float *__restrict__ y,
                                                           int loss, float *__restrict__ out) {
  const int lane = threadIdx.x % kWave;
  const int64_t u = int64_t(blockIdx.x) * kGradWaves + threadIdx.x / kWave;  // (q, row group, segment)
  if (u >= units) return;
  const int seg = int(u % segs);
  const int64_t q = u / segs / groups, r0 = u / segs % groups * ROWS;
  const int64_t c0 = seg * seglen, c1 = c0 + seglen < d ? c0 + seglen : d;
  const float *w = W + q * d;
  const float *x[ROWS];
#pragma unroll
  for (int r = 0; r < ROWS; ++r) x[r] = X + (r0 + r < Nn ? r0 + r : Nn - 1) * d;
  float s[ROWS][4];
#pragma unroll
  for (int r = 0; r < ROWS; ++r)
#pragma unroll
    for (int e = 0; e < 4; ++e) s[r][e] = 0.f;
  int64_t c = c0 + 4 * lane;
#pragma unroll 2
  for (; c + 4 <= c1; c += 4 * kWave) {
    const v4fu b = *reinterpret_cast<const v4fu *>(w + c);
    v4fu a[ROWS];
#pragma unroll
    for (int r = 0; r < ROWS; ++r) a[r] = *reinterpret_cast<const v4fu *>(x[r] + c);
#pragma unroll
    for (int r = 0; r < ROWS; ++r)
#pragma unroll
      for (int e = 0; e < 4; ++e) s[r][e] = fmaf(a[r][e], b[e], s[r][e]);
  }
  for (; c < c1; ++c)  // the lane with the segment's last one to three columns
#pragma unroll
    for (int r = 0; r < ROWS; ++r) s[r][0] = fmaf(x[r][c], w[c], s[r][0]);
#pragma unroll
  for (int r = 0; r < ROWS; ++r) {
    const float v = wave_sum((s[r][0] + s[r][1]) + (s[r][2] + s[r][3]));
    if (lane == 0 && r0 + r < Nn)
      out[(q * Nn + r0 + r) * segs + seg] = segs == 1 ? loss_residual(v, y[r0 + r], loss) : v;
  }
}

// The residuals from the segments' sums, added in order.
__global__ __launch_bounds__(kGradThreads) void seg_residual_kernel(const float *__restrict__ zpart,
                                                                    const float *__restrict__ y, int64_t rows,
                                                                    int64_t Nn, int segs, int loss,
                                                                    float *__restrict__ resid) {
  const int64_t row = int64_t(blockIdx.x) * kGradThreads + threadIdx.x;  // q*N*n + i*n + r
  if (row >= rows) return;
  const float *zp = zpart + row * segs;
  float z = 0.f;
#pragma unroll 8
  for (int g = 0; g < segs; ++g) z += zp[g];
  resid[row] = loss_residual(z, y[row % Nn], loss);
}

// G[q][i][x] = sum_r residual(q, i, r) * X[i][r][x].  A block takes 1024 / RS columns; its waves
// split the rows RS ways (wave w the rows of slice w % RS) and the slices are summed in order.
template <int RS>
__global__ __launch_bounds__(kGradThreads) void xtr_kernel(const float *__restrict__ X,
                                                           const float *__restrict__ resid, int N, int n, int64_t d,
                                                           int64_t tiles, float *__restrict__ G) {
  __shared__ float rs[kResidStage];
  __shared__ float part[RS > 1 ? RS - 1 : 1][kGradThreads / RS][4];
  const int64_t tile = blockIdx.x % tiles;
  const int64_t q = blockIdx.x / tiles / N;
  const int64_t i = N - 1 - blockIdx.x / tiles % N;  // descending: the last rows read are still cached
  const int64_t qi = q * N + i;
  const int slice = RS > 1 ? threadIdx.x / (kGradThreads / RS) : 0;
  const int64_t x = (tile * (kGradThreads / RS) + threadIdx.x % (kGradThreads / RS)) * 4;
  // columns xs .. xs + 3: past the end the last four, of which those from x on are stored
  const int64_t xs = d < 4 || x + 4 <= d ? x : d - 4;
  const float *Xi = X + i * int64_t(n) * d;
  float acc[4] = {0.f, 0.f, 0.f, 0.f};
  for (int r0 = 0; r0 < n; r0 += kResidStage) {
    const int rn = n - r0 < kResidStage ? n - r0 : kResidStage;
    __syncthreads();
    for (int a = threadIdx.x; a < rn; a += kGradThreads) rs[a] = resid[qi * n + r0 + a];
    __syncthreads();
    const int per = (rn + RS - 1) / RS;
    int r = slice * per;
    const int re = r + per < rn ? r + per : rn;
    const float *xp = Xi + int64_t(r0) * d + xs;
    if (d >= 4) {
      for (; r + 8 <= re; r += 8) {
        v4fu v[8];
#pragma unroll
        for (int u = 0; u < 8; ++u) v[u] = *reinterpret_cast<const v4fu *>(xp + int64_t(r + u) * d);
#pragma unroll
        for (int u = 0; u < 8; ++u) {
          const float c = rs[r + u];
#pragma unroll
          for (int e = 0; e < 4; ++e) acc[e] = fmaf(c, v[u][e], acc[e]);
        }
      }
      for (; r < re; ++r) {
        const v4fu v = *reinterpret_cast<const v4fu *>(xp + int64_t(r) * d);
#pragma unroll
        for (int e = 0; e < 4; ++e) acc[e] = fmaf(rs[r], v[e], acc[e]);
      }
    } else {
      for (; r < re; ++r)
#pragma unroll
        for (int e = 0; e < 3; ++e)
          if (xs + e < d) acc[e] = fmaf(rs[r], xp[int64_t(r) * d + e], acc[e]);
    }
  }
  if constexpr (RS > 1) {
    const int col = threadIdx.x % (kGradThreads / RS);
    if (slice > 0)
#pragma unroll
      for (int e = 0; e < 4; ++e) part[slice - 1][col][e] = acc[e];
    __syncthreads();
    if (slice > 0) return;
#pragma unroll
    for (int v = 0; v < RS - 1; ++v)
#pragma unroll
      for (int e = 0; e < 4; ++e) acc[e] += part[v][col][e];
  }
  float *dst = G + qi * d + xs;
  if (x + 4 <= d) {
    *reinterpret_cast<v4fu *>(dst) = v4fu{acc[0], acc[1], acc[2], acc[3]};
  } else {
#pragma unroll
    for (int e = 0; e < 4; ++e)
      if (xs + e >= x && xs + e < d) dst[e] = acc[e];
  }
}

// Rows per wave, row groups and column segments of dot_kernel per point.  Segments of at least
// 4096 columns, whose sums' launch costs what shorter ones save (us, 1024 / 4096: X of 9 x 131 x 2101
// 16.4 / 14.2, 9 x 131 x 4101 17.2 / 15.0, 3 x 20 x 400001 56 / 42; one segment of 16385 40), as many
// as give every CU 32 waves; one row per wave where four would leave the CUs short of 8 waves.  The segments' sums go to G, which is
// written after they have been read: at most d / n segments.
struct DotPlan {
  int rows;
  int64_t groups, seglen;
  int segs;
};

inline DotPlan dot_plan(int N, int n, int64_t d, int b) {
  DotPlan dp{};
  const int64_t R = int64_t(N) * n, most = std::max<int64_t>(1, std::min(d / 4096, d / n));
  dp.rows = ceil_div(R, 4) * b * most < 2048 ? 1 : 4;
  dp.groups = ceil_div(R, dp.rows);
  const int64_t segs = std::max<int64_t>(1, std::min(ceil_div(8192, dp.groups * b), most));
  dp.seglen = ceil_div(ceil_div(d, segs), 4) * 4;
  dp.segs = int(ceil_div(d, dp.seglen));
  return dp;
}

constexpr int kFusedThreads = 512;
constexpr int kFusedWaves = kFusedThreads / kWave;
constexpr int kFusedMaxNV = 8;  // float4 per thread: d <= 512 * 4 * 8 = 16384

struct FusedPlan {
  int64_t blocks;          // blocks per evaluation point
  int64_t rows_per_block;  // <= n
};

// Splits of the columns that the workspace of a call in whole quads has partial sums for: up to 16, as
// many as fill whole rounds of 512 tiles of 128 rows x 128 or 64 points.
int64_t quad_splits(int N, int n, int64_t d, int b) {
  const int64_t tiles = int64_t(N) * ceil_div(n, 128) * ceil_div(b, b % 128 == 0 ? 128 : 64);
  int64_t splits = 1;
  double best = -1.0;
  for (int64_t sp = 1; sp <= 16; ++sp) {
    const int64_t kp = ceil_div(ceil_div(d, sp), 32) * 32;
    if (ceil_div(d, kp) != sp) continue;
    const int64_t blocks = tiles * sp;
    const double score = double(blocks) / double(ceil_div(blocks, 512) * 512) - 0.005 * double(sp);
    if (score > best + 1e-9) {
      best = score;
      splits = sp;
    }
  }
  return splits;
}

inline FusedPlan fused_plan(int N, int n) {
  const int64_t R = int64_t(N) * n;
  int64_t blocks = 512;  // two 512-thread blocks per CU on 256 CUs
  if (blocks < N) blocks = N;
  int64_t rpb = ceil_div(R, blocks);
  if (rpb > n) rpb = n;
  return FusedPlan{ceil_div(R, rpb), rpb};
}

template <int NV>
__global__ __launch_bounds__(kFusedThreads) void fused_grad_kernel(
    const float *__restrict__ X, const float *__restrict__ y, const float *__restrict__ W, int N,
    int n, int64_t d, int loss, int64_t rows_per_block, int64_t blocks, float *__restrict__ part) {
  __shared__ float red[2][kFusedWaves];
  const int q = blockIdx.y;
  const int64_t b = blockIdx.x;
  const int64_t R = int64_t(N) * n;
  const int64_t r0 = b * rows_per_block;
  const int64_t r1 = r0 + rows_per_block < R ? r0 + rows_per_block : R;
  const int64_t d4 = d / 4;
  const int lane = threadIdx.x % kWave, wave = threadIdx.x / kWave;

  v4fu w[NV], acc[NV];  // rows start on any float
  const v4fu *w4 = reinterpret_cast<const v4fu *>(W + int64_t(q) * d);
#pragma unroll
  for (int v = 0; v < NV; ++v) {
    const int64_t c = threadIdx.x + int64_t(kFusedThreads) * v;
    w[v] = c < d4 ? w4[c] : v4fu{0.f, 0.f, 0.f, 0.f};
    acc[v] = v4fu{0.f, 0.f, 0.f, 0.f};
  }
  const int64_t c0 = r0 / n;  // first chunk of this block
  int64_t cur = c0;
  float *slot = part + ((int64_t(q) * blocks + b) * 2) * d;

  auto flush = [&](int64_t chunk) {
    v4fu *dst = reinterpret_cast<v4fu *>(slot + (chunk - c0) * d);
#pragma unroll
    for (int v = 0; v < NV; ++v) {
      const int64_t c = threadIdx.x + int64_t(kFusedThreads) * v;
      if (c < d4) dst[c] = acc[v];
      acc[v] = v4fu{0.f, 0.f, 0.f, 0.f};
    }
  };

  for (int64_t r = r0; r < r1; ++r) {
    const int64_t c = r / n;
    if (c != cur) {
      flush(cur);
      cur = c;
    }
    const v4fu *x4 = reinterpret_cast<const v4fu *>(X + r * d);
    v4fu x[NV];
#pragma unroll
    for (int v = 0; v < NV; ++v) {
      const int64_t cc = threadIdx.x + int64_t(kFusedThreads) * v;
      x[v] = cc < d4 ? x4[cc] : v4fu{0.f, 0.f, 0.f, 0.f};
    }
    float s = 0.f;
#pragma unroll
    for (int v = 0; v < NV; ++v) {
      s = fmaf(x[v].x, w[v].x, s);
      s = fmaf(x[v].y, w[v].y, s);
      s = fmaf(x[v].z, w[v].z, s);
      s = fmaf(x[v].w, w[v].w, s);
    }
    s = wave_sum(s);
    const int par = int(r & 1);  // two buffers: one barrier per row suffices
    if (lane == 0) red[par][wave] = s;
    __syncthreads();
    float z = 0.f;
#pragma unroll
    for (int k = 0; k < kFusedWaves; ++k) z += red[par][k];
    const float u = loss_residual(z, y[r], loss);
#pragma unroll
    for (int v = 0; v < NV; ++v) {
      acc[v].x = fmaf(u, x[v].x, acc[v].x);
      acc[v].y = fmaf(u, x[v].y, acc[v].y);
      acc[v].z = fmaf(u, x[v].z, acc[v].z);
      acc[v].w = fmaf(u, x[v].w, acc[v].w);
    }
  }
  if (r1 > r0) flush(cur);
}

// G[q][i][x] = sum over the blocks b that touched chunk i (ascending) of their partial.
__global__ void reduce_partials_kernel(const float *__restrict__ part, int N, int n, int64_t d,
                                       int64_t rows_per_block, int64_t blocks, float *__restrict__ G) {
  const int64_t x4 = int64_t(blockIdx.x) * blockDim.x + threadIdx.x;
  const int64_t i = blockIdx.y;
  const int q = blockIdx.z;
  if (x4 * 4 >= d) return;
  const int64_t bfirst = (i * n) / rows_per_block;
  const int64_t blast = ((i + 1) * n - 1) / rows_per_block;
  v4fu s = {0.f, 0.f, 0.f, 0.f};
  for (int64_t b = bfirst; b <= blast; ++b) {
    const int64_t c0 = (b * rows_per_block) / n;
    const v4fu v = reinterpret_cast<const v4fu *>(part + ((int64_t(q) * blocks + b) * 2 + (i - c0)) * d)[x4];
    s.x += v.x; s.y += v.y; s.z += v.z; s.w += v.w;
  }
  reinterpret_cast<v4fu *>(G + (int64_t(q) * N + i) * d)[x4] = s;
}

}  // namespace
}  // namespace gcx

namespace {
bool fused_ok(int64_t d) { return d % 4 == 0 && d <= int64_t(gcx::kFusedThreads) * 4 * gcx::kFusedMaxNV; }
}  // namespace

namespace {
// X [N][n][d], W [b][d], G [b][N][d], residuals [b][N][n]
bool grad_sizes_ok(int32_t N, int32_t n, int64_t d, int32_t b) {
  return N >= 1 && n >= 1 && d >= 1 && b >= 1 && gcx::sizes_ok({N, n, d}) && gcx::sizes_ok({b, N, d}) &&
         gcx::sizes_ok({b, N, n});
}
}  // namespace

// The fused path's partials, else the residuals and, from 16 points in whole quads on, room for
// partial sums of the first product.
extern "C" size_t gc_chunk_grads_workspace_size(int32_t N, int32_t n, int64_t d, int32_t b) {
  if (!grad_sizes_ok(N, n, d, b)) return 0;
  const size_t resid = sizeof(float) * size_t(b) * size_t(N) * size_t(n);
  if (b >= 16 && b % 4 == 0 && d % 4 == 0) return resid * size_t(1 + gcx::quad_splits(N, n, d, b));
  if (fused_ok(d)) {
    const gcx::FusedPlan fp = gcx::fused_plan(N, n);
    return sizeof(float) * size_t(b) * size_t(fp.blocks) * 2 * size_t(d);
  }
  return resid;
}

extern "C" int gc_chunk_grads(const float *X, const float *y, const float *W, int32_t N, int32_t n,
                              int64_t d, int32_t b, int32_t loss, float *G, void *workspace,
                              size_t workspace_bytes, hipStream_t stream) {
  using namespace gcx;
  if (!grad_sizes_ok(N, n, d, b)) return GC_EINVAL;
  if (loss != GC_LOSS_LINEAR && loss != GC_LOSS_LOGISTIC) return GC_EINVAL;
  if (!X || !y || !W || !G || !workspace) return GC_EINVAL;
  if (workspace_bytes < gc_chunk_grads_workspace_size(N, n, d, b)) return GC_EINVAL;
  const int64_t rows = int64_t(b) * N * n;
  const bool vec4 = d % 4 == 0 && aligned16(X) && aligned16(W) && aligned16(G);
  const int64_t tiles = ceil_div(d, int64_t(kGradThreads) * (vec4 ? 4 : 1));
  if (!grid_ok(ceil_div(rows, kGradWaves), kGradThreads) || !grid_ok(int64_t(b) * N * tiles, kGradThreads))
    return GC_EINVAL;
  const int dev = check_device();
  if (dev != GC_OK) return dev;
  (void)hipGetLastError();
  // 16 points or more in whole quads are taken on 16-byte boundaries only
  if (b >= 16 && b % 4 == 0 && d % 4 == 0 && (!vec4 || !aligned16(y) || !aligned16(workspace))) return GC_EINVAL;
  const bool enough = workspace_bytes >= sizeof(float) * size_t(rows);  // the residuals, and below the partials
  // the fused kernel on 16-byte boundaries, and on any floats where its partials are all that the
  // workspace holds (rows of few columns)
  const bool fused = fused_ok(d) && ((vec4 && aligned16(workspace)) || !enough) &&
                     workspace_bytes >= sizeof(float) * size_t(b) * size_t(fused_plan(N, n).blocks) * 2 * size_t(d);
  // Calls that the fused kernel could take (its sums are short: one row's products spread over a block,
  // a block's rows) are summed in segments on the matrix cores, for no larger an error (X of 20 x 512 x
  // 16384, 4 points: fused 1.7e-7 in 0.46 ms, matrix cores 2.1e-7 in 0.23, in segments 1.5e-7 in
  // 0.27; 20 x 8192 x 512: 1.3e-7, 4.9e-7, 1.0e-7).  Whole quads from 16 points on had longer ones.
  const bool seg = fused_ok(d) && (b < 16 || b % 4 != 0);
  // partial sums of the first product that a workspace of the size asked for has room for beside the
  // residuals
  const int64_t room = int64_t(gc_chunk_grads_workspace_size(N, n, d, b) / (sizeof(float) * size_t(rows))) - 1;
  if (enough && mfma_eligible(N, n, d, b, fused, seg, room)) {
    launch_mfma_grads(X, y, W, N, n, d, b, loss, seg, room, G, workspace, stream);
    return launch_status();
  }
  if (fused) {
    const FusedPlan fp = fused_plan(N, n);
    if (!grid_ok(fp.blocks * b, kFusedThreads)) return GC_EINVAL;
    float *part = static_cast<float *>(workspace);
    const int nv = int(ceil_div(d, int64_t(kFusedThreads) * 4));
    const dim3 g1(unsigned(fp.blocks), unsigned(b));
#define GC_FUSED(NV)                                                                              \
  hipLaunchKernelGGL(fused_grad_kernel<NV>, g1, dim3(kFusedThreads), 0, stream, X, y, W, N, n, d, \
                     loss, fp.rows_per_block, fp.blocks, part)
    if (nv <= 1) GC_FUSED(1);
    else if (nv <= 2) GC_FUSED(2);
    else if (nv <= 4) GC_FUSED(4);
    else GC_FUSED(8);
#undef GC_FUSED
    const dim3 g2(unsigned(ceil_div(d / 4, 256)), unsigned(N), unsigned(b));
    hipLaunchKernelGGL(reduce_partials_kernel, g2, dim3(256), 0, stream, part, N, n, d,
                       fp.rows_per_block, fp.blocks, G);
    return launch_status();
  }
  float *resid = static_cast<float *>(workspace);
  const DotPlan dp = dot_plan(N, n, d, b);
  float *sums = dp.segs > 1 ? G : resid;
  const int64_t units = dp.groups * dp.segs * b;
  const dim3 g1(unsigned(ceil_div(units, kGradWaves)));
  if (dp.rows == 4)
    hipLaunchKernelGGL(dot_kernel<4>, g1, dim3(kGradThreads), 0, stream, X, W, int64_t(N) * n, d, dp.groups,
                       dp.segs, dp.seglen, units, y, loss, sums);
  else
    hipLaunchKernelGGL(dot_kernel<1>, g1, dim3(kGradThreads), 0, stream, X, W, int64_t(N) * n, d, dp.groups,
                       dp.segs, dp.seglen, units, y, loss, sums);
  if (dp.segs > 1)
    hipLaunchKernelGGL(seg_residual_kernel, dim3(unsigned(ceil_div(rows, kGradThreads))), dim3(kGradThreads), 0,
                       stream, sums, y, rows, int64_t(N) * n, dp.segs, loss, resid);
  // few column tiles: four waves of a block split the rows instead of the columns
  const int64_t wide = ceil_div(d, 4 * kGradThreads) * N * b;
  if (wide >= 4 * int64_t(cu_count())) {
    hipLaunchKernelGGL(xtr_kernel<1>, dim3(unsigned(wide)), dim3(kGradThreads), 0, stream, X, resid, N, n, d,
                       ceil_div(d, 4 * kGradThreads), G);
  } else {
    const int64_t tiles = ceil_div(d, kGradThreads);
    hipLaunchKernelGGL(xtr_kernel<4>, dim3(unsigned(tiles * N * b)), dim3(kGradThreads), 0, stream, X, resid, N,
                       n, d, tiles, G);
  }
  return launch_status();
}
