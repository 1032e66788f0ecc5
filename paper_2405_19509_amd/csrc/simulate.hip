// The paper's straggler simulation (Sec. 4) on the GPU: worker progress at a
// grid of deadlines, and exact-GC completion times for the proposed protocol and
// for original GC.  Worker j processes the chunks of its order one after the
// other; the chunk at position t is finished at sum_{u <= t} tau[r][j][u]; a
// failed worker finishes nothing.  All times are fp64 and summed in position
// order, so every comparison with a deadline is reproducible bit for bit.
#include "common.h"

namespace gcx {
namespace {

constexpr int kSimThreads = 256;
constexpr int kSimWaves = kSimThreads / kWave;

// psi[r][g][j] = #{t : sum_{u <= t} tau[r][j][u] <= T[g]}, 0 for failed workers.  One thread per
// (trial, worker).  D: the finish times are summed once and held in registers (delta <= D); 0: any
// delta, summed again for every deadline (m = 200, delta = 8, 200 trials, 16 deadlines: 6 us
// against 15).
template <int D>
__global__ __launch_bounds__(kSimThreads) void progress_kernel(const double *__restrict__ tau,
                                                               const uint8_t *__restrict__ failed,
                                                               int64_t R, int m, int delta,
                                                               const double *__restrict__ T, int G,
                                                               int32_t *__restrict__ psi) {
  const int64_t e = int64_t(blockIdx.x) * kSimThreads + threadIdx.x;  // (r, j)
  if (e >= R * m) return;
  const int64_t r = e / m;
  const int j = int(e % m);
  const double *tj = tau + e * delta;
  const bool dead = failed != nullptr && failed[e] != 0;
  if constexpr (D > 0) {
    double at[D];  // loaded together, then summed in position order; +NaN past delta: never <= T
#pragma unroll
    for (int t = 0; t < D; ++t) at[t] = tj[t < delta ? t : delta - 1];
    double c = 0.0;
#pragma unroll
    for (int t = 0; t < D; ++t) {
      c += at[t];
      at[t] = t < delta && !dead ? c : __longlong_as_double(0x7ff8000000000000ll);
    }
    for (int g = 0; g < G; ++g) {
      const double Tg = T[g];
      int cnt = 0;
#pragma unroll
      for (int t = 0; t < D; ++t) cnt += at[t] <= Tg ? 1 : 0;
      psi[(r * G + g) * m + j] = cnt;
    }
  } else {
    for (int g = 0; g < G; ++g) {
      int cnt = 0;
      if (!dead) {
        double c = 0.0;
        for (int t = 0; t < delta; ++t) {
          c += tj[t];
          cnt += c <= T[g] ? 1 : 0;
        }
      }
      psi[(r * G + g) * m + j] = cnt;
    }
  }
}

// The ell-th smallest of a stream of values, kept as a sorted prefix of ELLMAX.
template <int ELLMAX>
struct Smallest {
  double v[ELLMAX];
  __device__ void init() {
#pragma unroll
    for (int a = 0; a < ELLMAX; ++a) v[a] = INFINITY;
  }
  __device__ void push(double x) {
#pragma unroll
    for (int a = 0; a < ELLMAX; ++a) {
      const double lo = fmin(v[a], x), hi = fmax(v[a], x);
      v[a] = lo;
      x = hi;
    }
  }
};

// Chunk i reaches ell processed copies at the ell-th smallest finish time over its holders; the
// protocol can decode once every chunk has (the proposed protocol), and original GC once every
// chunk has ell holders that finished *all* their chunks.  A block per trial (and every
// gridDim.x-th one after it where the trials pass the launch limits): the workers'
// finish times are summed once, in position order, into LDS ([m][delta], +inf for failed
// workers), then one thread per chunk (m = 200, delta = 8, 200 trials: 7 us; a wave per trial that
// summed the times again for every holder took 42).  Where they do not fit (kCompleteLds), LDS is
// not used and every holder's times are summed where they are needed.
constexpr size_t kCompleteLds = 64 * 1024;

__global__ __launch_bounds__(kSimThreads) void completion_kernel(
    const double *__restrict__ tau, const uint8_t *__restrict__ failed, int64_t R, int N, int m, int delta,
    const int32_t *__restrict__ holder, const int32_t *__restrict__ hpos, int gamma, int ell, int staged,
    double *__restrict__ partial, double *__restrict__ original) {
  extern __shared__ double done[];  // [m][delta] (staged)
  __shared__ double red[2][kSimWaves];
  for (int64_t r = blockIdx.x; r < R; r += gridDim.x) {
  const double *tr = tau + r * int64_t(m) * delta;
  if (staged) {
    for (int j = threadIdx.x; j < m; j += kSimThreads) {
      const bool dead = failed != nullptr && failed[r * m + j] != 0;
      double c = 0.0;
      for (int t = 0; t < delta; ++t) {
        c += tr[j * delta + t];
        done[j * delta + t] = dead ? INFINITY : c;
      }
    }
    __syncthreads();
  }
  double worst_p = 0.0, worst_o = 0.0;
  for (int i = threadIdx.x; i < N; i += kSimThreads) {
    Smallest<GC_MAX_ELL> sp, so;
    sp.init();
    so.init();
    for (int u = 0; u < gamma; ++u) {
      const int j = holder[int64_t(i) * gamma + u], t = hpos[int64_t(i) * gamma + u];
      if (j < 0 || j >= m || t < 0 || t >= delta) continue;
      if (staged) {  // a failed worker's +inf changes nothing
        sp.push(done[j * delta + t]);
        so.push(done[j * delta + delta - 1]);
        continue;
      }
      if (failed != nullptr && failed[r * m + j] != 0) continue;
      const double *tj = tr + int64_t(j) * delta;
      double c = 0.0, at = 0.0;
      for (int v = 0; v < delta; ++v) {
        c += tj[v];
        if (v == t) at = c;
      }
      sp.push(at);
      so.push(c);
    }
    double fp = INFINITY, fo = INFINITY;
#pragma unroll
    for (int a = 0; a < GC_MAX_ELL; ++a)
      if (a == ell - 1) {
        fp = sp.v[a];
        fo = so.v[a];
      }
    worst_p = fmax(worst_p, fp);
    worst_o = fmax(worst_o, fo);
  }
#pragma unroll
  for (int off = 32; off > 0; off >>= 1) {
    worst_p = fmax(worst_p, __shfl_xor(worst_p, off, kWave));
    worst_o = fmax(worst_o, __shfl_xor(worst_o, off, kWave));
  }
  if (threadIdx.x % kWave == 0) {
    red[0][threadIdx.x / kWave] = worst_p;
    red[1][threadIdx.x / kWave] = worst_o;
  }
  __syncthreads();
  if (threadIdx.x == 0) {
    for (int w = 1; w < kSimWaves; ++w) {
      worst_p = fmax(worst_p, red[0][w]);
      worst_o = fmax(worst_o, red[1][w]);
    }
    partial[r] = worst_p;
    original[r] = worst_o;
  }
  if (r + gridDim.x < R) __syncthreads();  // the next trial overwrites the times and the waves' maxima
  }  // trials
}

// Sum over the wave by DPP, without LDS: lane i of each row of 16 adds lanes i - 1, i - 2, i - 4 and
// i - 8, so its lane 15 holds the row's sum; rows 1 and 3 add the row before, rows 2 and 3 the sum of
// rows 0 and 1; lane 63's total is returned to every lane.
template <int CTRL, int ROWS>
__device__ __forceinline__ double dpp_add(double v) {
  const int lo = __builtin_amdgcn_update_dpp(0, __double2loint(v), CTRL, ROWS, 0xf, false);
  const int hi = __builtin_amdgcn_update_dpp(0, __double2hiint(v), CTRL, ROWS, 0xf, false);
  return v + __hiloint2double(hi, lo);
}
__device__ __forceinline__ double wave_sum_dpp(double v) {
  v = dpp_add<0x111, 0xf>(v);  // row_shr:1
  v = dpp_add<0x112, 0xf>(v);  // row_shr:2
  v = dpp_add<0x114, 0xf>(v);  // row_shr:4
  v = dpp_add<0x118, 0xf>(v);  // row_shr:8
  v = dpp_add<0x142, 0xa>(v);  // row_bcast:15 into rows 1, 3
  v = dpp_add<0x143, 0xc>(v);  // row_bcast:31 into rows 2, 3
  return __hiloint2double(__builtin_amdgcn_readlane(__double2hiint(v), 63),
                          __builtin_amdgcn_readlane(__double2loint(v), 63));
}

// Original GC's approximate decoding for one pattern per wave: CGLS on min ||A_F r - 1|| (A the
// 0/1 support, F the workers that processed all their chunks), from r = 0 so it converges to the
// minimum-norm solution; fp64.  err = ||A_F r - 1||^2 at exit.
// An iteration is two sparse products and two sums over 2 x max(N, m) values, all latency: a wave
// per pattern needs no block barriers (a block per pattern took eight per iteration), its vectors
// are registers (C values per lane, chunks and finished workers lane, lane + 64, ...), and only
// the two gathered vectors and the tables (16-bit, transposed so that lanes read neighbours,
// shared by the block) are in LDS.  Workers that have not finished are left out of the list of
// columns and stay zero in the direction.  m = 200, delta = 8, 3200 patterns of up to 172
// iterations: 0.43 ms against 3.2, now bound by the gathers' LDS bank conflicts (about 14 clocks
// per read).
// Tables past kLsTables bytes stay in global memory (TL false).  GD: with at most GD holders and
// positions a lane's table entries are read once, into registers (two byte offsets each), so that
// every gather of a product is in flight at once (0.43 ms against 0.65 with table reads in the loop).
constexpr int kLsWaves = 4;
constexpr size_t kLsTables = 64 * 1024;

__host__ __device__ inline size_t ls_tables(int N, int m, int delta, int gamma) {
  return (2 * (size_t(gamma) * N + size_t(delta) * m) + 7) & ~size_t(7);
}
__host__ __device__ inline size_t ls_wave(int N, int m) {
  return (sizeof(double) * (size_t(N) + m + 2) + 2 * size_t(m) + 7) & ~size_t(7);
}

template <int C, bool TL, int GD>
__global__ __launch_bounds__(kLsWaves * kWave) void original_ls_kernel(
    const int32_t *__restrict__ psi, int64_t P, int N, int m, const int32_t *__restrict__ order, int delta,
    const int32_t *__restrict__ holder, int gamma, int max_iter, double tol, double *__restrict__ err,
    int32_t *__restrict__ iters) {
  extern __shared__ __align__(16) unsigned char ls_sh[];
  uint16_t *hold = reinterpret_cast<uint16_t *>(ls_sh);  // [gamma][N]; m: no holder
  uint16_t *ord = hold + size_t(gamma) * N;              // [delta][m]; N: no chunk
  const int lane = threadIdx.x % kWave, wave = threadIdx.x / kWave;
  double *resS = reinterpret_cast<double *>(ls_sh + (TL ? ls_tables(N, m, delta, gamma) : 0) +
                                            wave * ls_wave(N, m));  // [N + 1]; entry N: 0
  double *pvS = resS + N + 1;                                       // [m + 1]; entry m: 0
  uint16_t *fin = reinterpret_cast<uint16_t *>(pvS + m + 1);  // the finished workers, ascending
  auto holder_at = [&](int i, int u) {
    if constexpr (TL) return int(hold[u * N + i]);
    const int j = holder[int64_t(i) * gamma + u];
    return j >= 0 && j < m ? j : m;
  };
  auto chunk_at = [&](int j, int t) {
    if constexpr (TL) return int(ord[t * m + j]);
    const int c = order[int64_t(j) * delta + t];
    return c >= 0 && c < N ? c : N;
  };
  if constexpr (TL) {
    for (int e = threadIdx.x; e < N * gamma; e += blockDim.x) {
      const int j = holder[e];
      hold[(e % gamma) * N + e / gamma] = uint16_t(j >= 0 && j < m ? j : m);
    }
    for (int e = threadIdx.x; e < m * delta; e += blockDim.x) {
      const int c = order[e];
      ord[(e % delta) * m + e / delta] = uint16_t(c >= 0 && c < N ? c : N);
    }
  }
  __syncthreads();  // the only block barrier
  const int64_t p = int64_t(blockIdx.x) * kLsWaves + wave;
  if (p >= P) return;
  auto lds_done = [&]() {  // the wave's LDS writes are seen by its later reads
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
  };
  int nf = 0;
  for (int j0 = 0; j0 < m; j0 += kWave) {
    const int j = j0 + lane;
    int load = 0;
    for (int t = 0; t < delta && j < m; ++t) load += chunk_at(j, t) < N ? 1 : 0;
    const bool on = j < m && load > 0 && psi[p * m + j] >= load;
    const unsigned long long mk = __ballot(on);
    if (on) fin[nf + __popcll(mk & ((1ull << lane) - 1))] = uint16_t(j);
    if (j < m) pvS[j] = 0.0;
    nf += __popcll(mk);
  }
  if (lane == 0) {
    resS[N] = 0.0;
    pvS[m] = 0.0;
  }
  for (int i = lane; i < N; i += kWave) resS[i] = 1.0;
  lds_done();

  double res[C], q[C], sv[C], pv[C], rv[C];
  int col[C];  // this lane's finished workers, m past the last
#pragma unroll
  for (int c = 0; c < C; ++c) {
    const int k = lane + c * kWave;
    col[c] = k < nf ? fin[k] : m;
    res[c] = k < N ? 1.0 : 0.0;
    pv[c] = rv[c] = 0.0;
  }
  uint32_t hreg[GD > 0 ? C : 1][GD > 0 ? GD / 2 : 1], oreg[GD > 0 ? C : 1][GD > 0 ? GD / 2 : 1];
  if constexpr (GD > 0) {
#pragma unroll
    for (int c = 0; c < C; ++c) {
      const int k = lane + c * kWave;
#pragma unroll
      for (int u = 0; u < GD; u += 2) {
        uint32_t hw = 0, ow = 0;
#pragma unroll
        for (int e = 0; e < 2; ++e) {
          hw |= uint32_t(8 * (k < N && u + e < gamma ? holder_at(k, u + e) : m)) << (16 * e);
          ow |= uint32_t(8 * (col[c] < m && u + e < delta ? chunk_at(col[c], u + e) : N)) << (16 * e);
        }
        hreg[c][u / 2] = hw;
        oreg[c][u / 2] = ow;
      }
    }
  }
  // the sum of GD entries of a vector in LDS at packed byte offsets (past the last: its zero)
  auto gather = [&](const double *v, const uint32_t (&at)[GD > 0 ? GD / 2 : 1]) {
    double x[GD > 0 ? GD : 1];
#pragma unroll
    for (int u = 0; u < GD; u += 2) {
      x[u] = *reinterpret_cast<const double *>(reinterpret_cast<const char *>(v) + (at[u / 2] & 0xffffu));
      x[u + 1] = *reinterpret_cast<const double *>(reinterpret_cast<const char *>(v) + (at[u / 2] >> 16));
    }
    double a = 0.0;
#pragma unroll
    for (int u = 0; u < GD; ++u) a += x[u];
    return a;
  };
  auto AT = [&]() {  // sv = A_F^T res
    double part = 0.0;
#pragma unroll
    for (int c = 0; c < C; ++c) {
      sv[c] = 0.0;
      if constexpr (GD > 0) {  // columns past the last gather zeros
        sv[c] = c * kWave < nf ? gather(resS, oreg[c]) : 0.0;
        part += sv[c] * sv[c];
      } else if (c * kWave < nf) {
        double a = 0.0;
        const int j = col[c] < m ? col[c] : 0;
#pragma unroll 4
        for (int t = 0; t < delta; ++t) a += resS[chunk_at(j, t)];
        sv[c] = col[c] < m ? a : 0.0;
        part += sv[c] * sv[c];
      }
    }
    return wave_sum_dpp(part);
  };
  auto Ax = [&]() {  // q = A_F v, v in pvS
#pragma unroll
    for (int c = 0; c < C; ++c) {
      q[c] = 0.0;
      if constexpr (GD > 0) {
        q[c] = c * kWave < N ? gather(pvS, hreg[c]) : 0.0;
      } else if (c * kWave < N) {
        double a = 0.0;
        const int k = lane + c * kWave, i = k < N ? k : 0;
#pragma unroll 4
        for (int u = 0; u < gamma; ++u) a += pvS[holder_at(i, u)];
        q[c] = k < N ? a : 0.0;
      }
    }
  };
  auto put = [&](const double (&v)[C]) {  // a vector over the finished workers into pvS
#pragma unroll
    for (int c = 0; c < C; ++c)
      if (col[c] < m) pvS[col[c]] = v[c];
  };
  double gam = AT();
#pragma unroll
  for (int c = 0; c < C; ++c) pv[c] = sv[c];
  const double stop = tol * tol * gam;
  int it = 0;
  while (it < max_iter && gam > stop && gam > 0.0) {
    put(pv);
    lds_done();
    Ax();
    double part = 0.0;
#pragma unroll
    for (int c = 0; c < C; ++c) part += q[c] * q[c];
    const double qq = wave_sum_dpp(part);
    if (!(qq > 0.0)) break;
    const double alpha = gam / qq;
#pragma unroll
    for (int c = 0; c < C; ++c) {
      rv[c] += alpha * pv[c];
      res[c] -= alpha * q[c];
      if (lane + c * kWave < N) resS[lane + c * kWave] = res[c];
    }
    lds_done();
    const double gnew = AT();
    const double beta = gnew / gam;
#pragma unroll
    for (int c = 0; c < C; ++c) pv[c] = sv[c] + beta * pv[c];
    gam = gnew;
    ++it;
  }
  // recompute the residual from r for the reported error
  lds_done();
  put(rv);
  lds_done();
  Ax();
  double part = 0.0;
#pragma unroll
  for (int c = 0; c < C; ++c) {
    const double e = lane + c * kWave < N ? q[c] - 1.0 : 0.0;
    part += e * e;
  }
  const double e2 = wave_sum_dpp(part);
  if (lane == 0) {
    err[p] = e2;
    if (iters) iters[p] = it;
  }
}

}  // namespace
}  // namespace gcx

extern "C" int gc_progress(const double *tau, const uint8_t *failed, int64_t R, int32_t m,
                           int32_t delta, const double *T, int32_t G, int32_t *psi,
                           hipStream_t stream) {
  using namespace gcx;
  if (R < 0 || m < 1 || m > GC_MAX_M || delta < 1 || delta > GC_MAX_DELTA || G < 1) return GC_EINVAL;
  // tau [R][m][delta], psi [R][G][m]
  if (!sizes_ok({R, m, delta}) || !sizes_ok({R, G, m})) return GC_EINVAL;
  if (R == 0) return GC_OK;
  if (!tau || !T || !psi) return GC_EINVAL;
  const int64_t blocks = ceil_div(R * m, kSimThreads);
  if (!grid_ok(blocks, kSimThreads)) return GC_EINVAL;
  const int dev = check_device();
  if (dev != GC_OK) return dev;
  (void)hipGetLastError();
#define GC_PROGRESS(D)                                                                            \
  hipLaunchKernelGGL(progress_kernel<D>, dim3(unsigned(blocks)), dim3(kSimThreads), 0, stream, tau, \
                     failed, R, m, delta, T, G, psi)
  if (delta <= 8) GC_PROGRESS(8);
  else if (delta <= 16) GC_PROGRESS(16);
  else if (delta <= 32) GC_PROGRESS(32);
  else GC_PROGRESS(0);
#undef GC_PROGRESS
  return launch_status();
}

extern "C" int gc_completion_times(const double *tau, const uint8_t *failed, int64_t R, int32_t N,
                                   int32_t m, int32_t delta, const int32_t *holder,
                                   const int32_t *hpos, int32_t gamma, int32_t ell,
                                   double *partial, double *original, hipStream_t stream) {
  using namespace gcx;
  if (R < 0 || N < 1 || m < 1 || m > GC_MAX_M || delta < 1 || delta > GC_MAX_DELTA || gamma < 1 ||
      gamma > GC_MAX_DELTA || ell < 1 || ell > GC_MAX_ELL)
    return GC_EINVAL;
  if (!sizes_ok({R, m, delta}) || !sizes_ok({N, gamma})) return GC_EINVAL;  // tau, tables
  if (R == 0) return GC_OK;
  if (!tau || !holder || !hpos || !partial || !original) return GC_EINVAL;
  if (!grid_ok(ceil_div(R, kSimWaves), kSimThreads)) return GC_EINVAL;
  const int dev = check_device();
  if (dev != GC_OK) return dev;
  (void)hipGetLastError();
  const size_t lds = sizeof(double) * size_t(m) * delta;
  const bool staged = lds <= kCompleteLds;
  const int64_t blocks = R < 0xffffffffLL / kSimThreads ? R : 0xffffffffLL / kSimThreads;  // the launch limits
  hipLaunchKernelGGL(completion_kernel, dim3(unsigned(blocks)), dim3(kSimThreads), staged ? lds : 0, stream, tau,
                     failed, R, N, m, delta, holder, hpos, gamma, ell, staged ? 1 : 0, partial, original);
  return launch_status();
}

extern "C" int gc_original_ls(const int32_t *psi, int64_t P, int32_t N, int32_t m,
                              const int32_t *order, int32_t delta, const int32_t *holder,
                              int32_t gamma, int32_t max_iter, double tol, double *err,
                              int32_t *iters, hipStream_t stream) {
  using namespace gcx;
  if (P < 0 || N < 1 || N > GC_MAX_M || m < 1 || m > GC_MAX_M || delta < 1 ||
      delta > GC_MAX_DELTA || gamma < 1 || gamma > GC_MAX_DELTA || max_iter < 0 || !(tol >= 0.0))
    return GC_EINVAL;
  if (!sizes_ok({P, m})) return GC_EINVAL;  // psi [P][m]
  if (P == 0) return GC_OK;
  if (!psi || !order || !holder || !err) return GC_EINVAL;
  if (!grid_ok(ceil_div(P, kLsWaves), kLsWaves * kWave)) return GC_EINVAL;
  const int dev = check_device();
  if (dev != GC_OK) return dev;
  (void)hipGetLastError();
  // values per lane: 4 up to 256 chunks and workers, 8 up to 512, else 16
  const int most = N > m ? N : m;
  const bool tl = ls_tables(N, m, delta, gamma) <= kLsTables;
  const size_t lds = (tl ? ls_tables(N, m, delta, gamma) : 0) + kLsWaves * ls_wave(N, m);
#define GC_LS(C, TL, GD)                                                                                 \
  do {                                                                                               \
    const auto kern = original_ls_kernel<C, TL, GD>;                                                     \
    if (lds > 64 * 1024 &&                                                                           \
        hipFuncSetAttribute(reinterpret_cast<const void *>(kern),                                    \
                            hipFuncAttributeMaxDynamicSharedMemorySize, int(lds)) != hipSuccess)     \
      return GC_ELAUNCH;                                                                             \
    hipLaunchKernelGGL(kern, dim3(unsigned(ceil_div(P, kLsWaves))), dim3(kLsWaves * kWave), lds,     \
                       stream, psi, P, N, m, order, delta, holder, gamma, max_iter, tol, err, iters); \
  } while (0)
  const int deg = gamma > delta ? gamma : delta;
  if (!tl) GC_LS(16, false, 0);
  else if (most <= 4 * kWave && deg <= 8) GC_LS(4, true, 8);
  else if (most <= 4 * kWave && deg <= 16) GC_LS(4, true, 16);
  else if (most <= 4 * kWave) GC_LS(4, true, 0);
  else if (most <= 8 * kWave && deg <= 8) GC_LS(8, true, 8);
  else if (most <= 8 * kWave) GC_LS(8, true, 0);
  else GC_LS(16, true, 0);
#undef GC_LS
  return launch_status();
}
