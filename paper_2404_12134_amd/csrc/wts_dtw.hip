// wts_dtw.hip -- path recovery, DBA update, scores, medoid and barycenter
// initialisation for gfx950, and the float64 instances of the DTW sweep
// (wts_sweep.h).
#include "wts_sweep.h"
#include "wts_walk.h"

namespace wts {

namespace {

// Strip-level path recovery after a PATHT sweep.  That sweep tagged every
// cell with the top-row cell through which its optimal path enters the strip (code 2j for
// "from (i0-1, j)", 2j+1 for "from (i0-1, j-1)"), and kept that tag for the
// bottom row of every strip.  Walking the tags from (M-1, N-1) gives, per
// strip, where the path crosses its bottom row and its top row.
__global__ void chain_kernel(const PairDesc* __restrict__ pairs, int n_pairs,
                             const int* __restrict__ bnd_aux, const int* __restrict__ out_aux,
                             int2* __restrict__ seg, int* __restrict__ status,
                             const int* __restrict__ skip) {
  const int p = blockIdx.x * blockDim.x + threadIdx.x;
  if (p >= n_pairs || skipped(skip)) return;
  const PairDesc pd = pairs[p];
  int e = out_aux[pd.out];
  int jx = pd.N - 1;
  for (int s = pd.S - 1; s >= 0; --s) {
    const int jtop = e >> 1;
    if (jtop < 0 || jtop > jx) {   // inconsistent tags: mark every strip left empty
      atomicOr(status, kStatusBadPath);
      for (int q = s; q >= 0; --q) seg[pd.item_base + q] = make_int2(-1, -1);
      return;
    }
    seg[pd.item_base + s] = make_int2(jx, jtop);
    if (s == 0) break;
    const int jp = jtop - (e & 1);
    if (jp < 0) {
      atomicOr(status, kStatusBadPath);
      for (int q = s - 1; q >= 0; --q) seg[pd.item_base + q] = make_int2(-1, -1);
      return;
    }
    e = bnd_aux[pd.row_base + (int64_t)(s - 1) * row_stride(pd.N) + jp + 63];
    jx = jp;
  }
}

// Walks the optimal path through one strip (one wave), from its bottom-row
// crossing to its top-row cell (walk_strip), and records the run of columns
// [lo, hi] that the path occupies on each row.  A walk that does not end
// where the chain says marks the status word; its strip then contributes
// empty runs.
template <int RHO>
__global__ __launch_bounds__(kWave) void walk_kernel(WalkArgs a) {
  constexpr int H = kWave * RHO;
  const int lane = threadIdx.x;
  const int item = blockIdx.x;
  if (skipped(a.skip)) return;
  const int2 it = a.items[item];
  const PairDesc pd = uniform(a.pairs[uni(it.x)]);
  const int s = uni(it.y);
  const int i0 = s * H;
  const int iend = min(pd.M, i0 + H) - 1;
  const int jx = uni(a.seg[item].x), jtop = uni(a.seg[item].y);
  const uint32_t* codes = a.codes + pd.code_base + (int64_t)s * pd.WT * RHO * kWave;
  int2* runs = a.runs + (int64_t)pd.out * a.L + i0;
  bool ok = jx >= 0 && jx < pd.N && jtop >= 0 && jtop <= jx;
  if (ok) {
    Walk st{iend - i0, jx, jx, -1};
    const WalkEnd end = walk_strip<RHO>(st, 0, runs, [&](int b, int k, int r, uint32_t& nl, uint32_t& dd) {
      const uint32_t* p = codes + ((int64_t)b * 2 * RHO + r) * kWave + k;
      dd = p[0];
      nl = dd | p[RHO * kWave];
    });
    ok = end == kWalkDone && st.jtop == jtop;
  }
  if (!ok) {
    if (lane == 0) atomicOr(a.status, kStatusBadPath);
    for (int q = lane; q <= iend - i0; q += kWave) runs[q] = make_int2(0, -1);
  }
}

// The DBA update from the row runs: per cycle and row the sum of the cycle's
// samples over the run [lo, hi] in descending column order, folded over the
// cycles in ascending order with their weights, and the mean.  A workgroup
// takes ROWS rows and 256 / ROWS cycles at a time: each thread sums one
// (cycle, row) run, then one thread per (row, channel) folds the sums from
// LDS in order, so no per-cycle sums go through memory.  Bound by the launch and
// one trip to memory on small batches (4 us of the 62 of a DBA iteration on 8
// cycles of 230), else by the trips to memory of a workgroup's cycles.
// ROWS: 4, and 1 up to 512 rows (two workgroups a compute unit), where the
// cycles of a row are the more to share.  DBA iteration, us, at 16 / 4 / 1 rows: 1000 cycles
// of 1000 (L = 16) 783 / 381 / 272, 512 of 20k (L = 500) 4723 / 4426 / 4371, 300 of
// 1000 (L = 1000) 465 / 447 / 457, 512 of 8k (L = 8000, d = 6) 21.19 / 21.12 / 21.42 ms.
constexpr int kFoldThreads = 256;
constexpr int64_t kFoldFewRows = 512;
template <typename TY, int D, int ROWS>
__global__ __launch_bounds__(kFoldThreads)
void run_fold_kernel(const int2* __restrict__ runs, const int64_t* __restrict__ off, const void* y,
                     const double* __restrict__ w, int n, int64_t L, double* __restrict__ bout,
                     int64_t* __restrict__ counts, const int* skip) {
  constexpr int kCycles = kFoldThreads / ROWS;
  __shared__ double ps[kCycles][D][ROWS];
  __shared__ int pc[kCycles][ROWS];
  if (skipped(skip)) return;
  const TY* __restrict__ Y = static_cast<const TY*>(y);
  const int q = threadIdx.x / ROWS, row = threadIdx.x % ROWS;
  const int64_t l = blockIdx.x * (int64_t)ROWS + row;
  const int fc = threadIdx.x / ROWS;   // the channel this thread folds (fc < D)
  double S = 0.0, C = 0.0;
  int64_t K = 0;
  for (int p0 = 0; p0 < n; p0 += kCycles) {
    const int p = p0 + q;
    if (p < n && l < L) {
      const int2 rn = runs[(int64_t)p * L + l];
      const int64_t base = off[p];
      double acc[D];
#pragma unroll
      for (int c = 0; c < D; ++c) acc[c] = 0.0;
      int jj = rn.y;
      for (; jj >= rn.x + 7; jj -= 8) {   // long runs: eight samples in flight
        TY v[8][D];
#pragma unroll
        for (int u = 0; u < 8; ++u)
#pragma unroll
          for (int c = 0; c < D; ++c) v[u][c] = Y[(base + jj - u) * D + c];
#pragma unroll
        for (int u = 0; u < 8; ++u)
#pragma unroll
          for (int c = 0; c < D; ++c) acc[c] = acc[c] + static_cast<double>(v[u][c]);
      }
      for (; jj >= rn.x; --jj) {
#pragma unroll
        for (int c = 0; c < D; ++c) acc[c] = acc[c] + static_cast<double>(Y[(base + jj) * D + c]);
      }
#pragma unroll
      for (int c = 0; c < D; ++c) ps[q][c][row] = acc[c];
      pc[q][row] = rn.y - rn.x + 1;
    }
    __syncthreads();
    if (fc < D && l < L) {
      const int m = min(kCycles, n - p0);
#pragma unroll 4
      for (int e = 0; e < m; ++e) {
        const double wp = w ? w[p0 + e] : 1.0;
        const int k = pc[e][row];
        S = S + wp * ps[e][fc][row];
        C = C + wp * (double)k;
        K += k;
      }
    }
    __syncthreads();
  }
  if (fc < D && l < L) {
    bout[l * D + fc] = S / C;
    if (fc == 0) counts[l] = K;
  }
}

}  // namespace

// --------------------------------------------------------------- small kernels

__global__ void zero_i32_kernel(int* p, int64_t n) {
  for (int64_t k = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; k < n;
       k += (int64_t)gridDim.x * blockDim.x)
    p[k] = 0;
}

// Sentinel fill of the strip boundary rows before a sweep, and its item
// counter.
__global__ void fill_sent_kernel(unsigned long long* r, int64_t nr, int* x, int64_t nx, int* queue) {
  if (blockIdx.x == 0 && threadIdx.x == 0) *queue = 0;
  const int64_t stride = (int64_t)gridDim.x * blockDim.x;
  for (int64_t k = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; k < nr; k += stride)
    r[k] = kSentR;
  for (int64_t k = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; k < nx; k += stride)
    x[k] = kSentX;
}

// The path list of every pair from its row runs, and its length: a scan of
// the run lengths over the rows gives each row's place.  One workgroup per
// pair.
constexpr int kEmitThreads = 256;
__global__ __launch_bounds__(kEmitThreads)
void emit_kernel(const int2* __restrict__ runs, const int64_t* __restrict__ path_base, int64_t L,
                 int32_t* __restrict__ paths, int64_t* __restrict__ path_len, const int* skip) {
  __shared__ int part[kEmitThreads / kWave];
  if (skipped(skip)) return;
  const int pair = blockIdx.x, lane = threadIdx.x % kWave, wv = threadIdx.x / kWave;
  const int2* rn = runs + (int64_t)pair * L;
  int32_t* out = paths + 2 * path_base[pair];
  int64_t done = 0;
  for (int64_t i0 = 0; i0 < L; i0 += kEmitThreads) {
    const int64_t i = i0 + threadIdx.x;
    const int2 r = i < L ? rn[i] : make_int2(0, -1);
    const int len = r.y - r.x + 1;
    int inc = len;   // inclusive scan over the wave
#pragma unroll
    for (int d = 1; d < kWave; d <<= 1) {
      const int v = __shfl_up(inc, d);
      if (lane >= d) inc += v;
    }
    if (lane == kWave - 1) part[wv] = inc;
    __syncthreads();
    int before = 0, all = 0;
#pragma unroll
    for (int q = 0; q < kEmitThreads / kWave; ++q) {
      if (q < wv) before += part[q];
      all += part[q];
    }
    int64_t at = done + before + inc - len;
    for (int j = r.x; j <= r.y; ++j, ++at) {
      out[2 * at] = (int)i;
      out[2 * at + 1] = j;
    }
    done += all;
    __syncthreads();
  }
  if (threadIdx.x == 0) path_len[pair] = done;
}

__global__ void score_kernel(const double* __restrict__ dist, const int* __restrict__ len, int n,
                             double* __restrict__ score, int64_t* __restrict__ path_len) {
  const int p = blockIdx.x * blockDim.x + threadIdx.x;
  if (p >= n) return;
  const double dv = dist[p];
  const int lv = len[p];
  if (score) score[p] = dv / (double)lv;
  if (path_len) path_len[p] = lv;
}

// Medoid: D[a][b] = D[b][a] = DTW of pair (a, b); totals in ascending order.
__global__ void medoid_fill_kernel(const double* __restrict__ pair_dist,
                                   const int2* __restrict__ pair_ab, int n_pairs, int n,
                                   double* __restrict__ Dm) {
  const int64_t k = blockIdx.x * (int64_t)blockDim.x + threadIdx.x;
  if (k < n_pairs) {
    const int2 ab = pair_ab[k];
    Dm[(int64_t)ab.x * n + ab.y] = pair_dist[k];
    Dm[(int64_t)ab.y * n + ab.x] = pair_dist[k];
  }
  if (k < n) Dm[k * n + k] = 0.0;
}

__global__ void medoid_total_kernel(const double* __restrict__ Dm, int n,
                                    double* __restrict__ totals) {
  const int k = blockIdx.x * blockDim.x + threadIdx.x;
  if (k >= n) return;
  double s = 0.0;
  for (int i = 0; i < n; ++i) s = s + Dm[(int64_t)k * n + i];
  totals[k] = s;
}

__global__ void medoid_argmin_kernel(const double* __restrict__ totals, int n,
                                     int32_t* __restrict__ medoid) {
  if (blockIdx.x != 0 || threadIdx.x != 0) return;
  int best = 0;
  double bv = inf_d();
  for (int k = 0; k < n; ++k)
    if (totals[k] < bv) { bv = totals[k]; best = k; }
  *medoid = best;
}

// Resampling at t_l = l (N-1)/(L-1); source = one cycle, or (euclid = true)
// the per-index mean of all cycles padded with their last sample.
template <typename TY>
__global__ void init_kernel(const TY* __restrict__ Y, const int64_t* __restrict__ off, int n,
                            int d, int src, int64_t Nsrc, int64_t L, int euclid,
                            double* __restrict__ out) {
  const int64_t idx = blockIdx.x * (int64_t)blockDim.x + threadIdx.x;
  if (idx >= L * d) return;
  const int64_t l = idx / d;
  const int c = (int)(idx - l * d);
  auto sample = [&](int64_t tt) -> double {
    if (!euclid) return static_cast<double>(Y[(off[src] + tt) * d + c]);
    double s = 0.0;
    for (int p = 0; p < n; ++p) {
      const int64_t Np = off[p + 1] - off[p];
      const int64_t q = tt < Np ? tt : Np - 1;
      s = s + static_cast<double>(Y[(off[p] + q) * d + c]);
    }
    return s / (double)n;
  };
  const double pos = L == 1 ? 0.0 : ((double)l * (double)(Nsrc - 1)) / (double)(L - 1);
  const int64_t a0 = (int64_t)__builtin_floor(pos);
  double v;
  if (a0 >= Nsrc - 1) {
    v = sample(Nsrc - 1);
  } else {
    const double f = pos - (double)a0;
    const double ya = sample(a0), yb = sample(a0 + 1);
    v = ya + f * (yb - ya);
  }
  out[idx] = v;
}

// ------------------------------------------------------------------ dispatch

hipError_t launch_fwd(int d, int rho, int mode, bool euc, bool x_is_cycle, int ydtype, bool fp32,
                      const FwdArgs& a, int grid, hipStream_t st) {
  if (fp32) return launch_fwd32(d, rho, mode, euc, x_is_cycle, ydtype, a, grid, st);
  return launch_fwd_impl<double>(d, rho, mode, euc, x_is_cycle, ydtype, a, grid, st);
}

hipError_t launch_walk(int rho, const WalkArgs& a, int n_items, hipStream_t st) {
  if (rho == 4) hipLaunchKernelGGL(walk_kernel<4>, dim3(n_items), dim3(kWave), 0, st, a);
  else if (rho == 2) hipLaunchKernelGGL(walk_kernel<2>, dim3(n_items), dim3(kWave), 0, st, a);
  else if (rho == 5) hipLaunchKernelGGL(walk_kernel<5>, dim3(n_items), dim3(kWave), 0, st, a);
  else return hipErrorInvalidValue;
  return hipGetLastError();
}

hipError_t launch_chain(const PairDesc* pairs, int n_pairs, const int* bnd_aux,
                        const int* out_aux, int2* seg, int* status, const int* skip,
                        hipStream_t st) {
  hipLaunchKernelGGL(chain_kernel, dim3((n_pairs + 63) / 64), dim3(64), 0, st, pairs, n_pairs,
                     bnd_aux, out_aux, seg, status, skip);
  return hipGetLastError();
}

template <typename TY, int D>
static hipError_t launch_run_fold_t(const int2* runs, const int64_t* off, const void* y,
                                    const double* w, int n, int64_t L, double* bout,
                                    int64_t* counts, const int* skip, hipStream_t st) {
  auto go = [&](auto rows) {
    constexpr int R = decltype(rows)::value;
    hipLaunchKernelGGL((run_fold_kernel<TY, D, R>), dim3((unsigned)((L + R - 1) / R)),
                       dim3(kFoldThreads), 0, st, runs, off, y, w, n, L, bout, counts, skip);
  };
  if (L <= kFoldFewRows) go(std::integral_constant<int, 1>{});
  else go(std::integral_constant<int, 4>{});
  return hipGetLastError();
}

hipError_t launch_run_fold(int d, int ydtype, const int2* runs, const int64_t* off, const void* y,
                           const double* w, int n, int64_t L, double* bout, int64_t* counts,
                           const int* skip, hipStream_t st) {
#define CALLS(D, R) (ydtype == 0 ? launch_run_fold_t<float, D>(runs, off, y, w, n, L, bout, counts, skip, st) \
                                 : launch_run_fold_t<double, D>(runs, off, y, w, n, L, bout, counts, skip, st))
  WTS_D_SWITCH(d, 0, CALLS)
#undef CALLS
  return hipErrorInvalidValue;
}

hipError_t launch_emit(const int2* runs, const int64_t* path_base, int n, int64_t L,
                       int32_t* paths, int64_t* path_len, const int* skip, hipStream_t st) {
  hipLaunchKernelGGL(emit_kernel, dim3((unsigned)n), dim3(kEmitThreads), 0, st, runs, path_base, L,
                     paths, path_len, skip);
  return hipGetLastError();
}

hipError_t launch_zero(int* p, int64_t n, hipStream_t st) {
  if (n <= 0) return hipSuccess;
  const int64_t blocks = (n + 255) / 256;
  hipLaunchKernelGGL(zero_i32_kernel, dim3((unsigned)(blocks < 4096 ? blocks : 4096)), dim3(256),
                     0, st, p, n);
  return hipGetLastError();
}

hipError_t launch_fill_sentinels(double* r, int64_t nr, int* x, int64_t nx, int* queue,
                                 hipStream_t st) {
  const int64_t n = nr > nx ? nr : nx;
  const int64_t blocks = n > 0 ? (n + 255) / 256 : 1;
  hipLaunchKernelGGL(fill_sent_kernel, dim3((unsigned)(blocks < 8192 ? blocks : 8192)), dim3(256), 0,
                     st, reinterpret_cast<unsigned long long*>(r), nr, x, nx, queue);
  return hipGetLastError();
}

hipError_t launch_score(const double* dist, const int* len, int n, double* score,
                        int64_t* path_len, hipStream_t st) {
  hipLaunchKernelGGL(score_kernel, dim3((n + 255) / 256), dim3(256), 0, st, dist, len, n, score,
                     path_len);
  return hipGetLastError();
}

// Sub-DTW columns (a*, b*) as int64.
__global__ void sub_out_kernel(const int* __restrict__ start, const int* __restrict__ end, int n,
                               int64_t* __restrict__ a_star, int64_t* __restrict__ b_star) {
  const int p = blockIdx.x * blockDim.x + threadIdx.x;
  if (p >= n) return;
  a_star[p] = start[p];
  b_star[p] = end[p];
}

hipError_t launch_sub_out(const int* start, const int* end, int n, int64_t* a_star,
                          int64_t* b_star, hipStream_t st) {
  hipLaunchKernelGGL(sub_out_kernel, dim3((n + 255) / 256), dim3(256), 0, st, start, end, n,
                     a_star, b_star);
  return hipGetLastError();
}

hipError_t launch_medoid(const double* pair_dist, const int2* pair_ab, int n_pairs, int n,
                         double* Dm, double* totals, int32_t* medoid, hipStream_t st) {
  const int64_t m = n_pairs > n ? n_pairs : n;
  hipLaunchKernelGGL(medoid_fill_kernel, dim3((unsigned)((m + 255) / 256)), dim3(256), 0, st,
                     pair_dist, pair_ab, n_pairs, n, Dm);
  hipLaunchKernelGGL(medoid_total_kernel, dim3((n + 255) / 256), dim3(256), 0, st, Dm, n, totals);
  hipLaunchKernelGGL(medoid_argmin_kernel, dim3(1), dim3(64), 0, st, totals, n, medoid);
  return hipGetLastError();
}

hipError_t launch_init(int ydtype, const void* Y, const int64_t* off, int n, int d, int src,
                       int64_t Nsrc, int64_t L, int euclid, double* out, hipStream_t st) {
  const int64_t tot = L * d;
  const dim3 g((unsigned)((tot + 255) / 256));
  if (ydtype == 0)
    hipLaunchKernelGGL(init_kernel<float>, g, dim3(256), 0, st, static_cast<const float*>(Y), off,
                       n, d, src, Nsrc, L, euclid, out);
  else
    hipLaunchKernelGGL(init_kernel<double>, g, dim3(256), 0, st, static_cast<const double*>(Y),
                       off, n, d, src, Nsrc, L, euclid, out);
  return hipGetLastError();
}

}  // namespace wts
