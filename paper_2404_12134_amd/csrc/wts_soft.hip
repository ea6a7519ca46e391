// wts_soft.hip -- the one-wave Soft-DTW forward sweep, and the sums and steps
// around the gradient.
#include "wts_soft.h"

namespace wts {

namespace {

// --------------------------------------------------------------- forward

template <typename TY, int D, int RHO, bool BAND>
__global__ __launch_bounds__(kWave) void soft_fwd_kernel(SoftArgs a) {
  constexpr int H = kWave * RHO;
  constexpr int kChunk = 64;
  __shared__ double ys[D][kRing + 16];   // -2 y' of the columns (see sq_cost)
  __shared__ double yq[kRing + 16];      // |y'|^2
  __shared__ double binr[kChunk];       // the strip above's bottom row (+inf for the top strip)
  __shared__ double bor[kRing];
  __shared__ int s_item;
  const int lane = threadIdx.x;
  const TY* __restrict__ Y = static_cast<const TY*>(a.y);
  const double INF = inf_d();
  const double k = a.kscale;
  const double sk = __builtin_sqrt(k);   // x and y enter as sqrt(k) (x - mu), sqrt(k) (y - mu)
  if (skipped(a.skip)) return;   // every workgroup: no strip waits for another

  for (;;) {
    if (lane == 0) s_item = atomicAdd(a.queue, 1);
    __syncthreads();
    const int item = __builtin_amdgcn_readfirstlane(s_item);   // uniform: scalar loads below
    __syncthreads();
    if (item >= a.n_items) break;
    const int2 it = a.items[item];
    const PairDesc pd = uniform(a.pairs[uni(it.x)]);
    const int s = uni(it.y);
    const int M = pd.M, N = pd.N;
    double mu[D];
#pragma unroll
    for (int c = 0; c < D; ++c) mu[c] = a.x[pd.x_off * D + c];
    const int i0 = s * H;
    const int ib = i0 + lane * RHO;
    const double band_b = BAND ? band_halfwidth(M, N, a.band) : 0.0;
    int band_jlo = 0, band_jhi = N - 1;
    if (BAND) band_strip_cols(M, N, a.band, i0, min(i0 + H, M) - 1, &band_jlo, &band_jhi);
    // columns inside the band on every row of the strip (from the last row's
    // left edge to the first row's right edge; empty when they cross): a
    // group whose columns all lie there needs no band test.  The rows past
    // M - 1 of the last strip count too: the band test keeps them at +inf
    // where the band's formula puts them outside, and the unbanded arithmetic
    // would turn three +inf inputs into NaN.
    int band_in_lo = 0, band_in_hi = -1;
    if (BAND) band_strip_cols(M, N, a.band, i0 + H - 1, i0, &band_in_lo, &band_in_hi);
    const bool has_prev = s > 0;
    const bool has_next = s + 1 < pd.S;
    const int Tend = pd.WT * 16;
    const double* row_in = a.rows + pd.aux_base + (int64_t)(s - 1) * N;
    double* row_out = a.rows + pd.aux_base + (int64_t)s * N;
    double* st = a.states + pd.state_base + (int64_t)s * pd.WT * (RHO + 1) * kWave;
    int* prog_in = a.progress + pd.flag_base + s - 1;
    int* prog_out = a.progress + pd.flag_base + s;

    double xr[RHO][D], xx[RHO];
#pragma unroll
    for (int r = 0; r < RHO; ++r) {
#pragma unroll
      for (int c = 0; c < D; ++c)
        xr[r][c] = (ib + r < M) ? (a.x[(pd.x_off + ib + r) * D + c] - mu[c]) * sk : 0.0;
      xx[r] = sq_norm<D>(xr[r]);
    }
    double left[RHO];
#pragma unroll
    for (int r = 0; r < RHO; ++r) left[r] = INF;
    double upprev = (s == 0 && lane == 0) ? 0.0 : INF;
    double bot = INF;
    bool gave_up = false;       // wave-uniform
    int seen_prev = 0;          // last progress read from the strip above (uniform)
    bool have_next = false;     // pr_next holds the next chunk's upper input (uniform)
    double pr_next = INF;
    const __amdgpu_buffer_rsrc_t ro = rsrc(row_out, has_next ? N * 8 : 0);

    {
      double yc[D];
#pragma unroll
      for (int c = 0; c < D; ++c)
        yc[c] = lane < N ? (static_cast<double>(Y[(pd.y_off + lane) * D + c]) - mu[c]) * sk : 0.0;
      ring_col<D>(ys, yq, lane, yc);
    }
    __syncthreads();

    for (int t0 = 0; t0 < Tend; t0 += kChunk) {
      const int tcnt = min(kChunk, Tend - t0);
      const bool more = t0 + kChunk < Tend;
      // next chunk's Y columns: unconditional loads from a clamped column,
      // kept in the storage type until they are written to LDS after this
      // chunk (a conditional load would be waited for on the spot)
      TY yraw[D];
      {
        const int j = min(t0 + kChunk + lane, N - 1);
#pragma unroll
        for (int c = 0; c < D; ++c) yraw[c] = Y[(pd.y_off + j) * D + c];
      }
      if (has_prev) {
        // the strip above's bottom row for this chunk: prefetched during the
        // previous chunk when its counter already covered it, else read now
        // (one read of the counter usually covers many chunks)
        double pr = pr_next;
        if (!have_next) {
          const int need = min(N, t0 + kChunk);
          if (need > seen_prev && !gave_up) {
            int got = 0, quit = 0;
            if (lane == 0) {
              int polls = 0;
              got = ld_dev(prog_in);
              while (got < need) {
                poll_backoff(polls, a.relaxed_wait);
                if (++polls > kSpinLimit) {
                  atomicOr(a.status, kStatusSpinTimeout);
                  quit = 1;
                  break;
                }
                got = ld_dev(prog_in);
              }
            }
            seen_prev = __builtin_amdgcn_readfirstlane(got);
            gave_up = __builtin_amdgcn_readfirstlane(quit) != 0;
          }
          __atomic_signal_fence(__ATOMIC_SEQ_CST);
          const int j = t0 + lane;
          pr = j < N ? ld_dev(row_in + j) : INF;
        }
        binr[lane] = pr;
        __atomic_signal_fence(__ATOMIC_SEQ_CST);
        const int jn = t0 + kChunk + lane;
        have_next = more && seen_prev >= min(N, t0 + 2 * kChunk);
        if (have_next) pr_next = jn < N ? ld_dev(row_in + jn) : INF;
      } else {
        binr[lane] = INF;
      }
      __syncthreads();

      // FULL: every lane is inside the grid (no masking); INSIDE: every cell
      // is inside the band as well (the unbanded arithmetic, which gives an
      // in-band cell the same bits as the band test's path)
      auto group16 = [&](auto full_tag, auto inside_tag, int tb) {
        constexpr bool FULL = decltype(full_tag)::value;
        constexpr bool TEST = BAND && !decltype(inside_tag)::value;
        const int tg = t0 + tb;
        {   // checkpoint: the sweep state at the start of these 16 steps
          double* p = st + (int64_t)(tg >> 4) * (RHO + 1) * kWave + lane;
#pragma unroll
          for (int r = 0; r < RHO; ++r) p[r * kWave] = left[r];
          p[RHO * kWave] = upprev;
        }
        const int yb = (tg - lane) & (kRing - 1);   // ring slot of step 0's column
#pragma unroll
        for (int u = 0; u < 16; ++u) {
          const int t = tg + u;
          const int j = t - lane;
          const double bval = binr[tb + u];
          const double upin = shr1_f64(bot, bval);
          const double dg0 = upprev;
          upprev = upin;
          if (FULL || (j >= 0 && j < N)) {
            double y[D];
#pragma unroll
            for (int c = 0; c < D; ++c) y[c] = ys[c][yb + u];
            const double yy = yq[yb + u];
            double dg = dg0, up = upin;
            // band coordinate of row ib at column j (exact in float64)
            const double bd0 = (double)ib * (double)(N - 1) - (double)j * (double)(M - 1);
#pragma unroll
            for (int r = 0; r < RHO; ++r) {
              const double lf = left[r];
              double rv;
              if constexpr (TEST) {
                const bool inb = __builtin_fabs(bd0 + (double)r * (double)(N - 1)) <= band_b;
                const SoftMin sm = softmin3_band(dg, up, lf, inb);
                rv = inb ? sq_cost<D>(xr[r], xx[r], y, yy) + sm.v : INF;
              } else {
                const SoftMin sm = softmin3(dg, up, lf);
                rv = sq_cost<D>(xr[r], xx[r], y, yy) + sm.v;
              }
              dg = lf;
              up = rv;
              left[r] = rv;
            }
            bot = left[RHO - 1];
            if (has_next && lane == kWave - 1) bor[j & (kRing - 1)] = bot;
          }
        }
      };
      // a group whose columns (tg - 63 .. tg + 15 over the lanes) all lie
      // outside the strip's band keeps only its bookkeeping: checkpoint,
      // +inf state and bottom row, and lane 0's diagonal input of the next step
      auto skip16 = [&](int tb) {
        const int tg = t0 + tb;
        double* p = st + (int64_t)(tg >> 4) * (RHO + 1) * kWave + lane;
#pragma unroll
        for (int r = 0; r < RHO; ++r) p[r * kWave] = left[r];
        p[RHO * kWave] = upprev;
        // lanes with cells in the grid during the group end it at +inf; a lane
        // already past column N-1 keeps its values (as the sweep would)
        if (tg + 15 - lane >= 0 && tg - lane <= N - 1) {
#pragma unroll
          for (int r = 0; r < RHO; ++r) left[r] = INF;
          bot = INF;
        }
        upprev = (lane == 0 && has_prev) ? binr[tb + 15] : INF;
        if (has_next && lane < 16) {
          const int j = tg - (kWave - 1) + lane;
          if (j >= 0 && j < N) bor[j & (kRing - 1)] = INF;
        }
      };
      for (int tb = 0; tb < tcnt; tb += 16) {
        const int tg = t0 + tb;
        if (BAND && (tg + 15 < band_jlo || tg - (kWave - 1) > band_jhi)) {
          skip16(tb);
        } else if (tg >= kWave - 1 && tg + 16 <= N) {
          if (BAND && tg - (kWave - 1) >= band_in_lo && tg + 15 <= band_in_hi)
            group16(std::true_type{}, std::true_type{}, tb);
          else
            group16(std::true_type{}, std::false_type{}, tb);
        } else {
          group16(std::false_type{}, std::false_type{}, tb);
        }
      }
      __syncthreads();
      if (has_next) {
        // this chunk's columns of the bottom row (one store, dropped outside
        // the row), then the previous chunk's columns are announced: waiting
        // until at most this store is outstanding completes every older one
        const int jend = t0 + tcnt - (kWave - 1);
        const int j = t0 - (kWave - 1) + lane;
        const bool w = j >= 0 && j < N && j < jend;
        st_dev(ro, w ? j * 8 : kDrop, bor[j & (kRing - 1)]);
        mem_wait_all_but_1();
        if (lane == 0) st_dev(prog_out, min(N, max(0, t0 - (kWave - 1))));
      }
      if (more) {
        const int j = t0 + kChunk + lane;
        double yc[D];
#pragma unroll
        for (int c = 0; c < D; ++c) yc[c] = j < N ? (static_cast<double>(yraw[c]) - mu[c]) * sk : 0.0;
        ring_col<D>(ys, yq, j & (kRing - 1), yc);
      }
      __syncthreads();
    }
    if (has_next) {   // the last chunk's columns
      mem_drain();
      if (lane == 0) st_dev(prog_out, N);
    }
    if (ib <= M - 1 && M - 1 < ib + RHO) {
      const int rl = M - 1 - ib;
      double v = left[0];
#pragma unroll
      for (int r = 1; r < RHO; ++r)
        if (r == rl) v = left[r];
      a.value[pd.out] = v / k;
    }
    __syncthreads();
  }
}

// G_l = sum_k w_k * grad_k(l), h_l = sum_k w_k * mass_k(l), ascending k,
// starting from 0 or (accumulate) from the values already in grad / mass.
// Calls over consecutive cycle groups with accumulate = 1 after the first
// therefore perform the very additions of one call over all cycles.
__global__ void soft_reduce_kernel(const double* __restrict__ gsum, const double* __restrict__ hsum,
                                   const double* __restrict__ w, int n, int64_t L, int d,
                                   double* __restrict__ grad, double* __restrict__ mass,
                                   int accumulate) {
  const int64_t idx = blockIdx.x * (int64_t)blockDim.x + threadIdx.x;
  if (idx >= L * d) return;
  const int64_t l = idx / d;
  const int c = (int)(idx - l * d);
  double g = accumulate ? grad[idx] : 0.0;
  for (int p = 0; p < n; ++p) g = g + (w ? w[p] : 1.0) * gsum[((int64_t)p * L + l) * d + c];
  grad[idx] = g;
  if (c == 0 && mass) {
    double h = accumulate ? mass[l] : 0.0;
    for (int p = 0; p < n; ++p) h = h + (w ? w[p] : 1.0) * hsum[(int64_t)p * L + l];
    mass[l] = h;
  }
}

// Rows of a packed [sum N][d] gradient scaled by their cycle's weight:
// out[row] = w[k] * g[row] for the cycle k holding the row (offsets off[n+1]).
__global__ void soft_rows_scale_kernel(const double* __restrict__ g, const int64_t* __restrict__ off,
                                       int n, int d, const double* __restrict__ w,
                                       double* __restrict__ out) {
  const int64_t idx = blockIdx.x * (int64_t)blockDim.x + threadIdx.x;
  const int64_t rows = off[n];
  if (idx >= rows * d) return;
  const int64_t row = idx / d;
  int lo = 0, hi = n - 1;   // the cycle k with off[k] <= row < off[k + 1]
  while (lo < hi) {
    const int mid = (lo + hi + 1) >> 1;
    if (off[mid] <= row) lo = mid;
    else hi = mid - 1;
  }
  out[idx] = w ? w[lo] * g[idx] : g[idx];
}

// One preconditioned gradient step on the barycenter:
//   b_l <- b_l - eta * G_l / (2 h_l)
// With eta = 1 this is the soft-DBA update b_l = sum_j e y_j / sum_j e.
__global__ void precond_step_kernel(double* __restrict__ bary, const double* __restrict__ grad,
                                    const double* __restrict__ mass, int64_t L, int d,
                                    double eta) {
  const int64_t idx = blockIdx.x * (int64_t)blockDim.x + threadIdx.x;
  if (idx >= L * d) return;
  const int64_t l = idx / d;
  bary[idx] = bary[idx] - eta * grad[idx] / (2.0 * mass[l]);
}

}  // namespace

hipError_t launch_precond_step(double* bary, const double* grad, const double* mass, int64_t L,
                               int d, double eta, hipStream_t st) {
  const int64_t tot = L * d;
  hipLaunchKernelGGL(precond_step_kernel, dim3((unsigned)((tot + 255) / 256)), dim3(256), 0, st,
                     bary, grad, mass, L, d, eta);
  return hipGetLastError();
}

template <typename TY, int D>
static hipError_t launch_soft_fwd_t(const SoftArgs& a, int grid, hipStream_t st) {
  if (a.band > 0.0)
    hipLaunchKernelGGL((soft_fwd_kernel<TY, D, kSoftRho, true>), dim3(grid), dim3(kWave), 0, st, a);
  else
    hipLaunchKernelGGL((soft_fwd_kernel<TY, D, kSoftRho, false>), dim3(grid), dim3(kWave), 0, st, a);
  return hipGetLastError();
}

hipError_t launch_soft_fwd(int d, int ydtype, const SoftArgs& a, int grid, hipStream_t st) {
#define CALLS(D) (ydtype == 0 ? launch_soft_fwd_t<float, D>(a, grid, st) \
                              : launch_soft_fwd_t<double, D>(a, grid, st))
  WTS_SOFT_D_SWITCH(d, CALLS)
#undef CALLS
}

hipError_t launch_soft_rows_scale(const double* g, const int64_t* off, int n, int64_t rows, int d,
                                  const double* w, double* out, hipStream_t st) {
  const int64_t tot = rows * d;
  if (tot == 0) return hipSuccess;
  hipLaunchKernelGGL(soft_rows_scale_kernel, dim3((unsigned)((tot + 255) / 256)), dim3(256), 0, st,
                     g, off, n, d, w, out);
  return hipGetLastError();
}

hipError_t launch_soft_reduce(const double* gsum, const double* hsum, const double* w, int n,
                              int64_t L, int d, double* grad, double* mass, int accumulate,
                              hipStream_t st) {
  const int64_t tot = L * d;
  hipLaunchKernelGGL(soft_reduce_kernel, dim3((unsigned)((tot + 255) / 256)), dim3(256), 0, st,
                     gsum, hsum, w, n, L, d, grad, mass, accumulate);
  return hipGetLastError();
}

}  // namespace wts
