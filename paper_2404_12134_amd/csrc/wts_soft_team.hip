// wts_soft_team.hip -- the Soft-DTW forward sweep for batches of few strips.
//
// The one-wave sweep (wts_soft.hip) takes 160 to 180 ns a step when a strip
// has a SIMD to itself: the soft minima of a lane's two rows are a chain of 22
// dependent operations, and the costs, checkpoints and exchange issue around
// it.  Here a workgroup of four waves sweeps a strip: wave 0 the recurrence and
// its checkpoints, wave 1 the inputs, waves 2 and 3 the costs (half of a
// group's 16 steps each, through LDS), one barrier a group, as in the DTW team
// sweep.  A strip's bottom row is filled with a sentinel before the launch and
// the strip below polls the values themselves, 16 at a time, where the
// one-wave sweep announces whole chunks of 64 columns one chunk late: the
// strips of a pair follow each other by about 110 steps instead of 220.
// A step takes 121 to 138 ns, bound by that chain: 5 cycles of 18k in the 0.6
// band 9.4 -> 4.7 ms, 16 of 2k (d = 3) 0.98 -> 0.44 ms.
// The operations of a cell and what is left in the checkpoint buffer are
// those of the one-wave sweep.
#include "wts_soft.h"

namespace wts {

namespace {

constexpr int kTeamGroup = 16;
constexpr int kTeamWaves = 4;

template <typename TY, int D, int RHO, bool BAND>
__global__ __launch_bounds__(kWave * kTeamWaves) void soft_fwd_team_kernel(SoftArgs a) {
  static_assert(RHO == 2, "costs travel in pairs of rows");
  constexpr int H = kWave * RHO;
  constexpr int G = kTeamGroup;
  __shared__ double ys[D][kRing + G];      // -2 y' of the columns (see sq_cost), mirrored
  __shared__ double yq[kRing + G];         // |y'|^2
  __shared__ double2 dl[2][G][kWave];      // costs of a group's cells, rows 0 and 1
  __shared__ double binr[2][G];            // the strip above's bottom row (+inf for the top strip)
  __shared__ double stg[2][G + kWave + G]; // lane 63's bottom row; the other lanes' writes follow
  __shared__ int s_item;
  const int wv = uni((int)threadIdx.x / kWave);
  const int lane = threadIdx.x % kWave;
  const TY* __restrict__ Y = static_cast<const TY*>(a.y);
  const double INF = inf_d();
  const double k = a.kscale;
  const double sk = __builtin_sqrt(k);   // x and y enter as sqrt(k) (x - mu), sqrt(k) (y - mu)
  if (skipped(a.skip)) return;   // every workgroup: no strip waits for another

  for (;;) {
    if (threadIdx.x == 0) s_item = atomicAdd(a.queue, 1);
    __syncthreads();
    const int item = uni(s_item);
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
    const bool has_prev = s > 0;
    const bool has_next = s + 1 < pd.S;
    const int NG = pd.WT;
    // columns of the strip's band, and those inside the band on every row of
    // it (the rows past M - 1 of the last strip count too: see soft_fwd_kernel)
    int band_jlo = 0, band_jhi = N - 1, band_in_lo = 0, band_in_hi = -1;
    if (BAND) {
      band_strip_cols(M, N, a.band, i0, min(i0 + H, M) - 1, &band_jlo, &band_jhi);
      band_strip_cols(M, N, a.band, i0 + H - 1, i0, &band_in_lo, &band_in_hi);
    }
    // a group whose columns (tg - 63 .. tg + 15 over the lanes) all lie outside
    // the strip's band
    auto outside = [&](int tg) { return BAND && (tg + G - 1 < band_jlo || tg - (kWave - 1) > band_jhi); };

    if (wv == 0) {
      // ---- the recurrence
      const double band_b = BAND ? band_halfwidth(M, N, a.band) : 0.0;
      double* st = a.states + pd.state_base + (int64_t)s * NG * (RHO + 1) * kWave + lane;
      double left[RHO];
#pragma unroll
      for (int r = 0; r < RHO; ++r) left[r] = INF;
      double upprev = (s == 0 && lane == 0) ? 0.0 : INF;
      double bot = INF;
      const int sb = lane == kWave - 1 ? 0 : G + lane;   // staging slot of step 0
      auto group = [&](auto full_tag, auto inside_tag, int g) {
        constexpr bool FULL = decltype(full_tag)::value;
        constexpr bool TEST = BAND && !decltype(inside_tag)::value;
        constexpr int kPre = 2;   // steps between the read of a step's LDS operands and their use
        const int tg = g * G, b = g & 1;
        double2 dn[G];
        double bn[G];
        auto pre = [&](int u) {
          dn[u] = dl[b][u][lane];
          bn[u] = binr[b][u];
        };
#pragma unroll
        for (int u = 0; u < kPre; ++u) pre(u);
#pragma unroll
        for (int u = 0; u < G; ++u) {
          if (u + kPre < G) pre(u + kPre);
          const int j = tg + u - lane;
          const double upin = shr1_f64(bot, bn[u]);
          double dg = upprev, up = upin;
          upprev = upin;
          if (FULL || (j >= 0 && j < N)) {
            const double delta[RHO] = {dn[u].x, dn[u].y};
            // band coordinate of row ib at column j (exact in float64)
            const double bd0 = (double)ib * (double)(N - 1) - (double)j * (double)(M - 1);
#pragma unroll
            for (int r = 0; r < RHO; ++r) {
              const double lf = left[r];
              double rv;
              if constexpr (TEST) {
                const bool inb = __builtin_fabs(bd0 + (double)r * (double)(N - 1)) <= band_b;
                const SoftMin sm = softmin3_band(dg, up, lf, inb);
                rv = inb ? delta[r] + sm.v : INF;
              } else {
                rv = delta[r] + softmin3(dg, up, lf).v;
              }
              dg = lf;
              up = rv;
              left[r] = rv;
            }
            bot = left[RHO - 1];
          }
          stg[b][sb + u] = bot;
        }
      };
      team_barrier();   // phase -1
      for (int g = 0; g <= NG; ++g) {
        team_barrier();
        if (g == NG) break;
        const int tg = g * G;
        {   // checkpoint: the sweep state at the start of these 16 steps
          double* p = st + (int64_t)g * (RHO + 1) * kWave;
#pragma unroll
          for (int r = 0; r < RHO; ++r) p[r * kWave] = left[r];
          p[RHO * kWave] = upprev;
        }
        if (outside(tg)) {
          // only the bookkeeping: +inf state and bottom row, and lane 0's
          // diagonal input of the next step; a lane already past column N-1
          // keeps its values (as the sweep would)
          if (tg + G - 1 - lane >= 0 && tg - lane <= N - 1) {
#pragma unroll
            for (int r = 0; r < RHO; ++r) left[r] = INF;
            bot = INF;
          }
          upprev = (lane == 0 && has_prev) ? binr[g & 1][G - 1] : INF;
          if (lane < G) stg[g & 1][lane] = INF;
        } else if (tg >= kWave - 1 && tg + G <= N) {
          if (BAND && tg - (kWave - 1) >= band_in_lo && tg + G - 1 <= band_in_hi)
            group(std::true_type{}, std::true_type{}, g);
          else
            group(std::true_type{}, std::false_type{}, g);
        } else {
          group(std::false_type{}, std::false_type{}, g);
        }
      }
      if (ib <= M - 1 && M - 1 < ib + RHO) {
        const int rl = M - 1 - ib;
        double v = left[0];
#pragma unroll
        for (int r = 1; r < RHO; ++r)
          if (r == rl) v = left[r];
        a.value[pd.out] = v / k;
      }
    } else if (wv == 1) {
      // ---- inputs: Y columns and the strip above's bottom row
      const double* row_in = a.rows + pd.aux_base + (int64_t)(s - 1) * N;
      const __amdgpu_buffer_rsrc_t rr_in = rsrc(row_in, has_prev ? N * 8 : 0);
      bool gave_up = false;
      TY yv[D];
      auto load_cols = [&](int g) {   // columns 16 g .. 16 g + 15, from lanes 0 .. 15
        const int64_t row = (pd.y_off + min(g * G + (lane & (G - 1)), N - 1)) * D;
#pragma unroll
        for (int c = 0; c < D; ++c) yv[c] = Y[row + c];
      };
      auto put_cols = [&](int g) {
        if (lane < G) {
          const int j = g * G + lane;
          double yc[D];
#pragma unroll
          for (int c = 0; c < D; ++c) yc[c] = j < N ? (static_cast<double>(yv[c]) - mu[c]) * sk : 0.0;
          ring_col<D>(ys, yq, j & (kRing - 1), yc);
        }
      };
      double pr = 0.0;
      auto fetch = [&](int g) {
        const int j = g * G + lane;
        pr = ld_dev(rr_in, lane < G && j < N ? j * 8 : kDrop);
      };
      auto settle = [&](int g) {   // waits until none of the group's values is a sentinel any more
        const int j = g * G + lane;
        if (has_prev && !gave_up) {
          auto ready = [&]() {
            return lane >= G || j >= N || (unsigned long long)__double_as_longlong(pr) != kSentR;
          };
          int polls = 0;
          while (!__all(ready())) {
            if (polls > 8) poll_backoff(polls, a.relaxed_wait);
            if (++polls > kSpinLimit) {   // never expected: report and carry on
              if (lane == 0) atomicOr(a.status, kStatusSpinTimeout);
              gave_up = true;
              break;
            }
            fetch(g);
          }
        }
        if (lane < G) binr[g & 1][lane] = has_prev && j < N ? pr : INF;
      };
      load_cols(0);
      fetch(0);
      put_cols(0);
      load_cols(1);
      team_barrier();   // phase -1
      for (int g = -1; g < NG; ++g) {
        if (g + 1 < NG) {
          put_cols(g + 2);
          load_cols(g + 3);
          settle(g + 1);
          fetch(g + 2);
        }
        team_barrier();
      }
    } else {
      // ---- costs of steps cs .. cs + 7 of a group
      const int cs = (wv - 2) * (G / 2);
      double* row_out = a.rows + pd.aux_base + (int64_t)s * N;
      const __amdgpu_buffer_rsrc_t ro = rsrc(row_out, has_next ? N * 8 : 0);
      double xr[RHO][D], xx[RHO];
#pragma unroll
      for (int r = 0; r < RHO; ++r) {
#pragma unroll
        for (int c = 0; c < D; ++c)
          xr[r][c] = (ib + r < M) ? (a.x[(pd.x_off + ib + r) * D + c] - mu[c]) * sk : 0.0;
        xx[r] = sq_norm<D>(xr[r]);
      }
      team_barrier();   // phase -1
      for (int g = -1; g <= NG; ++g) {
        if (wv == 2 && has_next && g > 0) {
          // bottom row of group g - 1: columns 16 (g - 1) - 63 .. + 15
          const int j = (g - 1) * G - (kWave - 1) + lane;
          const bool w = lane < G && j >= 0 && j < N;
          st_dev(ro, w ? j * 8 : kDrop, stg[(g - 1) & 1][lane & (G - 1)]);
        }
        if (g == NG) break;
        if (g + 1 < NG && !outside((g + 1) * G)) {
          const int yb = ((g + 1) * G + cs - lane) & (kRing - 1);
          const int b = (g + 1) & 1;
#pragma unroll
          for (int u = 0; u < G / 2; ++u) {
            double y[D];
#pragma unroll
            for (int c = 0; c < D; ++c) y[c] = ys[c][yb + u];
            const double yy = yq[yb + u];
            dl[b][cs + u][lane] = make_double2(sq_cost<D>(xr[0], xx[0], y, yy), sq_cost<D>(xr[1], xx[1], y, yy));
          }
        }
        team_barrier();
      }
    }
    __syncthreads();   // the staging buffers and s_item are free again
  }
}

}  // namespace

template <typename TY, int D>
static hipError_t launch_soft_team_t(const SoftArgs& a, int groups, hipStream_t st) {
  const dim3 block(kWave * kTeamWaves);
  if (a.band > 0.0)
    hipLaunchKernelGGL((soft_fwd_team_kernel<TY, D, kSoftRho, true>), dim3(groups), block, 0, st, a);
  else
    hipLaunchKernelGGL((soft_fwd_team_kernel<TY, D, kSoftRho, false>), dim3(groups), block, 0, st, a);
  return hipGetLastError();
}

hipError_t launch_soft_team(int d, int ydtype, const SoftArgs& a, int groups, hipStream_t st) {
#define CALLS(D) (ydtype == 0 ? launch_soft_team_t<float, D>(a, groups, st) \
                              : launch_soft_team_t<double, D>(a, groups, st))
  WTS_SOFT_D_SWITCH(d, CALLS)
#undef CALLS
}

}  // namespace wts
