// wts_team.h -- the DTW sweep for batches of few strips, shared by the
// float64 (wts_team2.hip, wts_team4.hip) and the float32-decision instances (wts_team32.hip).
//
// With one strip per SIMD or fewer, the one-wave sweep (wts_sweep.h) is bound
// by the issue of its own instructions: 60 to 90 a step, one every four
// cycles, while the other SIMDs of the compute unit idle.  Here a workgroup
// of four waves sweeps a strip, one wave to a SIMD:
//   wave 0      the recurrence: minima, sums, argmins and tags;
//   wave 1      reads the Y columns and the bottom row of the strip above;
//   waves 2, 3  the costs, half of a group's 16 steps each, through LDS;
//               wave 2 also stores the strip's own bottom row.
// In each phase (one barrier) wave 0 sweeps group g while the costs of group
// g + 1, its upper row and the columns of group g + 2 are brought in and the
// bottom row of group g - 1 goes out.  A value sweep is then 3 instructions a
// row and about 8 a step for wave 0, whatever the channel count.  What bounds
// it is wave 0's chain: 7.5 ns a row (value) or 16 (length, codes) and 25 to
// 29 ns a step, where one wave a strip takes 169 ns a step of 4 rows (d = 3).
// Scores of one cycle of 4.8k (L = 4077) 970 -> 560 us, paths of 24 cycles of
// 2k (d = 6, with their recovery) 793 -> 432 us.
// The operations of a cell, and so its bits, are those of the one-wave sweep;
// so are the strip rows, checkpoints and codes it leaves.
#pragma once
#include "wts_sweep.h"

namespace wts {

namespace {

constexpr int kTeamGroup = 16;   // steps per phase
constexpr int kTeamWaves = 4;

template <typename TX, typename TY, typename TC, int D, int RHO, int MODE, bool EUC>
__global__ __launch_bounds__(kWave * kTeamWaves) void dtw_team_kernel(FwdArgs a) {
  constexpr int H = kWave * RHO;
  constexpr int G = kTeamGroup;
  constexpr int RH = RHO / 2;      // rows come in pairs: one LDS access of two values
  constexpr bool kAux = MODE == MODE_DIST_LEN || MODE == MODE_SUB || MODE == MODE_PATHT;
  constexpr bool kCodes = MODE == MODE_PATHT;
  struct alignas(2 * sizeof(TC)) Two { TC v[2]; };
  __shared__ TC ys[D][kRing + G];          // Y ring; slots kRing .. mirror slots 0 .. G - 1
  __shared__ Two dl[2][G][RH][kWave];      // costs of a group, by step, row pair and lane
  __shared__ TC binr[2][G];                // the strip above's bottom row at a group's columns
  __shared__ int binx[2][G];
  __shared__ TC stg_r[2][G + kWave + G];   // lane 63's bottom row; the other lanes' writes follow
  __shared__ int stg_x[2][G + kWave + G];
  __shared__ int s_item;
  const int wv = uni((int)threadIdx.x / kWave);
  const int lane = threadIdx.x % kWave;
  const TX* __restrict__ X = static_cast<const TX*>(a.x);
  const TY* __restrict__ Y = static_cast<const TY*>(a.y);
  const TC INF = (TC)inf_d();
  if (skipped(a.skip)) return;   // every workgroup: no strip waits for another

  // Launched with a workgroup a strip, so each takes one and its second pop ends
  // it.  Built without the loop the kernel was slower where teams share compute
  // units: scores of 32 x 4.4k (L = 4000, d = 6) 925 -> 1049 us.
  for (;;) {
    if (threadIdx.x == 0) s_item = atomicAdd(a.queue, 1);
    __syncthreads();
    const int item = uni(s_item);
    if (item >= a.n_items) break;
    const int2 it = a.items[item];
    const PairDesc pd = uniform(a.pairs[uni(it.x)]);
    const int s = uni(it.y);
    const int M = pd.M, N = pd.N;
    const int i0 = s * H;
    const int ib = i0 + lane * RHO;
    const bool has_prev = s > 0;
    const bool has_next = s + 1 < pd.S;
    const int NG = pd.WT;                  // groups of 16 steps
    const int RS = row_stride(N);
    constexpr int kB = (int)sizeof(TC);

    if (wv == 0) {
      // ---- the recurrence
      TC left[RHO];
      int lx[RHO];
      uint32_t accd[RHO], accu[RHO];
#pragma unroll
      for (int r = 0; r < RHO; ++r) { left[r] = INF; lx[r] = border_tag<MODE>(ib + r); accd[r] = accu[r] = 0u; }
      TC upprev = (s == 0 && lane == 0) ? (TC)0 : INF;   // r(-1,-1) = 0 at the origin
      int upprevx = border_tag<MODE>(ib - 1);
      TC bot = INF;
      int botx = border_tag<MODE>(ib + RHO - 1);
      const bool last_strip = s + 1 == pd.S;
      const int rl_last = M - 1 - ib;
      TC sub_best = INF;
      int sub_end = 0, sub_start = 0;
      const int sb = lane == kWave - 1 ? 0 : G + lane;   // staging slot of step 0

      auto group = [&](auto full_tag, int g) {
        constexpr bool FULL = decltype(full_tag)::value;
        constexpr int kPre = 3;   // steps between the read of a step's LDS operands and their use
        const int tg = g * G, b = g & 1;
        Two dn[G][RH];
        TC bn[G];
        int bxn[G];
        auto pre = [&](int u) {
#pragma unroll
          for (int h = 0; h < RH; ++h) dn[u][h] = dl[b][u][h][lane];
          bn[u] = binr[b][u];
          bxn[u] = MODE == MODE_DIST_LEN || MODE == MODE_SUB ? binx[b][u] : 0;
        };
#pragma unroll
        for (int u = 0; u < kPre; ++u) pre(u);
#pragma unroll
        for (int u = 0; u < G; ++u) {
          const int t = tg + u;
          const int j = t - lane;
          if (u + kPre < G) pre(u + kPre);
          const TC upin = shr1_t(bot, bn[u]);
          int upinx = 0, dgx0 = 0;
          if (MODE == MODE_DIST_LEN) {
            upinx = shr1_i32(botx, bxn[u]);
            dgx0 = upprevx;
          } else if (MODE == MODE_PATHT) {
            upinx = shr1_i32(botx, 2 * t);
            dgx0 = lane == 0 ? upinx + 1 : upprevx;
          } else if (MODE == MODE_SUB) {
            upinx = shr1_i32(botx, s == 0 ? t : bxn[u]);
            dgx0 = s == 0 && lane == 0 ? upinx : upprevx;
          }
          TC dg = upprev, up = upin;
          int dgx = dgx0, upx = upinx;
          upprev = upin;
          upprevx = upinx;
          bool isd_r[RHO], isu_r[RHO];
#pragma unroll
          for (int r = 0; r < RHO; ++r) { isd_r[r] = false; isu_r[r] = false; }
          if (FULL || (j >= 0 && j < N)) {
#pragma unroll
            for (int r = 0; r < RHO; ++r) {
              // the minimum with the row above's fresh value comes last (that
              // value is the chain of the step); dg <= m is dg <= min(up, lf)
              const TC lf = left[r];
              const TC m = min_t(up, min_t(dg, lf));
              const TC rv = dn[u][r / 2].v[r % 2] + m;
              int rxv = 0;
              if (kAux || kCodes) {
                // the select that takes the row above's fresh tag comes last
                const bool isd = dg <= m;
                const bool isu = up <= lf;
                const int lfx = MODE == MODE_DIST_LEN ? lx[r] + 1 : lx[r];
                const int t1 = __builtin_unpredictable(isd) ? dgx : lfx;
                rxv = __builtin_unpredictable(isu && !isd) ? upx : t1;
                isd_r[r] = isd;
                isu_r[r] = isu;
              }
              dg = lf;
              dgx = lx[r];
              up = rv;
              upx = rxv;
              left[r] = rv;
              lx[r] = rxv;
            }
            bot = left[RHO - 1];
            botx = lx[RHO - 1];
            if (MODE == MODE_SUB && last_strip) {
              TC v = left[0];
              int vx = lx[0];
#pragma unroll
              for (int r = 1; r < RHO; ++r)
                if (r == rl_last) { v = left[r]; vx = lx[r]; }
              const bool better = v < sub_best;
              sub_best = better ? v : sub_best;
              sub_end = better ? j : sub_end;
              sub_start = better ? vx : sub_start;
            }
          }
          if (kCodes) {
#pragma unroll
            for (int r = 0; r < RHO; ++r) {
              accd[r] = push_bit(accd[r], isd_r[r]);
              accu[r] = push_bit(accu[r], isu_r[r]);
            }
          }
          stg_r[b][sb + u] = bot;
          if (kAux) stg_x[b][sb + u] = botx;
        }
      };
      team_barrier();   // phase -1
      for (int g = 0; g <= NG; ++g) {
        team_barrier();
        if (g == NG) break;
        if (MODE == MODE_CKPT && (g & 3) == 0) {   // the sweep state every 64 steps
          TC* p = reinterpret_cast<TC*>(a.states) + pd.state_base +
                  ((int64_t)s * ((NG + 3) >> 2) + (g >> 2)) * (RHO + 1) * kWave + lane;
#pragma unroll
          for (int r = 0; r < RHO; ++r) p[r * kWave] = left[r];
          p[RHO * kWave] = upprev;
        }
        if (g * G >= kWave - 1 && g * G + G <= N) group(std::true_type{}, g);
        else group(std::false_type{}, g);
        if (kCodes && (g & 1)) {
          uint32_t* cw = a.codes + pd.code_base + (int64_t)(s * NG + g - 1) * RHO * kWave + lane;
#pragma unroll
          for (int r = 0; r < RHO; ++r) {
            cw[r * kWave] = accd[r];
            cw[(RHO + r) * kWave] = accu[r];
          }
        }
      }
      if (ib <= M - 1 && M - 1 < ib + RHO) {
        const int rl = M - 1 - ib;
        TC v = left[0];
        int vx = lx[0];
#pragma unroll
        for (int r = 1; r < RHO; ++r)
          if (r == rl) { v = left[r]; vx = lx[r]; }
        if (MODE == MODE_SUB) {
          a.out_dist[pd.out] = sub_best;
          a.out_aux[pd.out] = sub_start;
          a.out_end[pd.out] = sub_end;
        } else {
          a.out_dist[pd.out] = v;
          if (kAux) a.out_aux[pd.out] = MODE == MODE_DIST_LEN ? vx + M - 1 : vx;
        }
      }
    } else if (wv == 1) {
      // ---- inputs: Y columns and the strip above's bottom row
      const TC* r_in = reinterpret_cast<const TC*>(a.bnd_r) + pd.row_base + (int64_t)(s - 1) * RS;
      const int* x_in = a.bnd_aux + pd.row_base + (int64_t)(s - 1) * RS;
      const __amdgpu_buffer_rsrc_t rr_in = rsrc(r_in, has_prev ? RS * kB : 0);
      const __amdgpu_buffer_rsrc_t rx_in = rsrc(x_in, has_prev ? RS * 4 : 0);
      bool gave_up = false;
      TY yv[D];
      auto load_cols = [&](int g) {   // columns 16 g .. 16 g + 15, from lanes 0 .. 15
        const int64_t row = (pd.y_off + min(g * G + (lane & (G - 1)), N - 1)) * D;
#pragma unroll
        for (int c = 0; c < D; ++c) yv[c] = Y[row + c];
      };
      auto put_cols = [&](int g) {
        if (lane < G) {
          const int j = g * G + lane, slot = j & (kRing - 1);
#pragma unroll
          for (int c = 0; c < D; ++c) {
            const TC v = j < N ? static_cast<TC>(yv[c]) : (TC)0;
            ys[c][slot] = v;
            if (slot < G) ys[c][slot + kRing] = v;
          }
        }
      };
      TC pr = (TC)0;
      int px = 0;
      auto fetch = [&](int g) {
        const int j = g * G + lane;
        const bool want = lane < G && j < N;
        pr = ld_row<TC>(rr_in, want ? (j + 63) * kB : kDrop);
        if (kAux) px = (int)__builtin_amdgcn_raw_buffer_load_b32(rx_in, want ? (j + 63) * 4 : kDrop, 0, 16);
      };
      // waits until none of the group's values is a sentinel any more
      auto settle = [&](int g) {
        const int j = g * G + lane;
        if (has_prev && !gave_up) {
          auto ready = [&]() {
            return lane >= G || j >= N || (!is_sent(pr) && (!kAux || px != kSentX));
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
        if (lane < G) {
          // above the first strip: +inf, or 0 for Sub-DTW (free start)
          binr[g & 1][lane] = has_prev ? (j < N ? pr : INF) : (MODE == MODE_SUB ? (TC)0 : INF);
          if (kAux) binx[g & 1][lane] = has_prev ? px : border_tag<MODE>(-1);
        }
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
      TC* r_out = reinterpret_cast<TC*>(a.bnd_r) + pd.row_base + (int64_t)s * RS;
      int* x_out = a.bnd_aux + pd.row_base + (int64_t)s * RS;
      const __amdgpu_buffer_rsrc_t rr_out = rsrc(r_out, RS * kB);
      const __amdgpu_buffer_rsrc_t rx_out = rsrc(x_out, RS * 4);
      TC xr[RHO][D];
#pragma unroll
      for (int r = 0; r < RHO; ++r)
#pragma unroll
        for (int c = 0; c < D; ++c)
          xr[r][c] = static_cast<TC>(X[(pd.x_off + min(ib + r, M - 1)) * D + c]);
      team_barrier();   // phase -1
      for (int g = -1; g <= NG; ++g) {
        if (wv == 2 && has_next && g > 0) {
          // bottom row of group g - 1: columns 16 (g - 1) - 63 .. + 15, at
          // indices 16 (g - 1) .. of the strip's row
          const int tg = (g - 1) * G;
          const int j = tg - 63 + lane;
          const bool w = lane < G && j >= 0 && j < N;
          st_dev(rr_out, w ? (tg + lane) * kB : kDrop, stg_r[(g - 1) & 1][lane & (G - 1)]);
          if (kAux) st_dev(rx_out, w ? (tg + lane) * 4 : kDrop, stg_x[(g - 1) & 1][lane & (G - 1)]);
        }
        if (g == NG) break;
        if (g + 1 < NG) {
          const int tg = (g + 1) * G;
          const int yb = (tg + cs - lane) & (kRing - 1);
          const int b = (g + 1) & 1;
#pragma unroll
          for (int u = 0; u < G / 2; ++u) {
            TC y[D];
#pragma unroll
            for (int c = 0; c < D; ++c) y[c] = ys[c][yb + u];
#pragma unroll
            for (int h = 0; h < RH; ++h) {
              Two d2;
#pragma unroll
              for (int q = 0; q < 2; ++q) {
                TC delta = sq_cost<TC, D>(xr[2 * h + q], y);
                if constexpr (EUC) delta = __builtin_sqrt(delta);
                d2.v[q] = delta;
              }
              dl[b][cs + u][h][lane] = d2;
            }
          }
        }
        team_barrier();
      }
    }
    __syncthreads();   // the staging buffers and s_item are free again
  }
}

template <typename TX, typename TY, typename TC, int D, int RHO, int MODE, bool EUC>
hipError_t launch_team_one(const FwdArgs& a, int groups, hipStream_t st) {
  hipLaunchKernelGGL((dtw_team_kernel<TX, TY, TC, D, RHO, MODE, EUC>), dim3((unsigned)groups),
                     dim3(kWave * kTeamWaves), 0, st, a);
  return hipGetLastError();
}

template <typename TX, typename TY, typename TC, int D, int RHO>
hipError_t launch_team_t(int mode, bool euc, const FwdArgs& a, int groups, hipStream_t st) {
  if (mode == MODE_CKPT) return launch_team_one<TX, TY, TC, D, RHO, MODE_CKPT, false>(a, groups, st);
  if (mode == MODE_PATHT) return launch_team_one<TX, TY, TC, D, RHO, MODE_PATHT, false>(a, groups, st);
  if (mode == MODE_SUB && !euc) return launch_team_one<TX, TY, TC, D, RHO, MODE_SUB, false>(a, groups, st);
  if (mode != MODE_DIST_LEN) return hipErrorInvalidValue;
  if (euc) {
    if constexpr (sizeof(TC) == 8) return launch_team_one<TX, TY, TC, D, RHO, MODE_DIST_LEN, true>(a, groups, st);
    return hipErrorInvalidValue;
  }
  return launch_team_one<TX, TY, TC, D, RHO, MODE_DIST_LEN, false>(a, groups, st);
}

// Value sweeps between two cycles (medoid): X is a cycle.
template <typename TC, int D, int RHO>
hipError_t launch_team_d(int mode, bool euc, bool x_is_cycle, int ydtype, const FwdArgs& a,
                         int groups, hipStream_t st) {
  if (x_is_cycle != (mode == MODE_DIST)) return hipErrorInvalidValue;
  if (ydtype == 0) {
    if (x_is_cycle) return launch_team_one<float, float, TC, D, RHO, MODE_DIST, false>(a, groups, st);
    return launch_team_t<double, float, TC, D, RHO>(mode, euc, a, groups, st);
  }
  if constexpr (sizeof(TC) == 8) {
    if (x_is_cycle) return launch_team_one<double, double, TC, D, RHO, MODE_DIST, false>(a, groups, st);
    return launch_team_t<double, double, TC, D, RHO>(mode, euc, a, groups, st);
  }
  return hipErrorInvalidValue;
}

template <typename TC, int RHO>
hipError_t launch_team_impl(int d, int mode, bool euc, bool x_is_cycle, int ydtype,
                            const FwdArgs& a, int groups, hipStream_t st) {
#define CALLT(D, R) launch_team_d<TC, D, R>(mode, euc, x_is_cycle, ydtype, a, groups, st)
  WTS_D_SWITCH(d, RHO, CALLT)
#undef CALLT
}

}  // namespace

}  // namespace wts
