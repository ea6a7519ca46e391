// wts_soft_wave.hip -- the Soft-DTW backward, one wave to a strip, for batches
// whose tiles with a non-zero e keep the compute units busy (many pairs, a wide
// E, or every tile swept: plan option dense_e).
//
// The workgroup form (wts_soft_bwd.hip) gives a strip a whole compute unit,
// because the chain of a pair's strips bounds batches of few pairs.  Where the
// arithmetic bounds it, one wave that replays, pushes and sums its tiles in
// turn, two or three to a SIMD, spends fewer instructions a tile and needs no
// barriers: wts_rules.h (bwd_wave_tiles) has the times of both and the line
// between them.  2000 cycles of 1000 (d = 3, narrow / wide E) 1.84 / 3.59 ms by
// workgroups, 1.02 / 2.1 by waves; every tile swept (d = 6): 128 x 8k 24.5 / 16.9,
// 512 x 800 1.54 / 1.16, 64 x 4k 3.3 / 3.5.
// The operations of a cell, and so its bits, are those of the workgroup form.
#include "wts_soft_link.h"

namespace wts {

namespace {

template <typename TY, int D, int RHO, bool BAND>
__global__ __launch_bounds__(kWave, D <= 3 && !BAND ? 3 : 2) void soft_bwd_wave_kernel(SoftArgs a) {
  constexpr int H = kWave * RHO;
  __shared__ double ys[D][kRing + 16];     // -2 y' of the columns (see sq_cost)
  __shared__ double yq[kRing + 16];        // |y'|^2
  __shared__ double bin_fwd[kTile];        // lane 0's upper input for the replay
  __shared__ float bin_up[kTile];          // lane 63's pushes from the strip below
  __shared__ float bin_dg[kTile];
  // lane 0's pushes for the strip above in slots 0..15; slots 16 + lane + u
  // take the other lanes' writes
  __shared__ float bout_up[kTile + kWave + kTile];
  __shared__ float bout_dg[kTile + kWave + kTile];
  __shared__ int s_item;
  const int lane = threadIdx.x;
  const int bsl = lane == 0 ? 0 : kTile + lane;
  const TY* __restrict__ Y = static_cast<const TY*>(a.y);
  const double INF = inf_d();
  const double k = a.kscale;
  const double sk = __builtin_sqrt(k);   // x and y enter as sqrt(k) (x - mu), sqrt(k) (y - mu)
  if (skipped(a.skip)) return;   // every workgroup: no strip waits for another
  // the whole queue, or what the workgroups handed over
  int first = 0;
  int* queue = a.queue;
  if (a.wave_tiles > 0) {
    first = uni(ld_dev(a.queue + kHandOver)) - 1;
    if (first < 0) return;
    queue = a.queue + kHandQueue;
  }

  for (;;) {
    if (lane == 0) s_item = first + atomicAdd(queue, 1);
    __syncthreads();
    const int item = __builtin_amdgcn_readfirstlane(s_item);   // uniform: scalar loads below
    __syncthreads();
    if (item >= a.n_items) break;
    const int2 it = a.items[item];
    const PairDesc pd = uniform(a.pairs[uni(it.x)]);
    double mu[D];
#pragma unroll
    for (int c = 0; c < D; ++c) mu[c] = a.x[pd.x_off * D + c];
    // first gradient row of this pair (per-cycle blocks of L rows, or the packed X rows)
    const int64_t grow = uni(a.rows_packed ? pd.x_off : (int64_t)pd.out * a.L);
    const int s = uni(it.y);
    const int M = pd.M, N = pd.N;
    const int i0 = s * H;
    const int ib = i0 + lane * RHO;
    const double band_b = BAND ? band_halfwidth(M, N, a.band) : 0.0;
    const bool has_above = s > 0;            // a strip above consumes our top-row pushes
    const bool has_below = s + 1 < pd.S;     // the strip below feeds our bottom row
    const int G = pd.WT;                     // 16-step tiles
    // Sakoe-Chiba band: a tile whose columns (tg - 63 .. tg + 15 over the
    // lanes) all lie outside the band of the strip's rows has e = 0 in every
    // cell (a cell outside the band gets nothing from its successors: their
    // weight towards a +inf cell is 0), so the sweep runs tiles g_lo .. g_hi
    // only.
    int g_lo = 0, g_hi = G - 1;
    if (BAND) {
      int jlo_b, jhi_b;
      band_strip_cols(M, N, a.band, i0, min(i0 + H, M) - 1, &jlo_b, &jhi_b);
      g_hi = min(G - 1, (jhi_b + kWave - 1) / 16);   // last tile with tg - 63 <= jhi_b
      g_lo = min(g_hi, jlo_b / 16);                  // first tile with tg + 15 >= jlo_b
    }
    const double* row_fwd = a.rows + pd.aux_base + (int64_t)(s - 1) * N;
    const double* st = a.states + pd.state_base + (int64_t)s * G * (RHO + 1) * kWave;
    const __amdgpu_buffer_rsrc_t rf_in = rsrc(row_fwd, has_above ? N * 8 : 0);
    BwdLink link(a, pd, s, g_lo, 0, a.relaxed_wait);
    // the cell that closes the path, (M-1, N-1), receives e = 1: it is
    // pending as a left push into that cell before the sweep starts (lane
    // k_last computes no cell of its rows to the right of column N-1)
    const bool last = s + 1 == pd.S;
    const int k_last = (M - 1 - i0) / RHO;
    const int r_last = (M - 1 - i0) - k_last * RHO;

    double xr[RHO][D], xx[RHO];
#pragma unroll
    for (int r = 0; r < RHO; ++r) {
#pragma unroll
      for (int c = 0; c < D; ++c)
        xr[r][c] = (ib + r < M) ? (a.x[(pd.x_off + ib + r) * D + c] - mu[c]) * sk : 0.0;
      xx[r] = sq_norm<D>(xr[r]);
    }

    // float64 row accumulators: sum_j e and sum_j e (-2 y'_j)
    double acc_e[RHO], acc_ey[RHO][D];
    float pl[RHO], pdg[RHO];                  // pending left / diagonal pushes into each row
#pragma unroll
    for (int r = 0; r < RHO; ++r) {
      acc_e[r] = 0.0;
      pl[r] = (last && lane == k_last && r == r_last) ? 1.0f : 0.0f;
      pdg[r] = 0.0f;
#pragma unroll
      for (int c = 0; c < D; ++c) acc_ey[r][c] = 0.0;
    }
    float up0 = 0.0f, dg0 = 0.0f;             // this lane's row-0 pushes, sent up next step
    float recv_dg = 0.0f;                     // diagonal push received last step
    // any push still travelling inside the strip (wave-uniform)
    auto pending = [&]() {
      bool p = up0 != 0.0f || dg0 != 0.0f || recv_dg != 0.0f;
#pragma unroll
      for (int r = 0; r < RHO; ++r) p = p || pl[r] != 0.0f || pdg[r] != 0.0f;
      return __builtin_amdgcn_ballot_w64(p) != 0;
    };
    // a tile's replay inputs: the forward's sweep state at its first step and
    // (lanes 0..15) the strip above's bottom row at its 16 columns (the top
    // strip reads an empty buffer and uses +inf; columns past N are never used)
    double st_n[RHO + 1];
    double rf_n;
    auto load_tile_inputs = [&](int gg) {
#pragma unroll
      for (int r = 0; r <= RHO; ++r) st_n[r] = st[((int64_t)gg * (RHO + 1) + r) * kWave + lane];
      const int j = 16 * gg + lane;
      rf_n = __builtin_bit_cast(
          double, __builtin_amdgcn_raw_buffer_load_b64(rf_in, lane < kTile && j < N ? j * 8 : kDrop, 0, 0));
    };
    // the Y columns of tile gg (63 + 16 of them, through the ring)
    auto fill_ring = [&](int gg) {
      const int jlo = 16 * gg - (kWave - 1);
      for (int q = lane; q < 16 + kWave - 1; q += kWave) {
        const int j = jlo + q;
        double yc[D];
#pragma unroll
        for (int c = 0; c < D; ++c)
          yc[c] = (j >= 0 && j < N) ? (static_cast<double>(Y[(pd.y_off + j) * D + c]) - mu[c]) * sk
                                    : 0.0;
        ring_col<D>(ys, yq, j & (kRing - 1), yc);
      }
    };
    int n_swept = 0;
    bool ready = false;   // tile g's replay inputs and Y columns are here or in flight
    for (int g = g_hi; g >= g_lo; --g) {
      if (a.zero_skip && !pending()) {
        const int next = link.search(g);
        ready = ready && next == g;
        g = next;
        if (g < 0) break;
      } else {
        link.learn_start();
      }
      if (!ready) {
        load_tile_inputs(g);
        fill_ring(g);
        ready = true;
      }
      ++n_swept;
      const int tg = 16 * g;
      const int yb = (tg - lane) & (kRing - 1);   // ring slot of step 0's column
      // next tile's 16 new Y columns, stored after this tile
      // (unconditional loads from a clamped column, kept in the storage type
      // until the store: a conditional load would be waited for on the spot)
      TY yraw[D];
      const int jn = tg - 16 - (kWave - 1) + lane;
      {
        const int jc = min(max(jn, 0), N - 1);
#pragma unroll
        for (int c = 0; c < D; ++c) yraw[c] = Y[(pd.y_off + jc) * D + c];
      }
      // lane 0's upper input for the replay (bottom row of the strip above),
      // loaded during the previous tile
      if (lane < kTile) bin_fwd[lane] = has_above ? rf_n : INF;
      // lane 63's inputs: pushes of the strip below's top row at columns
      // tg-63 ..  The strip below usually runs far ahead: one read of its
      // counter covers many tiles, and only a counter short of what this
      // tile needs is read again.
      if (has_below) link.wait_below(tg - (kWave - 1));
      // the pushes are only needed by the backward half: loaded now (one
      // unconditional load each, zero outside the row or without a strip
      // below) and written to LDS after the replay
      float in_up, in_dg;
      link.load_in(tg - (kWave - 1) + lane, lane < kTile, in_up, in_dg);
      __syncthreads();

      // ---- replay the tile forward, keeping the soft-min weights
      double left[RHO];
#pragma unroll
      for (int r = 0; r < RHO; ++r) left[r] = st_n[r];
      double upprev = st_n[RHO];
      double bot = left[RHO - 1];
      // normalised soft-min weights of the up and left predecessors (the
      // diagonal takes the rest of the cell's e, so every cell passes on
      // exactly what it received)
      float wu[16][RHO], wl[16][RHO];
      const bool full = tg >= kWave - 1 && tg + 16 <= N;
      // The banded instances (two waves per SIMD, less latency hidden by
      // the other waves) read the LDS inputs of the lane shifts one step ahead.
      double bf_n = bin_fwd[0];
#pragma unroll
      for (int u = 0; u < 16; ++u) {
        const int t = tg + u;
        const int j = t - lane;
        double bf;
        if constexpr (BAND) {
          bf = bf_n;
          if (u + 1 < 16) bf_n = bin_fwd[u + 1];
        } else {
          bf = bin_fwd[u];
        }
        const double upin = shr1_f64(bot, bf);
        const double dgi = upprev;
        upprev = upin;
        if (full || (j >= 0 && j < N)) {
          double y[D];
#pragma unroll
          for (int c = 0; c < D; ++c) y[c] = ys[c][yb + u];
          const double yy = yq[yb + u];
          double dg = dgi, up = upin;
          const double bd0 = (double)ib * (double)(N - 1) - (double)j * (double)(M - 1);
#pragma unroll
          for (int r = 0; r < RHO; ++r) {
            const double lf = left[r];
            const bool inb = !BAND || __builtin_fabs(bd0 + (double)r * (double)(N - 1)) <= band_b;
            const double rv = replay_cell<D, BAND>(dg, up, lf, xr[r], xx[r], y, yy, inb, wu[u][r], wl[u][r]);
            dg = lf;
            up = rv;
            left[r] = rv;
          }
          bot = left[RHO - 1];
        }
      }

      if (lane < kTile) {
        bin_up[lane] = in_up;
        bin_dg[lane] = in_dg;
      }
      // the next tile's replay inputs, in flight during the backward half
      // (unconditional: the last tile reloads its own)
      load_tile_inputs(max(g - 1, 0));
      __syncthreads();

      // ---- backward over the tile
      float bu_n = bin_up[15], bd_n = bin_dg[15];
#pragma unroll
      for (int u = 15; u >= 0; --u) {
        const int t = tg + u;
        const int j = t - lane;
        float bu, bd;
        if constexpr (BAND) {
          bu = bu_n;
          bd = bd_n;
          if (u > 0) {
            bu_n = bin_up[u - 1];
            bd_n = bin_dg[u - 1];
          }
        } else {
          bu = bin_up[u];
          bd = bin_dg[u];
        }
        // pushes of the lane below (rows i+1): its up push for column j now,
        // its diagonal push for column j-1 next step
        const float recv_up = shl1_f32(up0, bu);
        const float recv_dg_next = shl1_f32(dg0, bd);
        if (full || (j >= 0 && j < N)) {
          double y[D];
#pragma unroll
          for (int c = 0; c < D; ++c) y[c] = ys[c][yb + u];
          float below_up = recv_up;          // push up from (i+1, j)
          float new_pdg[RHO], er[RHO];
#pragma unroll
          for (int r = RHO - 1; r >= 0; --r) {
            const float din = (r == RHO - 1) ? recv_dg : pdg[r];
            const float e = (below_up + pl[r]) + din;
            // (the split over the predecessors: see wts_soft_bwd.hip)
            const float pu_ = e * wu[u][r];
            const float pl_ = e * wl[u][r];
            const float dpush = (e - pu_) - pl_;
            below_up = pu_;
            pl[r] = pl_;
            if (r > 0) new_pdg[r - 1] = dpush;
            else dg0 = dpush;
            er[r] = e;
          }
          up0 = below_up;
#pragma unroll
          for (int r = 0; r + 1 < RHO; ++r) pdg[r] = new_pdg[r];
#pragma unroll
          for (int r = RHO - 1; r >= 0; --r) {
            const double e64 = er[r];
            acc_e[r] += e64;
#pragma unroll
            for (int c = 0; c < D; ++c) acc_ey[r][c] = __builtin_fma(e64, y[c], acc_ey[r][c]);
          }
        }
        // lane 0's pushes into slot u (a column past N holds a stale value,
        // never published), the other lanes' into scratch slots: no branch
        bout_up[bsl + u] = up0;
        bout_dg[bsl + u] = dg0;
        recv_dg = recv_dg_next;
      }
      __syncthreads();
      link.publish(g, bout_up[lane & (kTile - 1)], bout_dg[lane & (kTile - 1)]);
      if (g > 0 && lane < 16) {
        const bool in = jn >= 0 && jn < N;
        double yc[D];
#pragma unroll
        for (int c = 0; c < D; ++c) yc[c] = in ? (static_cast<double>(yraw[c]) - mu[c]) * sk : 0.0;
        ring_col<D>(ys, yq, jn & (kRing - 1), yc);
      }
      __syncthreads();
    }
    link.finish();
    if (a.tiles != nullptr && lane == 0) {
      atomicAdd(a.tiles, (unsigned long long)n_swept);
      atomicAdd(a.tiles + 1, (unsigned long long)(g_hi - g_lo + 1));
    }
    // per-row sums of this cycle: gradient 2 (b sum_j e - sum_j e y_j), which
    // is (2 x' sum_j e + sum_j e (-2 y'_j)) / sk, and mass
#pragma unroll
    for (int r = 0; r < RHO; ++r) {
      const int i = ib + r;
      if (i < M) {
        const int64_t o = grow + i;
#pragma unroll
        for (int c = 0; c < D; ++c)
          a.gsum[o * D + c] = (2.0 * xr[r][c] * acc_e[r] + acc_ey[r][c]) / sk;
        a.hsum[o] = acc_e[r];
      }
    }
    __syncthreads();
  }
}

}  // namespace

template <typename TY, int D>
static hipError_t launch_soft_wave_t(const SoftArgs& a, int grid, hipStream_t st) {
  if (a.band > 0.0)
    hipLaunchKernelGGL((soft_bwd_wave_kernel<TY, D, kSoftRho, true>), dim3(grid), dim3(kWave), 0, st, a);
  else
    hipLaunchKernelGGL((soft_bwd_wave_kernel<TY, D, kSoftRho, false>), dim3(grid), dim3(kWave), 0, st, a);
  return hipGetLastError();
}

hipError_t launch_soft_bwd_wave(int d, int ydtype, const SoftArgs& a, int grid, hipStream_t st) {
#define CALLS(D) (ydtype == 0 ? launch_soft_wave_t<float, D>(a, grid, st) \
                              : launch_soft_wave_t<double, D>(a, grid, st))
  WTS_SOFT_D_SWITCH(d, CALLS)
#undef CALLS
}

}  // namespace wts
