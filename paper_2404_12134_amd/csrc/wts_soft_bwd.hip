// wts_soft_bwd.hip -- the Soft-DTW backward sweep (wts_soft.h describes it), a
// workgroup to a strip.
#include "wts_soft_link.h"

namespace wts {

namespace {

// -------------------------------------------------------------- backward

// A workgroup sweeps a strip, its waves in step by one barrier a phase:
//   wave 0       the push sweep of one 16-step tile a phase, the search for the
//                next tile with a non-zero e, the exchange with the strips
//                below and above;
//   waves 1..4   the replay: each takes every fourth tile, four steps of it a
//                phase, and leaves the soft-min weights in LDS;
//   waves 5, 6   the row sums (a row of the lane each) of the tile pushed in the
//                phase before; wave 5 also brings in the Y columns of the tile
//                whose replay begins in the next phase.
// What bounds it is the chain of a pair's strips: a strip's e reaches the
// strip above only after 63 + 128 steps (the lanes' skew and the columns a path
// moves in 128 rows), so a tile's time counts twelve times a strip.  One wave
// that replayed, pushed and summed its tiles in turn took 5.5 to 7 us a tile;
// a phase takes 1.0 to 1.3 us, four steps of replay (2400 cycles) or the push
// sweep (2200).  128 cycles of 20k (d = 6) 14.8 -> 4.8 ms, 5 of 18k (d = 1)
// 10.7 -> 3.5 ms, 16 of 2k (d = 3) 1.30 -> 0.42 ms.
constexpr int kBwdReplay = 4;                 // replay waves, and phases a tile's replay takes
constexpr int kBwdWaves = kBwdReplay + 3;
constexpr int kBwdBufs = kBwdReplay + 1;      // tiles whose weights are in LDS at a time
constexpr int kBwdSteps = kTile / kBwdReplay; // steps a replay wave takes a phase
constexpr int kBwdRing = 256;                 // Y columns in LDS: seven tiles and the lanes' skew

// Live tiles above wave_tiles, over all strips left, from which the rest of the
// queue is handed to the waves: what the change itself takes, 0.1 to 0.15 ms.
constexpr int kBwdHandOver = 50000;
constexpr int kBwdWindow = 256;   // strips between two looks at the live tiles

// The workgroup that popped item `it`, every window of strips, compares the live
// tiles of the strips finished since the last look with wave_tiles (one thread;
// each strip costs one atomic that nobody waits for).  To hand over, it moves
// the item counter past the end, so that no workgroup pops any more, and leaves
// the first item that was not popped for the waves.
__device__ __forceinline__ void watch_width(const SoftArgs& a, int it) {
  const int now = ld_dev(a.queue + kLiveTiles), before = ld_dev(a.queue + kLiveBefore);
  st_dev(a.queue + kLiveBefore, now);
  const int64_t over = (int64_t)(unsigned)(now - before) - (int64_t)kBwdWindow * a.wave_tiles;
  if (over * (a.n_items - it) <= (int64_t)kBwdWindow * kBwdHandOver) return;
  const int left = atomicAdd(a.queue, a.n_items);
  if (left < a.n_items) st_dev(a.queue + kHandOver, left + 1);
}

template <typename TY, int D, int RHO, bool BAND>
__global__ __launch_bounds__(kWave * kBwdWaves) void soft_bwd_kernel(SoftArgs a) {
  static_assert(RHO == 2, "weights travel in pairs of rows");
  constexpr int H = kWave * RHO;
  __shared__ double ys[D][kBwdRing + kTile];     // -2 y' of the columns (see sq_cost), mirrored
  __shared__ double yq[kBwdRing + kTile];        // |y'|^2
  __shared__ float4 wb[kBwdBufs][kTile][kWave];  // up, left weights of rows 0 and 1
  __shared__ float2 eb[2][kTile][kWave];         // e of rows 0 and 1
  __shared__ double bfw[kBwdReplay][kTile];      // lane 0's upper input for the replay
  __shared__ float2 bin[kTile];                  // lane 63's pushes (up, diagonal) from below
  // lane 0's pushes for the strip above in slots 0..15; slots 16 + lane + u
  // take the other lanes' writes
  __shared__ float2 bout[kTile + kWave + kTile];
  __shared__ int ctl[3];                         // [phase & 1]: stop; [2]: next tile, -1 at the end
  __shared__ int s_item;
  const int wv = uni((int)threadIdx.x / kWave);
  const int lane = threadIdx.x % kWave;
  const TY* __restrict__ Y = static_cast<const TY*>(a.y);
  const double INF = inf_d();
  const double k = a.kscale;
  const double sk = __builtin_sqrt(k);   // x and y enter as sqrt(k) (x - mu), sqrt(k) (y - mu)
  if (skipped(a.skip)) return;   // every workgroup: no strip waits for another

  for (;;) {
    if (threadIdx.x == 0) {
      const int it = atomicAdd(a.queue, 1);
      s_item = it;
      if (a.wave_tiles > 0 && it > 0 && it % kBwdWindow == 0 && it < a.n_items) watch_width(a, it);
    }
    __syncthreads();
    const int item = uni(s_item);
    if (item >= a.n_items) break;
    const int2 it = a.items[item];
    const PairDesc pd = uniform(a.pairs[uni(it.x)]);
    const int s = uni(it.y);
    double mu[D];
#pragma unroll
    for (int c = 0; c < D; ++c) mu[c] = a.x[pd.x_off * D + c];
    const int M = pd.M, N = pd.N;
    const int i0 = s * H;
    const int ib = i0 + lane * RHO;
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
    // rows of the replay and of the row sums
    double xr[RHO][D], xx[RHO];
#pragma unroll
    for (int r = 0; r < RHO; ++r) {
#pragma unroll
      for (int c = 0; c < D; ++c)
        xr[r][c] = (ib + r < M) ? (a.x[(pd.x_off + ib + r) * D + c] - mu[c]) * sk : 0.0;
      xx[r] = sq_norm<D>(xr[r]);
    }
    // one Y column into the ring (zero outside the grid)
    auto put_col = [&](int j, const TY (&raw)[D]) {
      const bool in = j >= 0 && j < N;
      const int slot = j & (kBwdRing - 1);
      double q = 0.0;
#pragma unroll
      for (int c = 0; c < D; ++c) {
        const double v = in ? (static_cast<double>(raw[c]) - mu[c]) * sk : 0.0;
        q = c == 0 ? v * v : __builtin_fma(v, v, q);
        ys[c][slot] = -2.0 * v;
        if (slot < kTile) ys[c][slot + kBwdRing] = -2.0 * v;
      }
      yq[slot] = q;
      if (slot < kTile) yq[slot + kBwdRing] = q;
    };
    auto get_col = [&](int j, TY (&raw)[D]) {
      const int jc = min(max(j, 0), N - 1);
#pragma unroll
      for (int c = 0; c < D; ++c) raw[c] = Y[(pd.y_off + jc) * D + c];
    };
    // fills the ring for the first four tiles of a run that begins at tile g0
    auto fill_ring = [&](int g0) {
      const int j = 16 * (g0 - (kBwdReplay - 1)) - (kWave - 1) + (int)threadIdx.x;
      if (j < 16 * g0 + kTile) {
        TY raw[D];
        get_col(j, raw);
        put_col(j, raw);
      }
    };

    if (wv == 0) {
      // ---- push sweep, search and exchange
      const int bsl = lane == 0 ? 0 : kTile + lane;
      BwdLink link(a, pd, s, g_lo, 4, 0);
      // the cell that closes the path, (M-1, N-1), receives e = 1: it is
      // pending as a left push into that cell before the sweep starts (lane
      // k_last computes no cell of its rows to the right of column N-1)
      const bool last = s + 1 == pd.S;
      const int k_last = (M - 1 - i0) / RHO;
      const int r_last = (M - 1 - i0) - k_last * RHO;
      float pl[RHO], pdg[RHO];                  // pending left / diagonal pushes into each row
#pragma unroll
      for (int r = 0; r < RHO; ++r) {
        pl[r] = (last && lane == k_last && r == r_last) ? 1.0f : 0.0f;
        pdg[r] = 0.0f;
      }
      float up0 = 0.0f, dg0 = 0.0f;             // this lane's row-0 pushes, sent up next step
      float recv_dg = 0.0f;                     // diagonal push received last step
      int n_swept = 0;
      // any push still travelling inside the strip (wave-uniform)
      auto pending = [&]() {
        bool p = up0 != 0.0f || dg0 != 0.0f || recv_dg != 0.0f;
#pragma unroll
        for (int r = 0; r < RHO; ++r) p = p || pl[r] != 0.0f || pdg[r] != 0.0f;
        return __builtin_amdgcn_ballot_w64(p) != 0;
      };
      int g = g_hi;
      bool more = false;   // the next phase's input is in in_up, in_dg
      float in_up = 0.0f, in_dg = 0.0f;
      for (;;) {
        int g0 = g >= g_lo ? g : -1;
        if (g0 >= 0 && a.zero_skip && !pending()) g0 = link.search(g);
        else if (g0 >= 0) link.learn_start();
        more = false;
        if (lane == 0) ctl[2] = g0;
        team_barrier();
        if (g0 < 0) break;
        fill_ring(g0);
        team_barrier();
        g = g0;
        for (int ph = -kBwdReplay;; ++ph) {
          bool stop = false;
          if (ph >= 0) {
            const int tg = 16 * g;
            const int jl = tg - (kWave - 1) + lane;
            if (!more) {
              if (has_below) link.wait_below(tg - (kWave - 1));
              link.load_in(jl, lane < kTile, in_up, in_dg);
            }
            int pv = 0;   // the strip below's progress, read while the tile is swept
            const bool peek = has_below && !link.gave_up && link.seen_below < N - max(0, tg - 16 - (kWave - 1));
            if (peek && lane == 0) pv = ld_dev(link.below.prog);
            if (lane < kTile) bin[lane] = make_float2(in_up, in_dg);
            __atomic_signal_fence(__ATOMIC_SEQ_CST);
            __builtin_amdgcn_wave_barrier();
            const int b = ph % kBwdBufs;
            auto push16 = [&](auto full_tag) {
              constexpr bool FULL = decltype(full_tag)::value;
              constexpr int kPre = 3;   // steps between the read of a step's weights and their use
              float4 wn[kTile];
              float2 bn[kTile];
              auto pre = [&](int u) {
                wn[u] = wb[b][u][lane];
                bn[u] = bin[u];
              };
#pragma unroll
              for (int u = kTile - 1; u > kTile - 1 - kPre; --u) pre(u);
#pragma unroll
              for (int u = kTile - 1; u >= 0; --u) {
                if (u - kPre >= 0) pre(u - kPre);
                const int j = tg + u - lane;
                // pushes of the lane below (rows i+1): its up push for column j
                // now, its diagonal push for column j-1 next step
                const float recv_up = shl1_f32(up0, bn[u].x);
                const float recv_dg_next = shl1_f32(dg0, bn[u].y);
                float2 ev = make_float2(0.0f, 0.0f);
                if (FULL || (j >= 0 && j < N)) {
                  const float wu[RHO] = {wn[u].x, wn[u].z};
                  const float wl[RHO] = {wn[u].y, wn[u].w};
                  float below_up = recv_up;          // push up from (i+1, j)
                  float new_pdg[RHO], er[RHO];
#pragma unroll
                  for (int r = RHO - 1; r >= 0; --r) {
                    const float din = (r == RHO - 1) ? recv_dg : pdg[r];
                    const float e = (below_up + pl[r]) + din;
                    // e in [0, 1] is carried in float32; the row sums take it in
                    // float64.  Split e over the three predecessors: up and left
                    // by their weights, the diagonal takes the rest, so the three
                    // pushes add up to e up to one rounding of each subtraction
                    // (unbiased, where weights that summed to 1 only to float32
                    // rounding would drain or add ~1e-8 of the mass at every
                    // cell, systematically).  Written out here and in the one-wave
                    // form: as a shared function it cost this form 2.5 %
                    const float pu_ = e * wu[r];
                    const float pl_ = e * wl[r];
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
                  ev = make_float2(er[0], er[1]);
                }
                eb[ph & 1][u][lane] = ev;
                // lane 0's pushes into slot u (a column past N holds a stale
                // value, never published), the other lanes' into scratch slots
                bout[bsl + u] = make_float2(up0, dg0);
                recv_dg = recv_dg_next;
              }
            };
            if (tg >= kWave - 1 && tg + kTile <= N) push16(std::true_type{});
            else push16(std::false_type{});
            ++n_swept;
            __atomic_signal_fence(__ATOMIC_SEQ_CST);
            __builtin_amdgcn_wave_barrier();
            if (peek) {
              link.seen_below = max(link.seen_below, __builtin_amdgcn_readfirstlane(pv));
              link.learn_end();
            }
            {
              const float2 o = bout[lane & (kTile - 1)];
              link.publish(g, o.x, o.y);
            }
            stop = g == g_lo || (a.zero_skip && !pending());
            --g;
            more = !stop && (!has_below || link.gave_up || link.seen_below >= N - max(0, 16 * g - (kWave - 1)));
            if (more) link.load_in(16 * g - (kWave - 1) + lane, lane < kTile, in_up, in_dg);
          }
          if (lane == 0) ctl[ph & 1] = stop ? 1 : 0;
          team_barrier();
          if (stop) break;
        }
      }
      if (a.wave_tiles > 0 && lane == 0) atomicAdd(a.queue + kLiveTiles, n_swept);
      link.finish();
      if (a.tiles != nullptr && lane == 0) {
        atomicAdd(a.tiles, (unsigned long long)n_swept);
        atomicAdd(a.tiles + 1, (unsigned long long)(g_hi - g_lo + 1));
      }
    } else if (wv <= kBwdReplay) {
      // ---- replay: tile q of a run (g0 - q) by wave 1 + q % 4, in the four
      // phases before the one that pushes it
      const int me = wv - 1;
      const double band_b = BAND ? band_halfwidth(M, N, a.band) : 0.0;
      const double* row_fwd = a.rows + pd.aux_base + (int64_t)(s - 1) * N;
      const double* st = a.states + pd.state_base + (int64_t)s * G * (RHO + 1) * kWave;
      const __amdgpu_buffer_rsrc_t rf_in = rsrc(row_fwd, has_above ? N * 8 : 0);
      // a tile's inputs: the forward's sweep state at its first step and
      // (lanes 0..15) the strip above's bottom row at its 16 columns (the top
      // strip reads an empty buffer and uses +inf; columns past N are never used)
      double st_n[RHO + 1], rf_n = 0.0;
      auto load_tile = [&](int g) {
        g = max(g, 0);
#pragma unroll
        for (int r = 0; r <= RHO; ++r) st_n[r] = st[((int64_t)g * (RHO + 1) + r) * kWave + lane];
        const int j = 16 * g + lane;
        rf_n = __builtin_bit_cast(
            double, __builtin_amdgcn_raw_buffer_load_b64(rf_in, lane < kTile && j < N ? j * 8 : kDrop, 0, 0));
      };
      for (;;) {
        team_barrier();
        const int g0 = uni(ctl[2]);
        if (g0 < 0) break;
        load_tile(g0 - me);
        fill_ring(g0);
        team_barrier();
        int ph = -kBwdReplay;
        bool stop = false;
        for (int w = 0; w < me && !stop; ++w, ++ph) {   // the waves start a phase after each other
          team_barrier();
          stop = uni(ctl[ph & 1]) != 0;
        }
        for (int q = me; !stop; q += kBwdReplay) {
          const int g = g0 - q;
          const int tg = 16 * g;
          const int b = q % kBwdBufs;
          const bool live = g >= g_lo;
          const bool full = tg >= kWave - 1 && tg + kTile <= N;
          double left[RHO];
#pragma unroll
          for (int r = 0; r < RHO; ++r) left[r] = st_n[r];
          double upprev = st_n[RHO];
          double bot = left[RHO - 1];
          if (lane < kTile) bfw[me][lane] = has_above ? rf_n : INF;
          __atomic_signal_fence(__ATOMIC_SEQ_CST);
          __builtin_amdgcn_wave_barrier();
          load_tile(g - kBwdReplay);   // in flight during this tile
          auto steps = [&](auto full_tag, int u0) {
            constexpr bool FULL = decltype(full_tag)::value;
            // the LDS operands of all four steps first: read next to their
            // use, they cost a trip to LDS in every step's chain
            const int yb = (tg + u0 - lane) & (kBwdRing - 1);   // ring slot of the first column
            double bf[kBwdSteps], yy[kBwdSteps], y[kBwdSteps][D];
#pragma unroll
            for (int u = 0; u < kBwdSteps; ++u) {
              bf[u] = bfw[me][u0 + u];
              yy[u] = yq[yb + u];
#pragma unroll
              for (int c = 0; c < D; ++c) y[u][c] = ys[c][yb + u];
            }
#pragma unroll
            for (int u = 0; u < kBwdSteps; ++u) {
              const int j = tg + u0 + u - lane;
              const double upin = shr1_f64(bot, bf[u]);
              const double dgi = upprev;
              upprev = upin;
              float wu[RHO] = {}, wl[RHO] = {};
              if (FULL || (j >= 0 && j < N)) {
                double dg = dgi, up = upin;
                const double bd0 = (double)ib * (double)(N - 1) - (double)j * (double)(M - 1);
#pragma unroll
                for (int r = 0; r < RHO; ++r) {
                  const double lf = left[r];
                  const bool inb = !BAND || __builtin_fabs(bd0 + (double)r * (double)(N - 1)) <= band_b;
                  const double rv = replay_cell<D, BAND>(dg, up, lf, xr[r], xx[r], y[u], yy[u], inb,
                                                         wu[r], wl[r]);
                  dg = lf;
                  up = rv;
                  left[r] = rv;
                }
                bot = left[RHO - 1];
              }
              wb[b][u0 + u][lane] = make_float4(wu[0], wl[0], wu[1], wl[1]);
            }
          };
          for (int sub = 0; sub < kBwdReplay && !stop; ++sub, ++ph) {
            if (live) {
              if (full) steps(std::true_type{}, sub * kBwdSteps);
              else steps(std::false_type{}, sub * kBwdSteps);
            }
            team_barrier();
            stop = uni(ctl[ph & 1]) != 0;
          }
        }
      }
    } else {
      // ---- row sums, and the Y columns of later tiles
      const int r = wv - (kBwdReplay + 1);   // the row of the lane this wave sums
      // float64 accumulators: sum_j e and sum_j e (-2 y'_j)
      double acc_e = 0.0, acc_ey[D];
#pragma unroll
      for (int c = 0; c < D; ++c) acc_ey[c] = 0.0;
      // The LDS operands of kSum steps ahead of their use: left to the compiler
      // they are waited for one by one in some instances (band, three channels
      // or more), and the sums outlast the phase: 5 cycles of 18k (d = 6, band 0.6)
      // 5.87 ms, so 3.98.  Larger groups hold up the push sweep's own reads: two
      // steps / four / eight at d = 3 3.49 / 3.55 / 3.59 ms, two / four at d = 6 with
      // the band 4.08 / 3.98.
      constexpr int kSum = D <= 5 ? 2 : 4;
      auto add_tile = [&](int g, int b) {   // cells outside the grid have e = 0 and y = 0
        const int yb = (16 * g - lane) & (kBwdRing - 1);
#pragma unroll
        for (int u0 = kTile - kSum; u0 >= 0; u0 -= kSum) {
          float2 ev[kSum];
          double y[kSum][D];
#pragma unroll
          for (int u = kSum - 1; u >= 0; --u) {
            ev[u] = eb[b][u0 + u][lane];
#pragma unroll
            for (int c = 0; c < D; ++c) y[u][c] = ys[c][yb + u0 + u];
          }
          __builtin_amdgcn_sched_barrier(0);
#pragma unroll
          for (int u = kSum - 1; u >= 0; --u) {
            const double e = r == 0 ? ev[u].x : ev[u].y;
            acc_e += e;
#pragma unroll
            for (int c = 0; c < D; ++c) acc_ey[c] = __builtin_fma(e, y[u][c], acc_ey[c]);
          }
        }
      };
      for (;;) {
        team_barrier();
        const int g0 = uni(ctl[2]);
        if (g0 < 0) break;
        fill_ring(g0);
        team_barrier();
        TY raw[D] = {};
        // the 16 columns that tile q adds to the ring, by lanes 0..15
        auto first_col = [&](int q) { return 16 * (g0 - q) - (kWave - 1) + (lane & (kTile - 1)); };
        int ph = -kBwdReplay;
        for (;; ++ph) {
          const int q = ph + kBwdReplay + 1;   // the tile whose replay begins in the next phase
          if (r == 0 && q >= kBwdReplay && lane < kTile) put_col(first_col(q), raw);
          if (r == 0 && q + 1 >= kBwdReplay) get_col(first_col(q + 1), raw);
          if (ph >= 1) add_tile(g0 - (ph - 1), (ph - 1) & 1);
          team_barrier();
          if (uni(ctl[ph & 1])) break;
        }
        add_tile(g0 - ph, ph & 1);
      }
      // per-row sums of this cycle: gradient 2 (b sum_j e - sum_j e y_j), which
      // is (2 x' sum_j e + sum_j e (-2 y'_j)) / sk, and mass; the first
      // gradient row of this pair: per-cycle blocks of L rows, or the packed X rows
      const int64_t grow = a.rows_packed ? pd.x_off : (int64_t)pd.out * a.L;
      const int i = ib + r;
      if (i < M) {
        const int64_t o = grow + i;
#pragma unroll
        for (int c = 0; c < D; ++c)
          a.gsum[o * D + c] = (2.0 * (r == 0 ? xr[0][c] : xr[1][c]) * acc_e + acc_ey[c]) / sk;
        a.hsum[o] = acc_e;
      }
    }
    __syncthreads();
  }
}

}  // namespace

template <typename TY, int D>
static hipError_t launch_soft_bwd_t(const SoftArgs& a, int groups, hipStream_t st) {
  const dim3 block(kWave * kBwdWaves);
  if (a.band > 0.0)
    hipLaunchKernelGGL((soft_bwd_kernel<TY, D, kSoftRho, true>), dim3(groups), block, 0, st, a);
  else
    hipLaunchKernelGGL((soft_bwd_kernel<TY, D, kSoftRho, false>), dim3(groups), block, 0, st, a);
  return hipGetLastError();
}

hipError_t launch_soft_bwd(int d, int ydtype, const SoftArgs& a, int groups, hipStream_t st) {
#define CALLS(D) (ydtype == 0 ? launch_soft_bwd_t<float, D>(a, groups, st) \
                              : launch_soft_bwd_t<double, D>(a, groups, st))
  WTS_SOFT_D_SWITCH(d, CALLS)
#undef CALLS
}

}  // namespace wts
