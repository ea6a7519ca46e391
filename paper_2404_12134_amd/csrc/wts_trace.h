// wts_trace.h -- path recovery from the checkpoints of a value sweep
// (MODE_CKPT), shared by the float64 (wts_trace.hip) and the float32-decision
// instances (wts_trace32.hip).
//
// The sweep keeps no argmin codes: every 64 steps it stores each lane's
// state (its RHO cumulative costs at the previous column and the diagonal
// input from above).  Only the tiles that a path crosses are swept again,
// now with the two comparisons and the bit packing of the codes, about 2 %
// of the cells on long pairs.
#pragma once
#include "wts_sweep.h"
#include "wts_walk.h"

namespace wts {

namespace {

constexpr int kTraceWaves = 8;   // tiles of 64 steps swept again at once
constexpr int kTraceCols = 64 * kTraceWaves + 64;

// One workgroup per pair.  From (M-1, N-1) upwards, strip by strip: the eight
// waves sweep the eight tiles ending at the step where the path enters the
// strip's bottom row (a path that moves as many columns as rows crosses six
// or seven of them at 5 rows per lane), leaving their codes in LDS, then wave
// 0 walks the strip on the scalar unit (walk_strip) and the workgroup goes on
// with the strip above.  Per row it records the run of columns [lo, hi] the
// path occupies.  The pairs run in parallel, the strips of a pair in turn, so
// what bounds it is the latency of one strip (14 us and 6 us a channel up to 256
// pairs: walk_pairs_pays): two of the tiles share a SIMD.  With the sweep
// that needs no codes, DBA on 512 cycles of 1k-20k (d = 6) 26.9 -> 22.9 ms, 40
// of 45k in float32 54.3 -> 43.1 ms.  Sweeping the strip above at a predicted
// place while a strip is walked gained 4 % there and nothing in float64.
template <typename TY, typename TC, int D, int RHO>
__global__ __launch_bounds__(kWave * kTraceWaves) void trace_kernel(TraceArgs a) {
  constexpr int H = kWave * RHO;
  __shared__ TC ys[D][kTraceCols];        // columns 64 w_lo - 63 .. 64 w_hi + 63
  __shared__ TC rin[kWave * kTraceWaves]; // bottom row of the strip above, from column 64 w_lo
  __shared__ uint32_t m_nl[2 * kTraceWaves][RHO][kWave];   // code words of 32 steps
  __shared__ uint32_t m_dd[2 * kTraceWaves][RHO][kWave];
  __shared__ int ctl[8];
  const int tid = threadIdx.x;
  const int wv = uni(tid / kWave);
  const int lane = tid % kWave;
  if (skipped(a.skip)) return;
  const double* __restrict__ X = static_cast<const double*>(a.x);
  const TY* __restrict__ Y = static_cast<const TY*>(a.y);
  const TC INF = (TC)inf_d();
  const PairDesc pd = uniform(a.pairs[blockIdx.x]);
  const int M = pd.M, N = pd.N;
  const int RS = row_stride(N);
  const int WC = (pd.WT + 3) >> 2;        // tiles per strip
  const TC* states = reinterpret_cast<const TC*>(a.states) + pd.state_base;
  int2* runs = a.runs + (int64_t)pd.out * a.L;

  TC xr[RHO][D];
  auto load_rows = [&](int s) {
    const int ib = s * H + lane * RHO;
#pragma unroll
    for (int r = 0; r < RHO; ++r)
#pragma unroll
      for (int c = 0; c < D; ++c)
        xr[r][c] = static_cast<TC>(X[(pd.x_off + min(ib + r, M - 1)) * D + c]);
  };
  load_rows(pd.S - 1);

  const float slope = (float)N / (float)M;   // columns per row
  bool bad = false;
  int jx = N - 1;   // where the path enters the current strip's bottom row
  for (int s = pd.S - 1; s >= 0; --s) {
    const int i0 = s * H;
    const int iend = min(M, i0 + H) - 1;
    const bool has_prev = s > 0;
    const TC* r_in = reinterpret_cast<const TC*>(a.bnd_r) + pd.row_base + (int64_t)(s - 1) * RS;
    if (jx < 0 || jx >= N) bad = true;
    Walk st;
    st.q = iend - i0;
    st.j = jx;
    st.hi = jx;
    st.jtop = -1;
    int end = bad ? kWalkBad : kWalkMore;
    while (end == kWalkMore) {
      const int k = st.q / RHO;
      const int w_hi = (st.j + k) >> 6;
      // as many tiles as the rows left should cross at the pair's mean slope,
      // a quarter and a tile more (the tiles share the compute unit, and a
      // walk that needs another one costs a round of its own)
      const int want = (int)((float)(st.q + 1) * slope * 1.25f) + k + 64;
      const int w_lo = max(max(0, w_hi - (kTraceWaves - 1)), (st.j + k - want) >> 6);
      const int nt = w_hi - w_lo + 1;
      const bool mine = wv < nt;
      TC left[RHO], upprev = INF;
#pragma unroll
      for (int r = 0; r < RHO; ++r) left[r] = INF;
      if (mine) {
        const TC* sp = states + ((int64_t)s * WC + w_lo + wv) * (RHO + 1) * kWave + lane;
#pragma unroll
        for (int r = 0; r < RHO; ++r) left[r] = sp[r * kWave];
        upprev = sp[RHO * kWave];
      }
      {
        const int j = 64 * w_lo + tid;
        rin[tid] = has_prev && j < N && tid < 64 * nt ? r_in[j + 63] : INF;
        const int c0 = 64 * w_lo - 63;
        for (int q = tid; q < 64 * nt + 63; q += kWave * kTraceWaves) {
          const int jj = min(max(c0 + q, 0), N - 1);
#pragma unroll
          for (int c = 0; c < D; ++c) ys[c][q] = static_cast<TC>(Y[(pd.y_off + jj) * D + c]);
        }
      }
      __syncthreads();
      if (mine) {
        const int t0 = 64 * (w_lo + wv);
        const int yb = 64 * wv + 63 - lane;   // slot of step 0's column
        TC bot = left[RHO - 1];
        uint32_t ad[RHO], au[RHO];
#pragma unroll
        for (int r = 0; r < RHO; ++r) ad[r] = au[r] = 0u;
        auto group16 = [&](auto full_tag, int ub) {
          constexpr bool FULL = decltype(full_tag)::value;
#pragma unroll
          for (int u = 0; u < 16; ++u) {
            const int j = t0 + ub + u - lane;
            TC y[D];
#pragma unroll
            for (int c = 0; c < D; ++c) y[c] = ys[c][yb + ub + u];
            const TC upin = shr1_t(bot, rin[64 * wv + ub + u]);
            TC dg = upprev, up = upin;
            upprev = upin;
            bool isd[RHO], isu[RHO];
#pragma unroll
            for (int r = 0; r < RHO; ++r) { isd[r] = false; isu[r] = false; }
            if (FULL || (j >= 0 && j < N)) {
#pragma unroll
              for (int r = 0; r < RHO; ++r) {
                const TC lf = left[r];
                const TC m1 = min_t(up, lf);
                const TC rv = sq_cost<TC, D>(xr[r], y) + min_t(dg, m1);
                isd[r] = dg <= m1;
                isu[r] = up <= lf;
                dg = lf;
                up = rv;
                left[r] = rv;
              }
              bot = left[RHO - 1];
            }
#pragma unroll
            for (int r = 0; r < RHO; ++r) {
              ad[r] = push_bit(ad[r], isd[r]);
              au[r] = push_bit(au[r], isu[r]);
            }
          }
        };
        for (int ub = 0; ub < 64; ub += 16) {
          if (t0 + ub >= kWave - 1 && t0 + ub + 16 <= N) group16(std::true_type{}, ub);
          else group16(std::false_type{}, ub);
          if (ub & 16) {   // 32 steps in the words
#pragma unroll
            for (int r = 0; r < RHO; ++r) {
              m_dd[2 * wv + (ub >> 5)][r][lane] = ad[r];
              m_nl[2 * wv + (ub >> 5)][r][lane] = ad[r] | au[r];
            }
          }
        }
      }
      __syncthreads();
      if (wv == 0) {
        end = walk_strip<RHO>(st, 64 * w_lo, runs + i0,
                              [&](int b, int k, int r, uint32_t& nl, uint32_t& dd) {
          nl = m_nl[b - 2 * w_lo][r][k];
          dd = m_dd[b - 2 * w_lo][r][k];
        });
        if (lane == 0) {
          ctl[0] = end;
          ctl[1] = st.q;
          ctl[2] = st.j;
          ctl[3] = st.hi;
        }
      }
      __syncthreads();
      end = uni(ctl[0]);
      st.q = uni(ctl[1]);
      st.j = uni(ctl[2]);
      st.hi = uni(ctl[3]);
    }
    if (s > 0) load_rows(s - 1);
    if (end == kWalkBad) {   // empty runs from here up
      bad = true;
      if (tid == 0) atomicOr(a.status, kStatusBadPath);
      for (int i = i0 + tid; i <= iend; i += kWave * kTraceWaves) runs[i] = make_int2(0, -1);
    }
    jx = st.j;   // -1 above the first row
  }
}

template <typename TY, typename TC, int D, int RHO>
hipError_t launch_trace_t(const TraceArgs& a, int n_pairs, hipStream_t st) {
  hipLaunchKernelGGL((trace_kernel<TY, TC, D, RHO>), dim3(n_pairs), dim3(kWave * kTraceWaves), 0, st, a);
  return hipGetLastError();
}

template <typename TC, int D, int RHO>
hipError_t launch_trace_d(int ydtype, const TraceArgs& a, int n_pairs, hipStream_t st) {
  if (ydtype == 0) return launch_trace_t<float, TC, D, RHO>(a, n_pairs, st);
  if constexpr (sizeof(TC) == 8) return launch_trace_t<double, TC, D, RHO>(a, n_pairs, st);
  return hipErrorInvalidValue;
}

template <typename TC>
hipError_t launch_trace_impl(int d, int rho, int ydtype, const TraceArgs& a, int n_pairs,
                             hipStream_t st) {
#define CALLT(D, R) launch_trace_d<TC, D, R>(ydtype, a, n_pairs, st)
  if (rho == 4) { WTS_D_SWITCH(d, 4, CALLT) }
  if (rho == 2) { WTS_D_SWITCH(d, 2, CALLT) }
  if (rho == 5) { WTS_D_SWITCH(d, 5, CALLT) }
#undef CALLT
  return hipErrorInvalidValue;
}

}  // namespace

}  // namespace wts
