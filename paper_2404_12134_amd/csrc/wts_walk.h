// wts_walk.h -- the path walk shared by both path recoveries.
//
// Argmin codes come as two bit planes, D (diagonal chosen) and U (up not
// above left), in words of 32 sweep steps per row, the first step in the top
// bit: higher bits are columns further left.  The walk takes 64 rows at a
// time, a lane per row.  Each lane cuts the 64 columns left of the walk's
// column out of its row's words, so bit b of every lane is the same column,
// and the rows are then followed on the scalar unit: a run to the left ends
// at the first set "not left" bit, one shift and one find-first-bit however
// long it is.  About a dozen scalar instructions a row and one rarely taken
// branch, where a step by step walk took 60 instructions and six branches a
// cell (85 us a strip of 320 rows).
#pragma once
#include "wts_device.h"

namespace wts {

namespace {

typedef unsigned long long u64_t;

__device__ __forceinline__ u64_t readlane64(u64_t v, int lane) {
  const uint32_t lo = (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)v, lane);
  const uint32_t hi = (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)(v >> 32), lane);
  return ((u64_t)hi << 32) | lo;
}

// Rows I .. 63 of a window (lane I's row after lane I-1's): sh is the walk's
// column as a bit of the window, rec[lane I] receives the bit where the path
// leaves row I upwards.  Returns the first row that the window does not
// finish (its "not left" bits from sh on are all zero), or 64.
template <int I>
__device__ __forceinline__ int walk_rows(u64_t nl, u64_t dd, int& sh, int& rec) {
  if constexpr (I < kWave) {
    const u64_t x = readlane64(nl, I) >> sh;
    if (x == 0) return I;
    sh += (int)__builtin_ctzll(x);
    __asm__("v_writelane_b32 %0, %1, %2" : "+v"(rec) : "s"(sh), "n"(I));
    sh += (int)(readlane64(dd, I) >> sh) & 1;
    return walk_rows<I + 1>(nl, dd, sh, rec);
  } else {
    return kWave;
  }
}

// A walk in progress (wave-uniform).
struct Walk {
  int q, j;      // row of the strip and column the walk is at
  int hi;        // the column where the path entered row q
  int jtop;      // the column where the path left the last finished row
};
enum WalkEnd { kWalkDone = 0, kWalkMore = 1, kWalkBad = 2 };
constexpr int kWalkNarrow = 24;   // columns of a window below which more tiles are asked for

// Follows the path upwards from `st` to the strip's first row and writes the
// columns [lo, hi] of every row's run.  word(b, k, r, nl, dd) gives lane k's
// code words of its row r for steps 32 b .. 32 b + 31 (the cell at column j
// is step j + k), which exist for steps >= step0.  Done: st.j = st.hi is the
// column where the path enters the strip above.  More: words to the left of
// step0 > 0 are needed; call again with them.
template <int RHO, typename Word>
__device__ __forceinline__ WalkEnd walk_strip(Walk& st, int step0, int2* runs, Word word) {
  const int lane = threadIdx.x % kWave;
  int q = st.q, j = st.j, hi = st.hi;
  WalkEnd end = kWalkDone;
  while (q >= 0) {
    if (j < 0) {
      end = kWalkBad;
      break;
    }
    const int rows = min(q + 1, kWave);
    const int nb = min(63, j + (q - rows + 1) / RHO - step0 + 1);   // columns every row has
    if (step0 > 0 && nb < kWalkNarrow) {
      end = kWalkMore;
      break;
    }
    const int ql = max(q - lane, 0);
    const int k = ql / RHO, r = ql - k * RHO;
    const int t = j + k;
    const int b0 = t >> 5, s = 31 - (t & 31);
    uint32_t wn[3], wd[3];
#pragma unroll
    for (int i = 0; i < 3; ++i) {
      wn[i] = wd[i] = 0u;
      if (32 * (b0 - i) >= step0) word(b0 - i, k, r, wn[i], wd[i]);
    }
    u64_t nl = ((u64_t)__builtin_amdgcn_alignbit(wn[2], wn[1], s) << 32) |
               __builtin_amdgcn_alignbit(wn[1], wn[0], s);
    const u64_t dd = ((u64_t)__builtin_amdgcn_alignbit(wd[2], wd[1], s) << 32) |
                     __builtin_amdgcn_alignbit(wd[1], wd[0], s);
    nl = lane < rows ? nl & ((1ull << nb) - 1) : 0ull;
    int sh = 0, rec = 0;
    const int done = min(walk_rows<0>(nl, dd, sh, rec), rows);
    const int lo = j - rec;
    const int next = lo - ((int)(dd >> rec) & 1);
    const int entry = __shfl_up(next, 1);
    if (lane < done) runs[q - lane] = make_int2(lo, lane == 0 ? hi : entry);
    if (done > 0) {
      st.jtop = __builtin_amdgcn_readlane(lo, done - 1);
      hi = j - sh;
    }
    q -= done;
    j -= done == rows ? sh : nb;   // a row the window did not finish goes on at its left edge
  }
  st.q = q;
  st.j = j;
  st.hi = hi;
  return end;
}

}  // namespace

}  // namespace wts
