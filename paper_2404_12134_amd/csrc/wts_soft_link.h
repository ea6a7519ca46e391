// wts_soft_link.h -- what the two forms of the Soft-DTW backward share, a workgroup
// to a strip (wts_soft_bwd.hip) and one wave to a strip (wts_soft_wave.hip): a
// replayed cell, and the exchange between the strips of a pair.  A strip of one
// form may follow a strip of the other.
//
// The pushes of a strip's top row travel to the strip above through one row of
// the pair: the strip below wrote it for us, we overwrite it for the strip above
// after reading.
#pragma once
#include "wts_soft.h"

namespace wts {

namespace {

// One cell of the replay: its cumulative cost and the normalised soft-min
// weights of its up and left predecessors.  Outside the band: cost +inf and
// weights (1, 0, 0), so the cell receives and passes on exactly nothing.
template <int D, bool BAND>
__device__ __forceinline__ double replay_cell(double dg, double up, double lf, const double (&x)[D],
                                              double xx, const double (&y)[D], double yy, bool inb,
                                              float& wu, float& wl) {
  if constexpr (BAND) {
    const SoftMin sm = softmin3_band(dg, up, lf, inb);
    const double rv = inb ? sq_cost<D>(x, xx, y, yy) + sm.v : inf_d();
    const float rs = __builtin_amdgcn_rcpf(inb ? sm.s : 1.0f);
    wu = inb ? sm.eu * rs : 0.0f;
    wl = inb ? sm.el * rs : 0.0f;
    return rv;
  } else {
    const SoftMin sm = softmin3(dg, up, lf);
    const double rv = sq_cost<D>(x, xx, y, yy) + sm.v;
    const float rs = __builtin_amdgcn_rcpf(sm.s);   // s >= 1: the minimum's term is 1
    wu = sm.eu * rs;
    wl = sm.el * rs;
    return rv;
  }
}

// A strip's words for the strip above (zeroed before the launch): columns
// published, counted from the right; the tile of its first non-zero push, plus
// one (-1: all its pushes are zero); the first column of its last published
// tile.  Pushes outside [end, 16 start + 15] are zero and are not written, so
// a strip waits on one word for the place where its input begins, however
// many zero tiles lie to the right of it.
struct BwdWords {
  int* prog;
  int* start;
  int* end;
};

// One strip's side of the exchange: used by one wave, every member uniform.
struct BwdLink {
  int lane, N, G, S, g_lo;
  bool has_above, has_below;     // a strip above consumes our pushes; one below feeds us
  int zero_skip;
  int quick, relaxed;            // polls without a sleep, and poll_backoff's kind of sleep
  int* status;
  BwdWords self, below;
  __amdgpu_buffer_rsrc_t pu_io, pd_io;
  bool gave_up = false;
  int seen_below = 0;            // last progress read from the strip below
  int in_hi = -1, in_lo = 0;     // columns of its pushes that may be non-zero
  bool in_known;                 // in_hi is known; without a strip below, no input
  bool in_done = false;          // ... and in_lo is
  bool started = false;          // this strip's start word is out
  int g_pub = 0;                 // last tile whose pushes were stored

  __device__ __forceinline__ BwdLink(const SoftArgs& a, const PairDesc& pd, int s, int g_lo_,
                                     int quick_, int relaxed_)
      : lane(threadIdx.x % kWave), N(pd.N), G(pd.WT), S(pd.S), g_lo(g_lo_), has_above(s > 0),
        has_below(s + 1 < pd.S), zero_skip(a.zero_skip), quick(quick_), relaxed(relaxed_),
        status(a.status), in_known(s + 1 == pd.S) {
    int* w = a.progress + pd.flag_base + s;
    self = BwdWords{w, w + a.n_flags, w + 2 * a.n_flags};
    below = BwdWords{w + 1, w + a.n_flags + 1, w + 2 * a.n_flags + 1};
    pu_io = rsrc(a.push_up + pd.bnd_base, N * 4);
    pd_io = rsrc(a.push_dg + pd.bnd_base, N * 4);
  }

  // waits until *word satisfies ok, and returns it; 0 after a timeout
  template <typename Ok>
  __device__ __forceinline__ int wait_word(const int* word, int limit, Ok ok) {
    int got = 0, quit = 0;
    if (lane == 0) {
      int polls = 0;
      got = ld_dev(word);
      while (!ok(got)) {
        if (polls > quick) poll_backoff(polls, relaxed);
        if (++polls > limit) {
          atomicOr(status, kStatusSpinTimeout);
          quit = 1;
          break;
        }
        got = ld_dev(word);
      }
    }
    gave_up = __builtin_amdgcn_readfirstlane(quit) != 0;
    const int r = __builtin_amdgcn_readfirstlane(got);
    __atomic_signal_fence(__ATOMIC_SEQ_CST);
    return r;
  }
  // The place where the input begins.  The strips below may sweep or pass over
  // every tile of the pair before they push anything up (their tiles until
  // then cover each column once, and five more a strip), a microsecond or two
  // a tile, about a poll: two seconds for 2^24 columns.
  __device__ __forceinline__ void learn_start() {
    if (in_known || gave_up) return;
    const int w = wait_word(below.start, kSpinLimit + 32 * (G + 16 * S), [](int v) { return v != 0; });
    in_known = true;
    in_hi = w > 0 ? min(16 * (w - 1) + kTile - 1, N - 1) : -1;
    if (w <= 0) { in_done = true; seen_below = N; }   // no input at all
  }
  __device__ __forceinline__ void learn_end() {
    if (in_done || seen_below < N) return;
    in_done = true;
    int e = 0;
    if (lane == 0) e = ld_dev(below.end);
    in_lo = __builtin_amdgcn_readfirstlane(e);
  }
  // waits until the strip below has published every column >= jlo
  __device__ __forceinline__ void wait_below(int jlo) {
    const int need = N - max(0, jlo);
    if (need > seen_below && !gave_up)
      seen_below = wait_word(below.prog, kSpinLimit, [&](int v) { return v >= need; });
    learn_end();
  }
  // the pushes into column c, a column a lane
  __device__ __forceinline__ void load_in(int c, bool want, float& u, float& v) {
    const int off = want && c >= max(in_lo, 0) && c <= in_hi ? c * 4 : kDrop;
    u = ld_dev_f32(pu_io, off);
    v = ld_dev_f32(pd_io, off);
  }
  // tiles gz .. g hold only zeros: published as such if earlier ones were
  __device__ __forceinline__ void publish_zeros(int gz, int g) {
    if (!has_above || !started || gz > g) return;
    for (int c = 16 * gz + lane; c < min(16 * g + kTile, N); c += kWave) {
      st_dev(pu_io, c * 4, 0.0f);
      st_dev(pd_io, c * 4, 0.0f);
    }
    mem_drain();
    g_pub = gz;
    if (lane == 0) st_dev(self.prog, N - min(N, 16 * gz));
  }
  // The next tile at or left of g that a push enters, with none travelling
  // inside the strip; -1: there is none.  e reaches a cell only through the
  // pushes of its successors, so every tile passed over has e = 0 in all its
  // cells and pushes nothing on: skipping it leaves every bit of the sums
  // as it is (a swept zero tile adds +0 and pushes 0 * w = 0).
  __device__ __forceinline__ int search(int g) {
    if (!has_below) return -1;
    learn_start();
    if (gave_up) return -1;
    g = min(g, (in_hi + kWave - 1) >> 4);
    while (g >= g_lo) {
      wait_below(16 * g - (kWave - 1));
      if (gave_up || (in_done && 16 * g - (kWave - kTile) < in_lo) || in_hi < 0) return -1;
      // tiles g .. ge: as far as the strip below has published, up to 16
      int ge = max(g_lo, g - 15);
      if (seen_below < N) ge = max(ge, (N - seen_below + (kWave - 1) + 15) >> 4);
      const int jlo = 16 * ge - (kWave - 1);
      const int cnt = 16 * (g - ge + 1);
      int hit = -1;
      float u[4], v[4];
#pragma unroll
      for (int q = 0; q < 4; ++q) load_in(jlo + lane + kWave * q, lane + kWave * q < cnt, u[q], v[q]);
#pragma unroll
      for (int q = 3; q >= 0; --q) {
        const unsigned long long m = __builtin_amdgcn_ballot_w64(u[q] != 0.0f || v[q] != 0.0f);
        if (hit < 0 && m != 0) hit = ge + ((kWave * q + 63 - __builtin_clzll(m)) >> 4);
      }
      publish_zeros(hit >= 0 ? hit + 1 : ge, g);
      if (hit >= 0) return hit;
      g = ge - 1;
    }
    return -1;
  }
  // The top row's pushes of tile g, column 16 g + lane in lanes 0..15 (two
  // stores, issued by every lane, dropped past the row), then the announcement
  // of the previous tile's columns: waiting until at most these two stores are
  // outstanding completes every older one.
  __device__ __forceinline__ void publish(int g, float up, float dg) {
    if (!has_above) return;
    const int j = 16 * g + lane;
    const bool w = lane < kTile && j < N;
    if (!started) {
      const bool nz = __builtin_amdgcn_ballot_w64(w && (up != 0.0f || dg != 0.0f)) != 0;
      started = nz || !zero_skip;
      if (started && lane == 0) st_dev(self.start, g + 1);
    }
    if (started) {
      st_dev(pu_io, w ? j * 4 : kDrop, up);
      st_dev(pd_io, w ? j * 4 : kDrop, dg);
      mem_wait_all_but_2();
      g_pub = g;
      if (lane == 0) st_dev(self.prog, N - min(N, 16 * g + kTile));
    }
  }
  // the last tile's columns; every one left of them is zero
  __device__ __forceinline__ void finish() {
    if (!has_above) return;
    if (lane == 0) {
      if (started) st_dev(self.end, 16 * g_pub);
      else st_dev(self.start, -1);
    }
    mem_drain();
    if (lane == 0) st_dev(self.prog, N);
  }
};

}  // namespace

}  // namespace wts
