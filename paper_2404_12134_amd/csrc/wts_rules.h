// wts_rules.h -- which kernels and how many rows a lane a plan's sweeps take
// (host code, built with the host compiler too by its test).
#pragma once

#include <algorithm>
#include <cmath>
#include <cstddef>
#include <cstdint>

namespace wts {
namespace rules {

constexpr int kLanes = 64;   // of a wave

constexpr size_t kAlign = 256;
inline size_t align_up(size_t v) { return (v + kAlign - 1) / kAlign * kAlign; }

// Scratch of wts_anomaly_score_noalloc.
constexpr size_t kScratchBytes = size_t(32) << 20;

// Strip row stride of the DTW sweeps (row_stride in wts_sweep.h).
inline int64_t row_stride_host(int32_t N) { return (N + kLanes - 1 + 3) & ~3; }

// Workspace of a score sweep with that many strip row elements (the layout of
// WTS_OP_SCORE).
inline size_t score_bytes(int64_t rows, int n) {
  return align_up(2 * sizeof(int)) + align_up(sizeof(double) * (size_t)rows) +
         align_up(sizeof(int) * (size_t)rows) + align_up(sizeof(double) * (size_t)n) +
         align_up(sizeof(int) * (size_t)n);
}

// Whether a set of `items` strips is swept by teams of four waves a strip
// (wts_team.h) or by one wave a strip.  Teams win while the strips leave
// compute units or SIMDs idle.  Score sweep / DBA iteration in us, team
// against one wave, float64, d = 3: 8 x 4.4k (L = 4000) 559 / 736 against
// 931 / 1136, 32 x 4.4k 761 / 903 against 957 / 1161; past five strips of two
// rows a lane per compute unit the two are even (48 x 4.4k: 961 / 1128 against
// 968 / 1168), and at seven the team loses (16 x 16k: 3941 / 4456 against
// 3599 / 4321).  Teams of four rows a lane hold 64 KB of LDS (float64), two a
// compute unit, and win up to that; in float32 they hold half of it.
inline bool team_pays(int rho, int64_t items, int cus, bool fp32) {
  if (rho == 2) return items <= 5 * (int64_t)cus;
  return rho == 4 && items <= (fp32 ? 4 : 2) * (int64_t)cus;
}

// What a set of strips asks of the one-wave DTW sweeps, in sweep steps.
struct SweepLoad {
  int64_t items = 0, pairs = 0;
  double steps = 0.0;        // of all strips
  double longest = 0.0;      // of a strip
  double shortest = 0.0;
  double chain = 0.0;        // of a pair's strips, each following the one above
  double strips = 0.0;       // of the pair with most
  void add(int64_t cols, int64_t n_strips) {
    const double one = (double)(cols + kLanes);
    items += n_strips;
    shortest = pairs == 0 ? one : std::min(shortest, one);
    ++pairs;
    steps += one * n_strips;
    longest = std::max(longest, one);
    chain = std::max(chain, one + 110.0 * (n_strips - 1));
    strips = std::max(strips, (double)n_strips);
  }
};

enum { kSweepValues = 0, kSweepScores, kSweepSub, kSweepPaths, kSweepKinds };

// Time of a one-wave sweep at `waves` to a SIMD, in steps of a lone wave, of
// which a step takes `q`: the longest chain, or the strips over the waves and the
// end of the last ones (the longer the more the pairs' lengths differ); where
// strips start later than others of their pair, those waiting below hold waves
// (float64).  A strip costs 120 steps of its own.
inline double sweep_time(const SweepLoad& l, int cus, int waves, double q, bool fp32) {
  const double slots = 4.0 * cus * waves;
  const double t = q * l.chain + 120.0;
  if (l.items <= slots) return t;
  const double work = (q * l.steps + 120.0 * l.items) / slots;
  const double mean = l.steps / l.items;
  const double tail = q * std::min(0.28 * l.longest, 1.5 * (l.longest - mean));
  const double deep = std::max(0.0, l.strips - slots / l.pairs);
  const double wait = waves > 1 && !fp32 ? q * std::min(200.0 * deep, 0.2 * l.longest) : 0.0;
  const double rounds = std::ceil(l.items / slots) * (q * (0.7 * l.shortest + 0.3 * mean) + 120.0);
  return std::max(std::max(t, work + tail + wait), rounds);
}

// Waves per SIMD of the one-wave DTW sweeps.  A second wave on a SIMD raises its
// throughput (a step of both takes q times a step of one) and slows the chain
// of every pair's strips by as much.  q, measured: 1.4 to 1.8 in float64 with the
// channels and rows (less for the lighter instruction mixes of Sub-DTW and of
// value sweeps), 1.05 to 1.1 in float32.  Over 1346 sweeps (45 shapes of 1.1 to 20
// strips a SIMD, of lengths that spread by two fifths and of equal ones, d = 1, 3, 6,
// 8, all kinds) the choice between one and more costs 0.30 % on average against the
// better of both, and 18 % at most.  Measured, us at 1 / 2 / 3: scores of 128 cycles of about 4k
// (d = 3) 1524 / 1743 / 1750, in float32 1407 / 1178 / 1170, of 1000 of 1000 (d = 1)
// 566 / 517 / 505; Sub-DTW of 256 of 4k (d = 1) 2684 / 2332 / 2197.
// A third gains 3 to 10 % where there are strips enough and the mix is light.
inline int sweep_waves(const SweepLoad& l, int kind, int cus, int d, int rho, bool fp32) {
  const double simds = 4.0 * cus;
  if (l.items <= simds) return 1;
  double q = kind == kSweepValues ? 1.23 + 0.06 * d : kind == kSweepSub ? 1.36 + 0.04 * d : 1.43 + 0.05 * d;
  q = std::min(1.03 * (rho == 5 ? q + 0.07 : q), 1.78);
  if (fp32) q = kind == kSweepValues || kind == kSweepSub ? 1.05 : 1.1;
  if (sweep_time(l, cus, 1, 1.0, fp32) <= sweep_time(l, cus, 2, q, fp32)) return 1;
  if (kind == kSweepValues && d <= 4) return 3;
  const bool light = fp32 ? kind != kSweepScores || l.items > 6 * simds : kind == kSweepSub && d <= 4;
  return light && l.items > 3 * simds && l.longest > 110.0 * l.strips ? 3 : 2;
}

// Path recovery.  Codes and entry tags for every cell (PATHT) cost the one-wave
// sweep 80 ns a step of 4 rows in float64 and 70 in float32, a fifth less
// above six strips a SIMD, and let all strips be walked at once.  From
// checkpoints (CKPT) the sweep is the value sweep, and each pair's strips are
// swept again along its path and walked in turn, 14 us and 6 us a channel a
// strip (0.7 of that in float32; above 256 pairs they share the compute units).
// DBA iteration, codes / checkpoints, us: 128 x 4k 1551 / 1143 (d = 1), 1801 / 1540 (d =
// 3), 1000 x 1000 720 / 657 and 871 / 1001, in float32 568 / 504 and 639 / 666; 512 of
// 1k-20k (L = 10,000, d = 6) 25.3 / 22.8 ms.  Over 114 batches the choice costs 0.4 %
// on average and 10 % at most.  A team's sweep costs less a strip than its walk:
// codes.
inline bool walk_pairs_pays(const SweepLoad& l, int cus, int d, int rho, bool fp32) {
  const double simds = 4.0 * cus;
  const double steps = std::max(l.chain, l.steps / simds);
  const double codes = (fp32 ? 70e-9 : 80e-9) * (l.items > 6 * simds ? 0.8 : 1.0) * rho / 4;
  const double trace = (14e-6 + 6e-6 * d) * (fp32 ? 0.7 : 1.0);
  return steps * codes > l.strips * trace * std::max(1.0, l.pairs / 256.0);
}

// The Soft-DTW forward: teams of four waves a strip (wts_soft_team.hip) or one
// wave a strip.  A team takes half the time a step and follows the strip above
// at half the distance; one wave a strip has fewer instructions a cell once
// the SIMDs are full.  Team against one wave, ms: 16 x 2k (256 strips, d = 3)
// 0.44 / 0.98, 5 x 18k 4.3 / 9.4, 25 x 18k (3600 strips) 10.0 / 14.9, 100 x 8k
// (6300 strips) 6.8 / 8.3 and at d = 6 8.7 / 9.1, 400 x 2k (6400) 1.77 / 2.01
// and at d = 6 2.27 / 2.23, 200 x 8k (12,600) 12.4 / 12.9 and at d = 6 16.3 /
// 14.6.
inline bool soft_team_pays(int64_t items, int cus) { return items <= 24 * (int64_t)cus; }

// The Soft-DTW backward: a workgroup a strip (wts_soft_bwd.hip) or one wave a
// strip (wts_soft_wave.hip).  A workgroup follows the strip below three to four
// times as closely, and the chain of a pair's strips bounds batches of few
// pairs or few live tiles (tiles with a non-zero e); one wave takes half the
// time a tile once the tiles fill the compute units.  Measured on 256 compute
// units, S strips a pair, n pairs, w live tiles a strip, in us:
//   workgroup  n S (w + 8) (4.7 + 0.23 d) / 1000, at least 12.5 S + 1.3 w
//   wave       S (72 + 3 d) + n S w (1.5 + 0.1 d) / 1000
// The result is the w from which the wave is faster: 31 at 512 pairs, 165 at
// 128, 10 at 1000.  w is 12 to 20 for a narrow E (a strip is 128 rows and
// 63 steps of skew) and grows with gamma, up to 20 (cycles of 300), 48 (2k) or
// 160 (20k) where every step is as likely: 1000 x 2k (d = 3) at 17 / 48 live tiles
// 1.94 / 4.40 ms by workgroups, 1.71 / 2.59 by waves; 512 x 2k 1.02 / 2.26
// against 1.52 / 1.96; 128 x 20k (d = 6) at 24 / 157 4.6 / 19.6 against 15.4 / 19.0.
inline int bwd_wave_tiles(int64_t items, int strips, int cus, int d) {
  const double n = (double)items / std::max(1, strips) * 256.0 / cus;
  const double a = 4.7 + 0.23 * d, b = 1.5 + 0.1 * d, c = 1000.0 * (72.0 + 3.0 * d);
  return (int)std::min(1e9, std::max(0.0, (c / std::max(n, 1e-3) - 8.0 * a) / (a - b)));
}

// Live tiles a strip can have, about, of a pair of that many rows and columns: its
// 128 rows' columns and the spread where every step is as likely (20 at 300 x
// 300, 48 at 2k x 2k, 160 at 20k x 20k).
inline double bwd_live_most(double rows, double cols) {
  return 8.0 * cols / std::max(1.0, rows) + std::sqrt(cols);
}

// Rows per lane of the barycenter sweeps when the caller leaves it open.
// Batches of few strips take 2 and are swept by teams (in float32 above four
// such strips a compute unit, teams of 4: 16 x 16k, d = 3, score / DBA 2526 /
// 2973 us against 2746 / 3431).  Others take 4, with one wave to a SIMD and
// one workgroup to a compute unit up to 1024 strips.  Float64 batches of two
// channels or more and of more than four strips a SIMD take 5 where the
// padding of the last strip allows it: a step costs about 2 d + 4
// instructions a row and 10 of its own, which 5 rows share (40 cycles of
// 40k-50k samples, d = 6, score / checkpointed sweep: 74.3 / 61.2 ms against
// 77.7 / 64.8; 25 of 30k: 22.9 / 19.2 against 20.6 / 18.2).  In float32 the
// score sweep is no faster at 5.  Up to four strips a SIMD the longest pair's
// chain (120 steps a strip) or the rounds of strips on the SIMDs decide, at
// about 2 d + 8 instructions a row and 38 a step: 5 rows a lane win where they
// save a strip or a round (500 cycles of 300, L = 300, one strip instead of
// two: 72 against 85 us; 512 of 320, L = 320, d = 6: 133 against 144).
inline int bary_rho(int64_t L, int n, int64_t nmax, int cus, int d, bool fp32, bool team) {
  auto strips = [&](int r) { return (L + 64 * r - 1) / (64 * r); };
  auto items = [&](int r) { return (int64_t)n * strips(r); };
  const int64_t simds = 4 * (int64_t)cus;
  if (team && fp32 && items(2) > simds && team_pays(4, items(4), cus, fp32)) return 4;
  if (team && team_pays(2, items(2), cus, fp32)) return 2;
  auto steps = [&](int r) { return strips(r) * (r * (2 * d + 4) + 10); };
  if (items(4) > 4 * simds) return d >= 2 && !fp32 && steps(5) < steps(4) ? 5 : 4;
  auto chain = [&](int r) {
    const int64_t rounds = (items(r) + simds - 1) / simds, one = nmax + kLanes;
    return std::max(one + 120 * strips(r), rounds * one) * (r * (2 * d + 8) + 38);
  };
  return chain(5) < chain(4) ? 5 : 4;
}

// Rows per lane of wts_anomaly_score_noalloc where the plan's own (rho) need more
// workspace than its scratch holds and fewer strip rows (more rows a lane) fit it:
// those of the one-wave sweeps, or 5 where that brings more strips than 13/16 of
// the SIMDs, and at most two a SIMD, under 13/16.  That was once the rule for 5
// rows, and a batch that fitted by it (14 cycles of 3000, L = 17,560: 28 MB
// against 35 at 4) still does.  0: the plan's own rows.  off: n + 1 offsets.
inline int scratch_rho(int rho, const int64_t* off, int n, int64_t L, int cus, int d, bool fp32) {
  int64_t nmax = 0;
  for (int k = 0; k < n; ++k) nmax = std::max(nmax, off[k + 1] - off[k]);
  auto strips = [&](int r) { return (L + kLanes * r - 1) / (kLanes * r); };
  auto fits = [&](int r) {
    int64_t rows = 0;
    for (int k = 0; k < n; ++k) rows += strips(r) * row_stride_host((int32_t)(off[k + 1] - off[k]));
    return score_bytes(rows, n) <= kScratchBytes;
  };
  if (fits(rho)) return 0;
  const int alt = bary_rho(L, n, nmax, cus, d, fp32, false);
  if (alt != rho && fits(alt)) return alt;
  const int64_t simds = 4 * (int64_t)cus, cap = simds * 13 / 16;
  const int64_t i4 = n * strips(4);
  return i4 > cap && i4 <= 2 * simds && n * strips(5) <= cap && fits(5) ? 5 : 0;
}

}  // namespace rules
}  // namespace wts
