// Rows per lane and score workspace of barycenter plans (wts_rules.h), read from
// stdin: d L fp32 team cus n, then n cycle lengths -> "rho bytes2 bytes4 bytes5"
// (rho: of the non-allocating score call), then the waves a SIMD of the one-wave
// sweeps at 4 rows (values, scores, Sub-DTW, paths) and whether paths are
// recovered from checkpoints.
#include <cstdio>
#include <vector>

#include "wts_rules.h"

int main() {
  using namespace wts::rules;
  int d, fp32, team, cus, n;
  long long L, len;
  while (std::scanf("%d %lld %d %d %d %d", &d, &L, &fp32, &team, &cus, &n) == 6) {
    std::vector<int64_t> off(1, 0);
    for (int k = 0; k < n; ++k) {
      if (std::scanf("%lld", &len) != 1) return 2;
      off.push_back(off.back() + len);
    }
    int64_t nmax = 0;
    for (int k = 0; k < n; ++k) nmax = std::max(nmax, off[k + 1] - off[k]);
    const int rho = bary_rho(L, n, nmax, cus, d, fp32 != 0, team != 0);
    const int less = scratch_rho(rho, off.data(), n, L, cus, d, fp32 != 0);
    std::printf("%d", less ? less : rho);
    for (int r : {2, 4, 5}) {
      int64_t rows = 0;
      for (int k = 0; k < n; ++k)
        rows += (L + kLanes * r - 1) / (kLanes * r) * row_stride_host((int32_t)(off[k + 1] - off[k]));
      std::printf(" %zu", score_bytes(rows, n));
    }
    SweepLoad load;
    for (int k = 0; k < n; ++k) load.add(off[k + 1] - off[k], (L + 4 * kLanes - 1) / (4 * kLanes));
    for (int kind = 0; kind < kSweepKinds; ++kind)
      std::printf(" %d", sweep_waves(load, kind, cus, d, 4, fp32 != 0));
    std::printf(" %d\n", (int)walk_pairs_pays(load, cus, d, 4, fp32 != 0));
  }
  return 0;
}
