// wts_team2.hip -- the float64 team sweeps (wts_team.h) of two rows a lane.
#include "wts_team.h"

namespace wts {

hipError_t launch_team(int d, int rho, int mode, bool euc, bool x_is_cycle, int ydtype, bool fp32,
                       const FwdArgs& a, int groups, hipStream_t st) {
  if (rho != 2 && rho != 4) return hipErrorInvalidValue;
  if (fp32) return launch_team32(d, rho, mode, euc, x_is_cycle, ydtype, a, groups, st);
  if (rho == 4) return launch_team4(d, mode, euc, x_is_cycle, ydtype, a, groups, st);
  return launch_team_impl<double, 2>(d, mode, euc, x_is_cycle, ydtype, a, groups, st);
}

}  // namespace wts
