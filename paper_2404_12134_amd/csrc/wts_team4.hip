// wts_team4.hip -- the float64 team sweeps (wts_team.h) of four rows a lane.
#include "wts_team.h"

namespace wts {

hipError_t launch_team4(int d, int mode, bool euc, bool x_is_cycle, int ydtype, const FwdArgs& a,
                        int groups, hipStream_t st) {
  return launch_team_impl<double, 4>(d, mode, euc, x_is_cycle, ydtype, a, groups, st);
}

}  // namespace wts
