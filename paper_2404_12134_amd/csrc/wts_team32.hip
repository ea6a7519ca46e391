// wts_team32.hip -- the float32-decision team sweeps (wts_team.h).
#include "wts_team.h"

namespace wts {

hipError_t launch_team32(int d, int rho, int mode, bool euc, bool x_is_cycle, int ydtype,
                         const FwdArgs& a, int groups, hipStream_t st) {
  if (rho == 4) return launch_team_impl<float, 4>(d, mode, euc, x_is_cycle, ydtype, a, groups, st);
  return launch_team_impl<float, 2>(d, mode, euc, x_is_cycle, ydtype, a, groups, st);
}

}  // namespace wts
