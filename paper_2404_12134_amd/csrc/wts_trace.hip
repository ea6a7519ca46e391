// wts_trace.hip -- the float64 instances of the path recovery from
// checkpoints (wts_trace.h).
#include "wts_trace.h"

namespace wts {

hipError_t launch_trace(int d, int rho, int ydtype, bool fp32, const TraceArgs& a, int n_pairs,
                        hipStream_t st) {
  if (n_pairs <= 0) return hipSuccess;
  if (fp32) return launch_trace32(d, rho, ydtype, a, n_pairs, st);
  return launch_trace_impl<double>(d, rho, ydtype, a, n_pairs, st);
}

}  // namespace wts
