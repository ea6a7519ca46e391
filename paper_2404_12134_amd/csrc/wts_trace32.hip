// wts_trace32.hip -- the float32-decision instances of the path recovery from
// checkpoints (wts_trace.h), a translation unit of its own so that the two
// sets compile in parallel.
#include "wts_trace.h"

namespace wts {

hipError_t launch_trace32(int d, int rho, int ydtype, const TraceArgs& a, int n_pairs,
                          hipStream_t st) {
  return launch_trace_impl<float>(d, rho, ydtype, a, n_pairs, st);
}

}  // namespace wts
