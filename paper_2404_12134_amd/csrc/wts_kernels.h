// wts_kernels.h -- host-side launchers of the WETSAND kernels.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "wts_device.h"

namespace wts {

struct WalkArgs {           // path recovery by strips (after a PATHT sweep)
  const PairDesc* pairs;
  const int2* items;
  const int2* seg;          // per item: (bottom-row column, top-row column) of the path
  int2* runs;               // [out][L]: the columns [lo, hi] of each row's path run
  const uint32_t* codes;
  int64_t L;
  int* status;              // device status word
  const int* skip;          // validation flag of the call (or null)
};

struct TraceArgs {          // path recovery from checkpoints (after a CKPT sweep)
  const PairDesc* pairs;
  const void* x;            // barycenter rows (float64)
  const void* y;            // cycle values
  const double* states;     // the sweep's checkpoints (see FwdArgs)
  const double* bnd_r;      // the sweep's strip rows
  int2* runs;               // [out][L]: the columns [lo, hi] of each row's path run
  int64_t L;
  int* status;
  const int* skip;
};

// fp32: the float32-decision instances (float32 cycles, squared cost only).
hipError_t launch_fwd(int d, int rho, int mode, bool euc, bool x_is_cycle, int ydtype, bool fp32,
                      const FwdArgs& a, int grid, hipStream_t st);
hipError_t launch_fwd32(int d, int rho, int mode, bool euc, bool x_is_cycle, int ydtype,
                        const FwdArgs& a, int grid, hipStream_t st);
// The team sweeps (four waves a strip, rho 2 or 4); groups: workgroups.
hipError_t launch_team(int d, int rho, int mode, bool euc, bool x_is_cycle, int ydtype, bool fp32,
                       const FwdArgs& a, int groups, hipStream_t st);
hipError_t launch_team4(int d, int mode, bool euc, bool x_is_cycle, int ydtype, const FwdArgs& a,
                        int groups, hipStream_t st);
hipError_t launch_team32(int d, int rho, int mode, bool euc, bool x_is_cycle, int ydtype,
                         const FwdArgs& a, int groups, hipStream_t st);
// Path recovery after a PATHT sweep: the strip chain (segments from the
// entry tags), then walks of all strips at once (row runs).
hipError_t launch_walk(int rho, const WalkArgs& a, int n_items, hipStream_t st);
hipError_t launch_chain(const PairDesc* pairs, int n_pairs, const int* bnd_aux,
                        const int* out_aux, int2* seg, int* status, const int* skip,
                        hipStream_t st);
// Path recovery after a CKPT sweep: one workgroup per pair (row runs).
hipError_t launch_trace(int d, int rho, int ydtype, bool fp32, const TraceArgs& a, int n_pairs,
                        hipStream_t st);
hipError_t launch_trace32(int d, int rho, int ydtype, const TraceArgs& a, int n_pairs,
                          hipStream_t st);
// The DBA update from the row runs: sums, counts and means.
hipError_t launch_run_fold(int d, int ydtype, const int2* runs, const int64_t* off, const void* y,
                           const double* w, int n, int64_t L, double* bout, int64_t* counts,
                           const int* skip, hipStream_t st);
// The path lists and their lengths from the row runs.
hipError_t launch_emit(const int2* runs, const int64_t* path_base, int n, int64_t L,
                       int32_t* paths, int64_t* path_len, const int* skip, hipStream_t st);
hipError_t launch_zero(int* p, int64_t n, hipStream_t st);
hipError_t launch_fill_sentinels(double* r, int64_t nr, int* x, int64_t nx, int* queue,
                                 hipStream_t st);
hipError_t launch_score(const double* dist, const int* len, int n, double* score,
                        int64_t* path_len, hipStream_t st);
hipError_t launch_sub_out(const int* start, const int* end, int n, int64_t* a_star,
                          int64_t* b_star, hipStream_t st);
hipError_t launch_medoid(const double* pair_dist, const int2* pair_ab, int n_pairs, int n,
                         double* Dm, double* totals, int32_t* medoid, hipStream_t st);
// Soft-DTW: the forward by one wave a strip (grid: waves) or by teams of four
// (groups: workgroups; rows filled with sentinels), the backward.
hipError_t launch_soft_fwd(int d, int ydtype, const SoftArgs& a, int grid, hipStream_t st);
hipError_t launch_soft_team(int d, int ydtype, const SoftArgs& a, int groups, hipStream_t st);
hipError_t launch_soft_bwd(int d, int ydtype, const SoftArgs& a, int groups, hipStream_t st);
hipError_t launch_soft_bwd_wave(int d, int ydtype, const SoftArgs& a, int grid, hipStream_t st);
hipError_t launch_soft_rows_scale(const double* g, const int64_t* off, int n, int64_t rows, int d,
                                  const double* w, double* out, hipStream_t st);
hipError_t launch_soft_reduce(const double* gsum, const double* hsum, const double* w, int n,
                              int64_t L, int d, double* grad, double* mass, int accumulate,
                              hipStream_t st);

// wts_aux.hip: input validation, the status word, the Eq. 7 objective.
struct ScanSeg {
  const void* p;   // values to check (or null)
  int64_t n;       // number of values
  int f32;         // 1: float32, 0: float64
};
hipError_t launch_finite_scan(const ScanSeg* segs, int nseg, int* flag, int* status,
                              hipStream_t st);
hipError_t launch_status_take(int* status, int* out, hipStream_t st);
hipError_t launch_objective(const double* values, const double* weights, int n, int accumulate,
                            double* out, hipStream_t st);
hipError_t launch_precond_step(double* bary, const double* grad, const double* mass, int64_t L,
                               int d, double eta, hipStream_t st);
hipError_t launch_init(int ydtype, const void* Y, const int64_t* off, int n, int d, int src,
                       int64_t Nsrc, int64_t L, int euclid, double* out, hipStream_t st);

}  // namespace wts
