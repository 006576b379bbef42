// Binning of the iterations with the baseline values in LDS.
#pragma once

#include <hip/hip_runtime.h>

#include <cstdint>

#include "dst_group.h"
#include "dst_internal.h"
#include "dst_runs.h"

namespace dst {

// Shape of the LDS form (blocks 0: not used): lanes per pixel, workgroups.
struct LdsShape {
  int lpp = 0;
  uint32_t blocks = 0;
};
// mode: 1 wherever the baselines fit, 0 never, -1 where it is the faster form.
LdsShape lds_shape(const View& vc, const Runs& W, int mode);
// Lanes per pixel for `runs` runs over n_obs pixels (a lane takes four runs
// per step, eight without angles).
int lds_lanes_for(int64_t runs, int64_t n_obs, bool t_only);
// part [blocks + 1]
hipError_t lds_build(const View& vc, const Runs& W, const LdsShape& s, uint32_t* part, LdsRuns* out, hipStream_t st);
// m = M^-1 A^T W F p as launch_bin_runs.
hipError_t launch_bin_lds(const View& vc, const LdsRuns& B, const LdsShape& s, bool f32, const double* pw4,
                          const double* Minv4, const uint8_t* valid, double* m4, const CgCtl* gate, hipStream_t st);
// The binning launch of a group's kind whose problems all have the LDS form.
hipError_t launch_group_bin_lds(const GroupLaunch& G, int kind, hipStream_t st);

}  // namespace dst
