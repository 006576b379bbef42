// Forms of the iterations' binning beside the plain one (dst_runs.h).
#pragma once

#include <hip/hip_runtime.h>

#include <cstdint>

#include "dst_group.h"
#include "dst_internal.h"
#include "dst_runs.h"

namespace dst {

enum { BIN_PLAIN = 0, BIN_LDS = 1, BIN_PIPE = 2 };

// Form, lanes per pixel and workgroups (BIN_PLAIN: launch_bin_runs).
struct BinShape {
  int form = BIN_PLAIN;
  int lpp = 0;
  uint32_t blocks = 0;
};
// mode: a form (BIN_LDS wherever the baselines fit and BIN_PIPE wherever there are
// q/u streams, else plain; radiometers: plain), or -1: the fastest for the
// problem's sizes.
BinShape bin_shape(const View& vc, const Runs& W, int mode);
// Lanes per pixel for `runs` runs over n_obs pixels (a lane takes four runs
// per step, eight without angles); whether that is sparse enough for BIN_PIPE;
// its workgroups.
int bin_form_lanes(int64_t runs, int64_t n_obs, bool t_only);
bool bin_sparse(int64_t runs, int64_t n_obs, bool angles);
uint32_t bin_pipe_blocks(int64_t n_obs, int lpp);
// part [blocks + 1] (BIN_LDS only)
hipError_t bin_build(const View& vc, const Runs& W, const BinShape& s, uint32_t* part, BinRuns* out, hipStream_t st);
// m = M^-1 A^T W F p as launch_bin_runs.
hipError_t launch_bin_form(const View& vc, const BinRuns& B, const BinShape& s, bool f32, const double* pw4,
                           const double* Minv4, const uint8_t* valid, double* m4, const CgCtl* gate, hipStream_t st);
// The binning launch of a group's kind in its slice's form.
hipError_t launch_group_bin_form(const GroupLaunch& G, int kind, hipStream_t st);

}  // namespace dst
