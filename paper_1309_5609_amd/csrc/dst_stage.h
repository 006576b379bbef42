// The rescan with its map values staged through LDS (dst_stage.hip).
#pragma once

#include <hip/hip_runtime.h>

#include <cstdint>

#include "dst_group.h"
#include "dst_internal.h"
#include "dst_runs.h"

namespace dst {

// Whether the problem can be staged (all but radiometers), and whether that is worth its setup.
inline bool stage_can(const View& vc, const Runs& W) { return !vc.iqu && W.n_obs > 0; }
bool stage_pays(const View& vc, const Runs& W);
int64_t stage_blocks(const View& vc);
int64_t stage_cap(const View& vc);
hipError_t stage_build(const View& vc, const Runs& W, const Stage& S, hipStream_t st);

// As launch_unbin_runs, with staged_parts(vc) partials of each kind.
int64_t staged_parts(const View& vc);
hipError_t launch_unbin_staged(const View& vc, const Runs& W, const Stage& S, const double* m4, const int32_t* nvalid,
                               const double* p, double* q, CgCtl* ctl, double* partials, hipStream_t st);

// The rescan of a group's kind whose problems are all staged.
hipError_t launch_group_unbin_staged(const GroupLaunch& G, int kind, hipStream_t st);

}  // namespace dst
