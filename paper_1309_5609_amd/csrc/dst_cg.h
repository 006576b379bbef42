// Bodies of the PCG vector steps (the solver paragraph closing the Algorithm
// section of arXiv:1309.5609, applied to Eq. 13), shared by the single
// solve's kernels and by the kernels that advance several independent
// problems in one launch.  A body takes the workgroup's position in its own
// problem's grid (vblock of vgrid) instead of blockIdx / gridDim.
#pragma once

#include <hip/hip_runtime.h>

#include <cstdint>

#include "dst_comp.h"
#include "dst_device.h"
#include "dst_internal.h"

namespace dst {

// Workgroups of a grid that finish a reduction for themselves: every one of
// them reads all partials of the kernel before it, in the same order, so all
// hold the same bits and no single-workgroup kernel stands between.  No field of
// CgCtl is both read and written in such a launch, since a workgroup (or one
// wavefront of it, which would leave the others without its share of a sum) may
// start when workgroup 0 has written already: the update keeps rz, iter and the
// stop for the direction in rz_old, iter_old and stop, and only the direction
// sets rz, iter and done, which it does not read.
//
// Sums of N rows of n_part partials, valid in every thread, in one order
// whatever the workgroup's size: partial j belongs to slot j mod 1024, the 64
// slots of a slice are added by a butterfly and the slices in turn, so a
// solve's bits do not depend on which kernel finishes the sums.
// lds: 16 N doubles.
template <int N>
__device__ __forceinline__ void sum_rows(const double* __restrict__ partials, int64_t n_part, double (&tot)[N],
                                         double* lds) {
  constexpr int kSlots = 1024;
  const int n_slice = (int)((n_part < kSlots ? n_part + 63 : kSlots) / 64);
  for (int s = threadIdx.x >> 6; s < n_slice; s += blockDim.x >> 6) {
#pragma unroll
    for (int i = 0; i < N; ++i) tot[i] = 0.0;
    for (int64_t j = s * 64 + dev::lane_id(); j < n_part; j += kSlots) {
#pragma unroll
      for (int i = 0; i < N; ++i) tot[i] += partials[i * n_part + j];
    }
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) {
#pragma unroll
      for (int i = 0; i < N; ++i) tot[i] += __shfl_xor(tot[i], off, 64);
    }
    if (dev::lane_id() == 0) {
#pragma unroll
      for (int i = 0; i < N; ++i) lds[i * 16 + s] = tot[i];
    }
  }
  __syncthreads();
#pragma unroll
  for (int i = 0; i < N; ++i) tot[i] = 0.0;
  for (int s = 0; s < n_slice; ++s) {
#pragma unroll
    for (int i = 0; i < N; ++i) tot[i] = s == 0 ? lds[i * 16] : tot[i] + lds[i * 16 + s];
  }
  __syncthreads();
}

// Outcome of p.(P K p): DONE_RUNNING with a step, or why there is none.
__device__ __forceinline__ int step_outcome(double pkp) {
  return !isfinite(pkp) ? DONE_NAN : (pkp <= 0.0 ? DONE_BREAKDOWN : DONE_RUNNING);
}

// Step length from the rescan's partials (n_part of each kind: p.q, T sum of
// q, T sum of p): the null-space projection of q = K p (one component: the
// mean mu over T-valid baselines, applied by the residual update; several:
// each component's mean removed from q in place) and alpha = r.z / p.(P K p).
// One workgroup; fixed summation order.  lds: 48 doubles; clds: 16 * 64.
__device__ inline void cg_alpha_body(int64_t n_part, CgCtl* ctl, const double* partials, const CompView& cv,
                                     double* q, const double* p, double* lds, double* clds) {
  if (ctl->done) return;
  double tot[3];
  sum_rows<3>(partials, n_part, tot, lds);
  const int ncomp = cv.ncomp ? *cv.ncomp : 0;
  double corr = 0.0;
  if (ncomp > 1) corr = comp_project_block(cv, ncomp, q, p, 1, 1, clds);
  if (threadIdx.x == 0) {
    const double mu = ncomp > 1 ? 0.0 : (ctl->n_e > 0.0 ? tot[1] / ctl->n_e : 0.0);
    const double pkp = ncomp > 1 ? tot[0] - corr : tot[0] - mu * tot[2];
    const int done = step_outcome(pkp);
    ctl->mu = mu;
    if (done)
      ctl->done = done;
    else
      ctl->alpha = ctl->rz / pkp;
  }
}

// a += alpha p;  r -= alpha P q;  z = J r;  the workgroup's partials of r.z
// and r.r at partials[vblock] and partials[vgrid + vblock].  STEP: alpha and
// mu from the rescan's n_step partials of each kind (one component); else as
// cg_alpha_body left them.  The first element's values are loaded before the
// partials are summed.  lds: 48 doubles.
template <bool STEP>
__device__ inline void cg_update_body(const View& v, double* __restrict__ a, double* __restrict__ r,
                                      double* __restrict__ z, const double* __restrict__ p,
                                      const double* __restrict__ q, const double* __restrict__ J, CgCtl* ctl,
                                      const double* __restrict__ step, int64_t n_step, double* __restrict__ partials,
                                      int64_t vblock, int64_t vgrid, double* lds) {
  const bool first = vblock == 0 && threadIdx.x == 0;
  const int stopped = ctl->done;
  if (stopped) {
    if (first) ctl->stop = stopped;
    return;
  }
  const int64_t N = (int64_t)v.n_streams * v.n_b;
  int64_t i = vblock * blockDim.x + threadIdx.x;
  double ji = 0.0, qi = 0.0, pi = 0.0, ai = 0.0, ri = 0.0;
  auto load = [&]() {
    if (i < N) {
      ji = J[i];
      qi = q[i];
      pi = p[i];
      ai = a[i];
      ri = r[i];
    }
  };
  load();
  double alpha, mu;
  if (STEP) {
    double tot[3];
    sum_rows<3>(step, n_step, tot, lds);
    const double n_e = ctl->n_e;
    mu = n_e > 0.0 ? tot[1] / n_e : 0.0;
    const double pkp = tot[0] - mu * tot[2];
    const int outcome = step_outcome(pkp);
    if (outcome) {
      if (first) ctl->stop = outcome;
      return;
    }
    alpha = ctl->rz / pkp;
  } else {
    alpha = ctl->alpha;
    mu = ctl->mu;
  }
  if (first) {
    ctl->rz_old = ctl->rz;
    ctl->iter_old = ctl->iter;
    ctl->stop = DONE_RUNNING;
  }
  double acc[2] = {0.0, 0.0};
  while (i < N) {
    const double qv = qi - ((v.rowT >= 0 && i < v.n_b && ji > 0.0) ? mu : 0.0);
    a[i] = ai + alpha * pi;
    const double rv = ri - alpha * qv;
    r[i] = rv;
    const double zi = ji * rv;
    z[i] = zi;
    acc[0] += rv * zi;
    acc[1] += rv * rv;
    i += vgrid * blockDim.x;
    load();
  }
  dev::block_sum<2>(acc, lds);
  if (threadIdx.x == 0) {
    partials[vblock] = acc[0];
    partials[vgrid + vblock] = acc[1];
  }
}

// Weighted interleaved copy of p, pw4[b] = (w_T p_T, w_q p_q, w_u p_u, 0), read
// by the pixel-order binning (dense_t: intensity-only, pw4[b] = w_T p_T, one
// double per baseline); with Z first p = z + beta p.  pre: the values of the
// thread's first baseline, loaded already.
struct DirectionPre {
  double z[3], p[3];
};
template <bool Z>
__device__ __forceinline__ void load_direction(const View& v, int64_t b, const double* __restrict__ p,
                                               const double* __restrict__ z, DirectionPre& x) {
  const int rows[3] = {v.rowT, v.rowQ, v.rowU};
#pragma unroll
  for (int k = 0; k < 3; ++k) {
    const bool in = b < v.n_b && rows[k] >= 0;
    x.p[k] = in ? p[rows[k] * v.n_b + b] : 0.0;
    x.z[k] = (Z && in) ? z[rows[k] * v.n_b + b] : 0.0;
  }
}
template <bool Z>
__device__ __forceinline__ void store_direction(const View& v, int64_t b, double beta, const DirectionPre& x,
                                                double* __restrict__ p, double* __restrict__ pw4, int dense_t) {
  const int rows[3] = {v.rowT, v.rowQ, v.rowU};
  double w4[3] = {0.0, 0.0, 0.0};
#pragma unroll
  for (int k = 0; k < 3; ++k) {
    if (rows[k] < 0) continue;
    const double pi = Z ? x.z[k] + beta * x.p[k] : x.p[k];
    if (Z) p[rows[k] * v.n_b + b] = pi;
    w4[k] = v.w[k] * pi;
  }
  if (dense_t) {
    pw4[b] = w4[0];
  } else {
    double2* o = reinterpret_cast<double2*>(pw4 + 4 * b);
    o[0] = make_double2(w4[0], w4[1]);
    o[1] = make_double2(w4[2], 0.0);
  }
}

// Stopping test on ||r|| and beta = r'.z' / r.z from the update's n_part
// partials of each kind, then p = z + beta p and its copy.  lds: 32 doubles.
__device__ inline void cg_direction_body(const View& v, double* __restrict__ p, const double* __restrict__ z,
                                         double* __restrict__ pw4, CgCtl* ctl, const double* __restrict__ partials,
                                         int64_t n_part, int dense_t, int64_t vblock, int64_t vgrid, double* lds) {
  const bool first = vblock == 0 && threadIdx.x == 0;
  const int stopped = ctl->stop;
  if (stopped) {
    if (first) ctl->done = stopped;
    return;
  }
  int64_t b = vblock * blockDim.x + threadIdx.x;
  DirectionPre x;
  load_direction<true>(v, b, p, z, x);
  double tot[2];
  sum_rows<2>(partials, n_part, tot, lds);
  const double rz_new = tot[0], rn = sqrt(tot[1]);
  const int iter = ctl->iter_old + 1;
  const int done = (!isfinite(rz_new) || !isfinite(rn))  ? DONE_NAN
                   : rn <= ctl->tol * ctl->b_norm        ? DONE_CONVERGED
                   : iter >= ctl->max_iter               ? DONE_MAXITER
                                                         : DONE_RUNNING;
  const double beta = rz_new / ctl->rz_old;
  if (first) {
    ctl->iter = iter;
    ctl->r_norm = rn;
    if (done)
      ctl->done = done;
    else
      ctl->rz = rz_new;
  }
  if (done) return;
  while (b < v.n_b) {
    store_direction<true>(v, b, beta, x, p, pw4, dense_t);
    b += vgrid * blockDim.x;
    load_direction<true>(v, b, p, z, x);
  }
}

}  // namespace dst
