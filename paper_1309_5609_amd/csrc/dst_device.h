// Device helpers shared by the multi-right-hand-side kernels: wavefront and
// workgroup sums (fixed order, so results do not depend on scheduling) and the
// 2psi rotation.
#pragma once

#include <hip/hip_runtime.h>

#include <cstdint>

#include "dst_trig.h"

namespace dst {
namespace dev {

constexpr int kBlock = 256;
constexpr int kWaves = kBlock / 64;

__device__ __forceinline__ int lane_id() { return threadIdx.x & 63; }

__device__ __forceinline__ void rot2(double psi, double& c, double& s) { fast_sincos(2.0 * psi, &s, &c); }

// Butterfly sum over lanes that differ in bits [log2(from), 6): after the
// call every lane holds the sum over its group of 64 / from lanes with equal
// (lane mod from).
template <int N>
__device__ __forceinline__ void lane_group_sum(double (&v)[N], int from) {
  for (int off = 32; off >= from; off >>= 1) {
#pragma unroll
    for (int i = 0; i < N; ++i) v[i] += __shfl_xor(v[i], off, 64);
  }
}

template <int N>
__device__ __forceinline__ void wave_sum(double (&v)[N]) {
#pragma unroll
  for (int off = 32; off > 0; off >>= 1) {
#pragma unroll
    for (int i = 0; i < N; ++i) v[i] += __shfl_xor(v[i], off, 64);
  }
}

// Sum over the whole workgroup; the result is valid in thread 0.
template <int N, typename T>
__device__ __forceinline__ void block_sum(T (&v)[N], T* lds) {
#pragma unroll
  for (int off = 32; off > 0; off >>= 1) {
#pragma unroll
    for (int i = 0; i < N; ++i) v[i] += __shfl_xor(v[i], off, 64);
  }
  const int wid = threadIdx.x >> 6;
  const int nw = blockDim.x >> 6;
  if (lane_id() == 0) {
#pragma unroll
    for (int i = 0; i < N; ++i) lds[i * 16 + wid] = v[i];
  }
  __syncthreads();
  if (threadIdx.x == 0) {
#pragma unroll
    for (int i = 0; i < N; ++i) {
      T acc = lds[i * 16];
      for (int w = 1; w < nw; ++w) acc += lds[i * 16 + w];
      v[i] = acc;
    }
  }
  __syncthreads();
}

// Four consecutive elements from p (aligned to its element only) as 16-byte
// accesses.
template <typename T>
struct Wide {
  typedef T type __attribute__((ext_vector_type(16 / sizeof(T)), aligned(sizeof(T))));
};
template <typename T>
__device__ __forceinline__ void load4(const T* p, T (&o)[4]) {
  using V = typename Wide<T>::type;
  constexpr int N = 16 / sizeof(T);
#pragma unroll
  for (int k = 0; k < 4; k += N) {
    const V v = *reinterpret_cast<const V*>(p + k);
#pragma unroll
    for (int j = 0; j < N; ++j) o[k + j] = v[j];
  }
}

// v of the next (previous) lane; lane 63 (0) keeps its own.
__device__ __forceinline__ int next_lane(int v) {
  return __builtin_amdgcn_update_dpp(v, v, 0x130, 0xf, 0xf, false);  // wave_shl:1
}
__device__ __forceinline__ int prev_lane(int v) {
  return __builtin_amdgcn_update_dpp(v, v, 0x138, 0xf, 0xf, false);  // wave_shr:1
}
__device__ __forceinline__ double next_lane(double v) {
  return __hiloint2double(next_lane(__double2hiint(v)), next_lane(__double2loint(v)));
}

// A wavefront's groups of LPP lanes, one list of `len` entries each (the same on
// every lane of a group, every lane active): whether lists marked `deep` are
// better swept by all 64 lanes one after another.  They are unless the groups'
// lists are about equally long (30 M samples on 768 pixels, all deep: setup +0.1
// ms when swept so).
template <int LPP>
__device__ __forceinline__ bool share_deep(bool deep, uint32_t len) {
  if (__ballot(deep) == 0ull) return false;
  uint32_t most = len, all = deep ? len : 0u;  // all: LPP times the deep lists' sum, in units of 64 entries
  all = (all + 63u) / 64u;
#pragma unroll
  for (int off = 32; off > 0; off >>= 1) {
    most = max(most, (uint32_t)__shfl_xor((int)most, off, 64));
    all += (uint32_t)__shfl_xor((int)all, off, 64);
  }
  return deep && (uint64_t)all * 4u < (uint64_t)most * 3u;
}

// Inverse (QQ, QU, UU) of a pixel's QU block [[a, b], [b, d]]; false, with inv
// untouched, unless its smaller eigenvalue is positive and at least rcond_cut
// times the larger.
__device__ __forceinline__ bool qu_block_inverse(double a, double b, double d, double rcond_cut, double* inv) {
  const double half = 0.5 * (a - d);
  const double rad = sqrt(half * half + b * b);
  const double lmax = 0.5 * (a + d) + rad;
  const double det = a * d - b * b;
  const double lmin = lmax > 0.0 ? det / lmax : 0.0;
  if (!(lmax > 0.0 && lmin > 0.0 && lmin >= rcond_cut * lmax)) return false;
  inv[0] = d / det;
  inv[1] = -b / det;
  inv[2] = a / det;
  return true;
}

// Copies n 4-byte words from global memory to a wavefront's own LDS range
// through the LDS-direct load path (one word per lane and instruction; lane l
// writes dst + 4 (i + l)), so a whole stage is in flight at once with no
// registers.  The source needs 4-byte alignment only.  Call from the whole
// wavefront with dst uniform; the data are in LDS after lds_copy_wait().
__device__ __forceinline__ void lds_copy_words(const void* src, void* dst, int n) {
  const uint32_t* s = static_cast<const uint32_t*>(src);
  uint32_t* d = static_cast<uint32_t*>(dst);
  const int lane = lane_id();
  for (int i = 0; i < n; i += 64) {
    if (i + lane < n) __builtin_amdgcn_global_load_lds(s + i + lane, d + i, 4, 0, 0);
  }
}

// Waits for every outstanding load of the wavefront (the LDS-direct ones
// included); the wave barrier keeps the compiler from moving LDS reads above.
__device__ __forceinline__ void lds_copy_wait() {
  __builtin_amdgcn_s_waitcnt(0);
  __builtin_amdgcn_wave_barrier();
}

}  // namespace dev
}  // namespace dst
