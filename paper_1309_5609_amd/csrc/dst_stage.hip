// The rescan q = F^T W (F p - A m) (Eqs. 10-12 of arXiv:1309.5609) with the map
// values staged through LDS, for dense problems.
//
// A gather costs the vector memory path about a cycle per lane whatever the
// lanes share, and with hundreds of runs per pixel the rescan is bound by that
// (90 days of intensity, 220 M runs: 0.49 ms, where the 4-byte keys stream in
// 0.19).  Baselines in the rescan order cross the same sky on different days:
// sixteen of them read each of their pixels ten times over.  A block's distinct
// pixels are therefore listed once per solve, its workgroup copies their values
// into LDS, and the runs, whose keys hold positions in the list, are gathered
// from there (64 random 8-byte reads: 8 to 12 cycles).  Half a CU's LDS per
// workgroup, so that one copies while another streams; a block whose list does
// not fit (fewer than one in twenty below) reads its values from memory.
// 90 days of intensity at N_side 512: 0.49 -> 0.30 ms a launch, 0.98 ms for the
// lists, solve 34.9 -> 32.1 ms; 30 days T/q/u FP64 at N_side 256 (39 M runs of
// 20 bytes): 0.205 -> 0.183 ms, lists 0.17 ms, solve 14.63 -> 14.07 ms.
// In a group, a survey of 365 days of intensity beside eight channels: rescans
// 3.45 -> 2.78 ms an iteration, lists 4 ms, 252.6 -> 246.4 ms; 60 days beside
// four: 72.6 -> 71.1 ms.
// The same for the intensity binning (64 pixels per workgroup, whose runs read
// a baseline four times): 0.49 -> 0.41 ms a launch, and 1.6 ms for its lists
// took that away again.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cstdint>
#include <type_traits>

#include "dst_device.h"
#include "dst_stage.h"

namespace dst {
namespace {

using dev::lane_id;

constexpr int kThreads = 512, kWaves = kThreads / 64;
constexpr int kLds = 10112;        // doubles: 79 KB, two workgroups per CU
constexpr int kBaselines = 16;     // per workgroup (and per wavefront of the lists' build)

constexpr int cap_of(bool has_t, bool has_qu) { return kLds / ((has_t ? 1 : 0) + (has_qu ? 2 : 0)); }

// ---------------------------------------------------------------- lists

constexpr int kBuild = 1024;       // threads
constexpr uint32_t kTab = 16384;   // hash table, at most kLds + 5 kBuild of it filled
constexpr uint32_t kEmpty = 0xffffffffu;
static_assert(kLds + 5 * kBuild < (int)kTab, "a probe always ends at a free entry");

// Sixteen consecutive indices share a hash, so the list keeps stretches of them
// together (its copies read whole lines); a probe goes on by an odd stride of
// the index's own, which visits every entry (by ones, stretches that meet made
// the probes long: 3.0 ms for 220 M runs).
__device__ __forceinline__ uint32_t hash_of(uint32_t i) {
  return (i & 15u) | ((((i >> 4) * 2654435761u) >> 22) << 4);
}
__device__ __forceinline__ uint32_t stride_of(uint32_t i) { return ((i * 2246822507u) >> 18) | 1u; }

// One workgroup per block of baselines: the distinct pixels of their runs into
// a hash table, their positions by table place, the list, and the keys with
// positions.  The numbering depends on the insertions' order; no result does.
__global__ void __launch_bounds__(kBuild) k_stage_build(int64_t n_b, const uint32_t* __restrict__ border,
                                                        const uint32_t* __restrict__ bstart,
                                                        const uint32_t* __restrict__ key, int nb, int cap,
                                                        uint32_t* __restrict__ lkey, uint32_t* __restrict__ list,
                                                        uint32_t* __restrict__ count) {
  __shared__ uint32_t tab[kTab];
  __shared__ uint16_t pos[kTab];
  __shared__ uint32_t wsum[kBuild / 64];
  __shared__ uint32_t n;
  constexpr int U = 4;
  const int lane = lane_id(), wave = threadIdx.x >> 6;
  const int64_t k0 = (int64_t)blockIdx.x * kBaselines;
  const int64_t k1 = k0 + kBaselines < n_b ? k0 + kBaselines : n_b;
  for (uint32_t i = threadIdx.x; i < kTab; i += kBuild) tab[i] = kEmpty;
  if (threadIdx.x == 0) n = 0;
  __syncthreads();
  auto peek = [](const uint32_t* x) { return __hip_atomic_load(x, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP); };
  // f(run, key) for the runs of the wavefront's baseline until stop()
  auto each = [&](auto&& stop, auto&& f) {
    for (int64_t k = k0 + wave; k < k1; k += kBuild / 64) {
      const int64_t b = border[k];
      const int64_t r0 = bstart[b], r1 = bstart[b + 1];
      for (int64_t rb = r0 + lane; rb < r1; rb += 64 * U) {
        if (stop()) return;
        uint32_t x[U];
#pragma unroll
        for (int u = 0; u < U; ++u) x[u] = rb + 64 * u < r1 ? key[rb + 64 * u] : 0u;
#pragma unroll
        for (int u = 0; u < U; ++u)
          if (rb + 64 * u < r1) f(rb + 64 * u, x[u]);
      }
    }
  };
  each([&] { return peek(&n) > (uint32_t)cap; },
       [&](int64_t, uint32_t x) {
         const uint32_t i = x >> nb;
         for (uint32_t h = hash_of(i);; h = (h + stride_of(i)) & (kTab - 1)) {
           uint32_t v = peek(&tab[h]);
           if (v == kEmpty) {
             v = atomicCAS(&tab[h], kEmpty, i);
             if (v == kEmpty) atomicAdd(&n, 1u);
           }
           if (v == kEmpty || v == i) break;
         }
       });
  __syncthreads();
  const bool over = n > (uint32_t)cap;
  if (threadIdx.x == 0) count[blockIdx.x] = over ? kStageOver : n;
  if (over) {
    each([] { return false; }, [&](int64_t r, uint32_t x) { lkey[r] = x; });
    return;
  }
  constexpr int PER = kTab / kBuild;
  uint32_t v[PER], mine = 0;
#pragma unroll
  for (int i = 0; i < PER; ++i) {
    v[i] = tab[threadIdx.x * PER + i];
    mine += v[i] != kEmpty;
  }
  uint32_t before = mine;
#pragma unroll
  for (int off = 1; off < 64; off <<= 1) {
    const uint32_t o = (uint32_t)__shfl_up((int)before, off, 64);
    if (lane >= off) before += o;
  }
  if (lane == 63) wsum[wave] = before;
  __syncthreads();
  uint32_t at = before - mine;
  for (int w = 0; w < wave; ++w) at += wsum[w];
#pragma unroll
  for (int i = 0; i < PER; ++i) {
    if (v[i] == kEmpty) continue;
    pos[threadIdx.x * PER + i] = (uint16_t)at;
    list[(int64_t)blockIdx.x * cap + at] = v[i];
    ++at;
  }
  __syncthreads();
  each([] { return false; },
       [&](int64_t r, uint32_t x) {
         const uint32_t i = x >> nb;
         uint32_t h = hash_of(i);
         while (tab[h] != i) h = (h + stride_of(i)) & (kTab - 1);
         lkey[r] = ((uint32_t)pos[h] << nb) | (x & ((1u << nb) - 1u));
       });
}

// ---------------------------------------------------------------- rescan

// As unbin_runs_body, a wavefront per baseline; sixteen baselines of the rescan
// order per workgroup.  STAGED: map values from LDS.
template <typename RT, bool HAS_T, bool HAS_QU, bool STAGED>
__device__ __forceinline__ void rescan_row(const uint32_t* __restrict__ key, const RT* __restrict__ rcs, int nb,
                                           int64_t r0, int64_t r1, const double* __restrict__ m4, const double* lds,
                                           double (&acc)[3]) {
  constexpr bool TONLY = HAS_T && !HAS_QU;
  constexpr int U = TONLY ? 8 : 4, CAP = cap_of(HAS_T, HAS_QU);
  const double* sT = lds;
  const double* sQ = lds + (HAS_T ? CAP : 0);
  const double* sU = sQ + CAP;
  const int lane = lane_id();
  const uint32_t nmask = (1u << nb) - 1u;
  uint32_t x[U];
  CS2<RT> a[U];
  // runs past the end read run r0 again and add nothing
  auto fetch = [&](int64_t rb) {
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const int64_t r = rb + 64 * u < r1 ? rb + 64 * u : r0;
      x[u] = key[r];
      if (HAS_QU) a[u] = reinterpret_cast<const CS2<RT>*>(rcs)[r];
    }
  };
  if (r0 >= r1) return;
  fetch(r0 + lane);
  for (int64_t rb = r0; rb < r1; rb += 64 * U) {
    uint32_t i[U];
    double n[U], C[U], S[U];
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const bool in = rb + lane + 64 * u < r1;
      i[u] = x[u] >> nb;
      n[u] = in ? (double)(int)((x[u] & nmask) + 1u) : 0.0;
      C[u] = (HAS_QU && in) ? (double)a[u].x : 0.0;
      S[u] = (HAS_QU && in) ? (double)a[u].y : 0.0;
    }
    fetch(rb + lane + 64 * U);
#pragma unroll
    for (int u = 0; u < U; ++u) {
      double mT = 0.0, mQ = 0.0, mU = 0.0;
      if (STAGED) {
        if (HAS_T) mT = sT[i[u]];
        if (HAS_QU) {
          mQ = sQ[i[u]];
          mU = sU[i[u]];
        }
      } else if (TONLY) {
        mT = m4[i[u]];
      } else {
        const double2* mp = reinterpret_cast<const double2*>(m4 + 4 * (int64_t)i[u]);
        const double2 m01 = mp[0];
        mT = m01.x;
        mQ = m01.y;
        mU = mp[1].x;
      }
      if (HAS_T) acc[0] += n[u] * mT;
      if (HAS_QU) {
        acc[1] += C[u] * mQ + S[u] * mU;
        acc[2] += C[u] * mU - S[u] * mQ;
      }
    }
  }
}

// vblock of vgrid: the workgroup's place in its problem's launch (vgrid and the
// problem's first workgroup multiples of 8).
template <typename RT, bool HAS_T, bool HAS_QU>
__device__ __forceinline__ void unbin_staged_body(double* lds, double (*red)[3], const View& v, const Stage& S,
                                                  const uint32_t* __restrict__ bstart,
                                                  const uint32_t* __restrict__ border, int nb,
                                                  const RT* __restrict__ rcs, const double* __restrict__ m4,
                                                  const int32_t* __restrict__ nvalid, const double* __restrict__ p,
                                                  double* __restrict__ q, bool cg, double* __restrict__ partials,
                                                  int64_t vblock, int64_t vgrid) {
  constexpr bool TONLY = HAS_T && !HAS_QU;
  constexpr int CAP = cap_of(HAS_T, HAS_QU);
  const int64_t n_blocks = S.blocks;
  const uint32_t* __restrict__ key = S.key;
  const int lane = lane_id(), wave = threadIdx.x >> 6;
  const int64_t n_b = v.n_b;
  // consecutive blocks on one XCD
  const int64_t g = (vblock & 7) * ((n_blocks + 7) / 8) + (vblock >> 3);
  double t[3] = {0.0, 0.0, 0.0};  // p.q, T sums of q and p
  if (g < n_blocks) {
    const uint32_t D = S.count[g];
    const bool staged = D != kStageOver;
    if (staged) {
      const uint32_t* l = S.list + g * CAP;
      for (uint32_t i = threadIdx.x; i < D; i += kThreads) {
        if (TONLY) {
          lds[i] = m4[l[i]];
        } else {
          const double2* mp = reinterpret_cast<const double2*>(m4 + 4 * (int64_t)l[i]);
          const double2 m01 = mp[0];
          const double mU = mp[1].x;
          if (HAS_T) lds[i] = m01.x;
          lds[(HAS_T ? CAP : 0) + i] = m01.y;
          lds[(HAS_T ? 2 * CAP : CAP) + i] = mU;
        }
      }
    }
    __syncthreads();
    const int64_t k1 = g * kBaselines + kBaselines < n_b ? g * kBaselines + kBaselines : n_b;
    for (int64_t k = g * kBaselines + wave; k < k1; k += kWaves) {
      const int64_t b = border[k];
      double acc[3] = {0.0, 0.0, 0.0};
      if (staged)
        rescan_row<RT, HAS_T, HAS_QU, true>(key, rcs, nb, bstart[b], bstart[b + 1], m4, lds, acc);
      else
        rescan_row<RT, HAS_T, HAS_QU, false>(key, rcs, nb, bstart[b], bstart[b + 1], m4, lds, acc);
#pragma unroll
      for (int off = 32; off > 0; off >>= 1) {
#pragma unroll
        for (int c = 0; c < 3; ++c) acc[c] += __shfl_xor(acc[c], off, 64);
      }
      if (lane != 0) continue;
      const int nT = nvalid[b], nQ = nvalid[n_b + b];
      if (HAS_T) {
        const double pb = p[v.rowT * n_b + b];
        const double o = v.w[0] * (pb * (double)nT - acc[0]);
        q[v.rowT * n_b + b] = o;
        t[0] += pb * o;
        if (nT > 0) {
          t[1] += o;
          t[2] += pb;
        }
      }
      if (HAS_QU) {
        const double pq = p[v.rowQ * n_b + b], pu = p[v.rowU * n_b + b];
        const double oq = v.w[1] * (pq * (double)nQ - acc[1]);
        const double ou = v.w[2] * (pu * (double)nQ - acc[2]);
        q[v.rowQ * n_b + b] = oq;
        q[v.rowU * n_b + b] = ou;
        t[0] += pq * oq + pu * ou;
      }
    }
  }
  if (!cg) return;
  if (lane == 0) {
#pragma unroll
    for (int j = 0; j < 3; ++j) red[wave][j] = t[j];
  }
  __syncthreads();
  if (threadIdx.x == 0) {
#pragma unroll
    for (int j = 0; j < 3; ++j) {
      double x = 0.0;
      for (int w = 0; w < kWaves; ++w) x += red[w][j];
      partials[j * vgrid + vblock] = x;
    }
  }
}

template <typename RT, bool HAS_T, bool HAS_QU>
__global__ void __launch_bounds__(kThreads, 4) k_unbin_staged(
    View v, Stage S, const uint32_t* __restrict__ bstart, const uint32_t* __restrict__ border, int nb,
    const RT* __restrict__ rcs, const double* __restrict__ m4, const int32_t* __restrict__ nvalid,
    const double* __restrict__ p, double* __restrict__ q, CgCtl* __restrict__ ctl, double* __restrict__ partials) {
  __shared__ double lds[kLds];
  __shared__ double red[kWaves][3];
  if (ctl && ctl->done) return;
  unbin_staged_body<RT, HAS_T, HAS_QU>(lds, red, v, S, bstart, border, nb, rcs, m4, nvalid, p, q, ctl != nullptr,
                                       partials, blockIdx.x, gridDim.x);
}

template <typename RT, int KIND>
__global__ void __launch_bounds__(kThreads, 4) k_group_unbin_staged(GroupLaunch G) {
  constexpr bool HT = KIND != GK_QU, HQ = KIND != GK_T;
  __shared__ double lds[kLds];
  __shared__ double red[kWaves][3];
  const GroupSlice& L = G.kind[KIND];
  const uint32_t b = blockIdx.x;
  const int j = group_of(L.unbin_start, L.count, b);
  const GroupProblem& P = G.prob[L.first + j];
  if (P.ctl->done) return;
  unbin_staged_body<RT, HT, HQ>(lds, red, P.v, P.stage, P.bstart, P.border, P.nb, static_cast<const RT*>(P.tcs), P.m4,
                                P.nvalid, P.p, P.q, true, P.part_unbin, b - L.unbin_start[j],
                                L.unbin_start[j + 1] - L.unbin_start[j]);
}

}  // namespace

// ---------------------------------------------------------------- launches

bool stage_pays(const View& vc, const Runs& W) {
  // The map beyond one L2 (4 MB), many runs, and enough of them per pixel for
  // the blocks' lists to be short.  us an iteration, plain and staged: 15 days
  // at N_side 256 (63 runs per pixel) T/q/u FP64 293, 274, FP32 245, 232, q/u
  // 202, 182; 20 and 40 days of intensity at N_side 512 (39, 78) 259, 230 and 463,
  // 406; but 10 days there (20) 125, 126, 15 days T/q/u (29) 449, 461, 8 days
  // at N_side 256 (33, 10 M runs) 175, 175, and maps in L2 lose: 40 days of
  // intensity at N_side 128 151, 176, 20 days at N_side 256 112.5, 111.8 and
  // the lists' 0.1 ms.
  const int64_t map_bytes = W.n_obs * (vc.rowQ >= 0 ? 32 : 8);
  return stage_can(vc, W) && W.R >= ((int64_t)1 << 24) && W.R >= 36 * W.n_obs && map_bytes > ((int64_t)4 << 20);
}
int64_t stage_blocks(const View& vc) { return (vc.n_b + kBaselines - 1) / kBaselines; }
int64_t stage_cap(const View& vc) { return cap_of(vc.rowT >= 0, vc.rowQ >= 0); }

hipError_t stage_build(const View& vc, const Runs& W, const Stage& S, hipStream_t st) {
  hipLaunchKernelGGL(k_stage_build, dim3((unsigned)S.blocks), dim3(kBuild), 0, st, vc.n_b, W.border, W.bstart, W.tkey,
                     W.nb, (int)stage_cap(vc), S.key, S.list, S.count);
  return hipGetLastError();
}

int64_t staged_parts(const View& vc) { return 8 * ((stage_blocks(vc) + 7) / 8); }

hipError_t launch_unbin_staged(const View& vc, const Runs& W, const Stage& S, const double* m4, const int32_t* nvalid,
                               const double* p, double* q, CgCtl* ctl, double* partials, hipStream_t st) {
  auto launch = [&](auto rt, auto T, auto Q) {
    using RT = decltype(rt);
    hipLaunchKernelGGL((k_unbin_staged<RT, decltype(T)::value, decltype(Q)::value>),
                       dim3((unsigned)staged_parts(vc)), dim3(kThreads), 0, st, vc, S, W.bstart, W.border, W.nb,
                       static_cast<const RT*>(W.tcs), m4, nvalid, p, q, ctl, partials);
  };
  auto by_streams = [&](auto rt) {
    if (vc.rowT >= 0 && vc.rowQ >= 0)
      launch(rt, std::true_type{}, std::true_type{});
    else if (vc.rowQ >= 0)
      launch(rt, std::false_type{}, std::true_type{});
    else
      launch(rt, std::true_type{}, std::false_type{});
  };
  if (W.f32)
    by_streams(0.0f);
  else
    by_streams(0.0);
  return hipGetLastError();
}

hipError_t launch_group_unbin_staged(const GroupLaunch& G, int kind, hipStream_t st) {
  const dim3 g(G.kind[kind].unbin_total);
  auto by_kind = [&](auto rt) {
    using RT = decltype(rt);
    if (kind == GK_T)
      hipLaunchKernelGGL((k_group_unbin_staged<RT, GK_T>), g, dim3(kThreads), 0, st, G);
    else if (kind == GK_QU)
      hipLaunchKernelGGL((k_group_unbin_staged<RT, GK_QU>), g, dim3(kThreads), 0, st, G);
    else
      hipLaunchKernelGGL((k_group_unbin_staged<RT, GK_TQU>), g, dim3(kThreads), 0, st, G);
  };
  if (G.f32)
    by_kind(0.0f);
  else
    by_kind(0.0);
  return hipGetLastError();
}

}  // namespace dst
