// Two more forms of the binning m = M^-1 A^T W F p (Eqs. 10-12 of
// arXiv:1309.5609) over the runs in pixel order, for problems that the plain
// form (k_bin_runs) serves badly.  Both load everything a pixel ahead of its
// use; sums run in a fixed order.
//
// BIN_LDS keeps the baseline values p in LDS instead of gathering them from L2:
// a wavefront's 64 scattered addresses take about a cycle each in the vector
// memory path, one or two gathers per run, where a random 8-byte LDS read of 64
// lanes takes three to four.  One workgroup per CU copies p and streams the
// runs of its pixels; what bounds it then is the instructions and the latency
// of one step (four runs per lane) at 16 wavefronts per CU.  Seven days FP32 at
// N_side 512 (18 M runs, 6,720 baselines): solve 10.6 -> 9.3 ms; per launch, 4
// days there 67 us less, 7 days FP64 at N_side 256 26 us less, 10 and 25 days of
// intensity at N_side 512 17 and 21 us less; no gain below 2 M runs or 65,536
// pixels (7 days at N_side 64: 3 us more), nor for radiometers, which keep the
// plain form.
// Baselines beyond one LDS were tried in bands (the runs copied band by band, a
// pixel's sums going through the map): 30 days FP64 in 7 bands 0.24 against
// 0.215 ms, 90 days of intensity in 4 bands 0.40 against 0.50 ms a launch but
// 1.7 ms more setup.
//
// BIN_PIPE gathers p, in wavefronts that each take several pixels: with few
// runs per pixel the plain form's chain of loads per pixel (range, runs, p,
// inverse) is what it waits for.  FP32 at N_side 512, 8, 16 and 31 runs per
// pixel: 133 -> 97, 175 -> 141, 301 -> 251 us a launch; FP64 at N_side 256, 8
// runs: 38 -> 31.  With 125 runs per pixel (30 days, N_side 256) it loses, 238
// -> 252 us, and so it does without angles (503 -> 590 us, 90 days).
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cstdint>
#include <type_traits>

#include "dst_forms.h"
#include "dst_device.h"

namespace dst {
namespace {

using dev::lane_id;

constexpr int kThreads = 1024, kWaves = kThreads / 64;
constexpr int kLdsDoubles = 20224;  // 158 KB of the CU's 160
constexpr int64_t kMinRuns = (int64_t)1 << 21, kMinPix = 65536;
constexpr double kSparse = 32.0;  // most runs per pixel of BIN_PIPE
constexpr unsigned kPipeBlocks = 4096;  // 1024 to 16384: 101, 100, 97, 110 us at 8 runs per pixel
constexpr int kPipeThreads = 256, kPipeWaves = kPipeThreads / 64;
constexpr int kU = 4;  // runs per lane whose loads are issued together (twice that without angles)
// A pixel of more steps than this is finished by the whole wavefront.  20 M
// samples FP32, 1000 pixels with 30 % of them: T/q/u 647 -> 136 us a launch (the
// plain form 436), intensity 289 -> 68 (149).
constexpr int kDeepSteps = 16;

// LDS values per baseline.
int columns_of(const View& v) { return (v.rowT >= 0 ? 1 : 0) + (v.rowQ >= 0 ? 2 : 0); }

// Sum over groups of LPP lanes (every lane gets it), by DPP moves up to 16.
template <int LPP, int N>
__device__ __forceinline__ void group_sum(double (&v)[N]) {
  auto step = [&](auto ctrl) {
    constexpr int C = decltype(ctrl)::value;
#pragma unroll
    for (int i = 0; i < N; ++i) {
      const int lo = __double2loint(v[i]), hi = __double2hiint(v[i]);
      v[i] += __hiloint2double(__builtin_amdgcn_update_dpp(hi, hi, C, 0xf, 0xf, false),
                               __builtin_amdgcn_update_dpp(lo, lo, C, 0xf, 0xf, false));
    }
  };
  if constexpr (LPP >= 2) step(std::integral_constant<int, 0xB1>{});    // quad_perm 1 0 3 2
  if constexpr (LPP >= 4) step(std::integral_constant<int, 0x4E>{});    // quad_perm 2 3 0 1
  if constexpr (LPP >= 8) step(std::integral_constant<int, 0x141>{});   // row_half_mirror
  if constexpr (LPP >= 16) step(std::integral_constant<int, 0x140>{});  // row_mirror
  if constexpr (LPP >= 32) {
#pragma unroll
    for (int i = 0; i < N; ++i) v[i] += __shfl_xor(v[i], 16, 64);
  }
}

// block of grid: the workgroup's place in its problem's launch.
template <typename RT, bool HT, bool HQ, int LPP, bool LDS>
__device__ __forceinline__ void bin_body(double* p_lds, const BinRuns& B, const double* __restrict__ pw4,
                                         const double* __restrict__ Minv4, const uint8_t* __restrict__ valid,
                                         double* __restrict__ m4, uint32_t block, uint32_t grid) {
  constexpr bool TONLY = HT && !HQ;
  constexpr int PPW = 64 / LPP, U = TONLY ? 2 * kU : kU;
  const int lane = lane_id(), wave = threadIdx.x >> 6;
  const int grp = lane / LPP, sub = lane % LPP;
  const int nb = B.nb, n_b = B.n_b;
  const uint32_t nmask = (1u << nb) - 1u;
  const CS2<RT>* cs = static_cast<const CS2<RT>*>(B.cs);
  if constexpr (LDS) {
    for (int i = threadIdx.x; i < n_b; i += kThreads) {
      if (TONLY) {
        p_lds[i] = pw4[i];
      } else {
        const double2* q = reinterpret_cast<const double2*>(pw4 + 4 * (int64_t)i);
        const double2 x = q[0];
        if (HT) p_lds[i] = x.x;
        if (HQ) {
          p_lds[(HT ? 1 : 0) * n_b + i] = x.y;
          p_lds[(HT ? 2 : 1) * n_b + i] = q[1].x;
        }
      }
    }
    __syncthreads();
  }
  const double* pT = p_lds;
  const double* pq = p_lds + (HT ? n_b : 0);
  const double* pu = pq + n_b;
  const int64_t c1 = LDS ? B.part[block + 1] : B.n_obs;
  const int64_t cfirst = LDS ? (int64_t)B.part[block] + wave * PPW + grp : ((int64_t)block * kPipeWaves + wave) * PPW + grp;
  const int64_t step = LDS ? kWaves * PPW : (int64_t)grid * kPipeWaves * PPW;
  if (cfirst - grp >= c1) return;  // the whole wavefront has no pixel
  // Software pipeline with every load issued a pixel before its use and no
  // branch around it (few wavefronts hide each other's latency here, and a
  // wait for a load is a wait for all issued before it): the run range two
  // pixels ahead, the runs, validity and inverse one ahead.
  auto range = [&](int64_t c, uint32_t& j0, uint32_t& j1) {
    const int64_t cc = c < c1 ? c : c1 - 1;
    const uint32_t x0 = (uint32_t)B.pstart[cc], x1 = (uint32_t)B.pstart[cc + 1];
    j0 = x0;
    j1 = c < c1 ? x1 : x0;
  };
  struct Fetched {
    uint32_t key[U];
    CS2<RT> ang[U];
  };
  auto fetch = [&](auto lanes, uint32_t j, uint32_t j1, Fetched& f) {
    constexpr int N = decltype(lanes)::value;
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const uint32_t jj = j + N * u < j1 ? j + N * u : 0u;
      f.key[u] = B.key[jj];
      if (HQ) f.ang[u] = cs[jj];
    }
  };
  struct Side {
    uint8_t ok;
    double2 i01, i23;
  };
  auto side = [&](int64_t c, Side& x) {
    const int64_t cc = c < c1 ? c : c1 - 1;
    x.ok = valid[cc];
    const double2* ip = reinterpret_cast<const double2*>(Minv4 + 4 * cc);
    if (TONLY) {
      x.i01.x = ip[0].x;
    } else {
      x.i01 = ip[0];
      x.i23 = ip[1];
    }
  };
  struct Gathered {
    double2 x[LDS ? 1 : U];
    double u[LDS ? 1 : U];
  };
  auto gather = [&](const Fetched& f, Gathered& g) {
    if constexpr (!LDS) {
#pragma unroll
      for (int u = 0; u < U; ++u) {
        const int64_t i = f.key[u] >> nb;
        if (TONLY) {
          g.x[u].x = pw4[i];
        } else {
          const double2* q = reinterpret_cast<const double2*>(pw4 + 4 * i);
          g.x[u] = q[0];
          if (HQ) g.u[u] = q[1].x;
        }
      }
    }
  };
  auto add = [&](auto lanes, const Fetched& f, const Gathered& g, uint32_t j, uint32_t j1, double (&acc)[3]) {
    constexpr int N = decltype(lanes)::value;
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const bool in = j + N * u < j1;
      const int i = in ? (int)(f.key[u] >> nb) : 0;
      const double n = in ? (double)((f.key[u] & nmask) + 1u) : 0.0;
      const double C = HQ && in ? (double)f.ang[u].x : 0.0, S = HQ && in ? (double)f.ang[u].y : 0.0;
      if (HT) acc[0] += n * (LDS ? pT[i] : g.x[u].x);
      if (HQ) {
        const double xq = LDS ? pq[i] : g.x[u].y, xu = LDS ? pu[i] : g.u[u];
        acc[1] += C * xq - S * xu;
        acc[2] += S * xq + C * xu;
      }
    }
  };
  // runs j, j + N, ... of a pixel past its first step
  auto more = [&](auto lanes, uint32_t j, uint32_t j1, double (&acc)[3]) {
    constexpr int N = decltype(lanes)::value;
    for (; j < j1; j += N * U) {
      Fetched f;
      fetch(lanes, j, j1, f);
      Gathered h;
      gather(f, h);
      add(lanes, f, h, j, j1, acc);
    }
  };
  const std::integral_constant<int, LPP> group{};
  uint32_t a0, a1, n0, n1;
  Fetched now, next;
  Side s_now, s_next;
  range(cfirst, a0, a1);
  range(cfirst + step, n0, n1);
  side(cfirst, s_now);
  fetch(group, a0 + sub, a1, now);
  for (int64_t c = cfirst; c - grp < c1; c += step) {
    Gathered g;
    gather(now, g);
    side(c + step, s_next);
    fetch(group, n0 + sub, n1, next);
    uint32_t f0, f1;
    range(c + 2 * step, f0, f1);
    double acc[3] = {0.0, 0.0, 0.0};
    add(group, now, g, a0 + sub, a1, acc);
    const bool deep = dev::share_deep<LPP>(a1 - a0 > (uint32_t)(kDeepSteps * LPP * U), a1 - a0);
    if (!deep) more(group, a0 + sub + LPP * U, a1, acc);
    for (unsigned long long m = __ballot(deep && sub == 0); m != 0; m &= m - 1) {
      const int src = __ffsll(m) - 1;
      const uint32_t j = __shfl(a0, src, 64) + LPP * U, j1 = __shfl(a1, src, 64);
      double t[3] = {0.0, 0.0, 0.0};
      more(std::integral_constant<int, 64>{}, j + lane, j1, t);
      // the group's lanes add a part each
      for (int i = 0; i < 3; ++i) {
#pragma unroll
        for (int off = 32; off >= LPP; off >>= 1) t[i] += __shfl_xor(t[i], off, 64);
        acc[i] += grp == src / LPP ? t[i] : 0.0;
      }
    }
    const Side x = s_now;
    now = next;
    s_now = s_next;
    a0 = n0;
    a1 = n1;
    n0 = f0;
    n1 = f1;
    group_sum<LPP>(acc);
    if (sub != 0 || c >= c1 || x.ok == 0) continue;  // m stays 0 on invalid pixels
    if (TONLY) {
      m4[c] = x.i01.x * acc[0];
      continue;
    }
    double2* mp = reinterpret_cast<double2*>(m4 + 4 * c);
    mp[0] = make_double2(x.i01.x * acc[0], x.i01.y * acc[1] + x.i23.x * acc[2]);
    mp[1] = make_double2(x.i23.x * acc[1] + x.i23.y * acc[2], 0.0);
  }
}

template <typename RT, bool HT, bool HQ, int LPP>
__global__ void __launch_bounds__(kThreads) k_bin_lds(BinRuns B, const double* __restrict__ pw4,
                                                       const double* __restrict__ Minv4,
                                                       const uint8_t* __restrict__ valid, double* __restrict__ m4,
                                                       const CgCtl* __restrict__ gate) {
  __shared__ double p_lds[kLdsDoubles];
  if (gate && gate->done) return;
  bin_body<RT, HT, HQ, LPP, true>(p_lds, B, pw4, Minv4, valid, m4, blockIdx.x, gridDim.x);
}

template <typename RT, bool HT, bool HQ, int LPP>
__global__ void __launch_bounds__(kPipeThreads, 4) k_bin_pipe(BinRuns B, const double* __restrict__ pw4,
                                                       const double* __restrict__ Minv4,
                                                       const uint8_t* __restrict__ valid, double* __restrict__ m4,
                                                       const CgCtl* __restrict__ gate) {
  if (gate && gate->done) return;
  bin_body<RT, HT, HQ, LPP, false>(nullptr, B, pw4, Minv4, valid, m4, blockIdx.x, gridDim.x);
}

template <typename RT, int KIND, int LPP>
__global__ void __launch_bounds__(kThreads) k_group_bin_lds(GroupLaunch G) {
  constexpr bool HT = KIND == GK_T || KIND == GK_TQU, HQ = KIND == GK_QU || KIND == GK_TQU;
  __shared__ double p_lds[kLdsDoubles];
  const GroupSlice& S = G.kind[KIND];
  const uint32_t b = blockIdx.x;
  const int j = group_of(S.bin_start, S.count, b);
  const GroupProblem& P = G.prob[S.first + j];
  if (P.ctl->done) return;
  bin_body<RT, HT, HQ, LPP, true>(p_lds, P.bin, P.pw4, P.Minv4, P.valid, P.m4, b - S.bin_start[j],
                                                S.bin_start[j + 1] - S.bin_start[j]);
}

template <typename RT, int KIND, int LPP>
__global__ void __launch_bounds__(kPipeThreads, 4) k_group_bin_pipe(GroupLaunch G) {
  constexpr bool HT = KIND == GK_T || KIND == GK_TQU, HQ = KIND == GK_QU || KIND == GK_TQU;
  const GroupSlice& S = G.kind[KIND];
  const uint32_t b = blockIdx.x;
  const int j = group_of(S.bin_start, S.count, b);
  const GroupProblem& P = G.prob[S.first + j];
  if (P.ctl->done) return;
  bin_body<RT, HT, HQ, LPP, false>(nullptr, P.bin, P.pw4, P.Minv4, P.valid, P.m4, b - S.bin_start[j],
                                          S.bin_start[j + 1] - S.bin_start[j]);
}

// Pixel ranges of the workgroups: as much work each, a pixel counting as
// `per_pixel` runs (a step's runs: balanced by runs alone, the workgroups of
// sparse pixels took 133 us where the mean was 48).
__global__ void k_lds_parts(int64_t n_obs, const int64_t* __restrict__ pstart, int64_t per_pixel, uint32_t blocks,
                             uint32_t* __restrict__ part) {
  const uint32_t g = blockIdx.x * blockDim.x + threadIdx.x;
  if (g > blocks) return;
  const int64_t want = (pstart[n_obs] + per_pixel * n_obs) * g / blocks;
  int64_t lo = 0, hi = n_obs;
  while (lo < hi) {
    const int64_t mid = (lo + hi) >> 1;
    if (pstart[mid] + per_pixel * mid < want)
      lo = mid + 1;
    else
      hi = mid;
  }
  part[g] = g == blocks ? (uint32_t)n_obs : (uint32_t)lo;
}

template <typename F>
void by_bool(bool b, F&& f) {
  if (b)
    f(std::true_type{});
  else
    f(std::false_type{});
}
template <typename F>
void by_lpp(int lpp, F&& f) {
  if (lpp <= 4)
    f(std::integral_constant<int, 4>{});
  else if (lpp == 8)
    f(std::integral_constant<int, 8>{});
  else if (lpp == 16)
    f(std::integral_constant<int, 16>{});
  else
    f(std::integral_constant<int, 32>{});
}

}  // namespace

int bin_form_lanes(int64_t runs, int64_t n_obs, bool t_only) {
  const double mean = (double)runs / (double)n_obs / (t_only ? 2.0 : 1.0);
  return mean <= 16.0 ? 4 : (mean <= 32.0 ? 8 : (mean <= 64.0 ? 16 : 32));
}

bool bin_sparse(int64_t runs, int64_t n_obs, bool angles) {
  return angles && runs >= kMinRuns && (double)runs <= kSparse * (double)n_obs;
}

uint32_t bin_pipe_blocks(int64_t n_obs, int lpp) {
  const int64_t per = kPipeWaves * (64 / lpp);
  return (uint32_t)std::max<int64_t>(1, std::min<int64_t>(kPipeBlocks, (n_obs + per - 1) / per));
}

BinShape bin_shape(const View& vc, const Runs& W, int mode) {
  BinShape s;
  if (mode == BIN_PLAIN || W.n_obs <= 0) return s;
  const bool fits = !vc.iqu && vc.n_b * columns_of(vc) <= kLdsDoubles, pipe = vc.rowQ >= 0;
  if (mode < 0) {
    if (fits && W.R >= kMinRuns && W.n_obs >= kMinPix)
      s.form = BIN_LDS;
    else if (bin_sparse(W.R, W.n_obs, vc.rowQ >= 0))
      s.form = BIN_PIPE;
  } else if (mode == BIN_LDS ? fits : pipe) {
    s.form = mode;
  }
  s.lpp = bin_form_lanes(W.R, W.n_obs, vc.rowT >= 0 && vc.rowQ < 0 && !vc.iqu);
  s.blocks = s.form == BIN_LDS ? (uint32_t)std::min<int64_t>(256, std::max<int64_t>(1, W.R / 16384))
                               : bin_pipe_blocks(W.n_obs, s.lpp);
  return s;
}

hipError_t bin_build(const View& vc, const Runs& W, const BinShape& s, uint32_t* part, BinRuns* out, hipStream_t st) {
  if (s.form == BIN_LDS)
    hipLaunchKernelGGL(k_lds_parts, dim3(s.blocks / 256 + 1), dim3(256), 0, st, W.n_obs, W.pstart,
                       (int64_t)s.lpp * kU, s.blocks, part);
  out->n_obs = W.n_obs;
  out->n_b = (int)vc.n_b;
  out->nb = W.nb;
  out->pstart = W.pstart;
  out->part = part;
  out->key = W.pkey;
  out->cs = W.pcs;
  return hipGetLastError();
}

hipError_t launch_bin_form(const View& vc, const BinRuns& B, const BinShape& s, bool f32, const double* pw4,
                           const double* Minv4, const uint8_t* valid, double* m4, const CgCtl* gate, hipStream_t st) {
  by_bool(f32, [&](auto f) {
    using RT = typename std::conditional<decltype(f)::value, float, double>::type;
    by_lpp(s.lpp, [&](auto l) {
      constexpr int LPP = decltype(l)::value;
      auto launch = [&](auto kern, int threads) {
        hipLaunchKernelGGL(kern, dim3(s.blocks), dim3(threads), 0, st, B, pw4, Minv4, valid, m4, gate);
      };
      const bool t = vc.rowT >= 0;
      if (s.form == BIN_PIPE && t)
        launch(k_bin_pipe<RT, true, true, LPP>, kPipeThreads);
      else if (s.form == BIN_PIPE)
        launch(k_bin_pipe<RT, false, true, LPP>, kPipeThreads);
      else if (t && vc.rowQ >= 0)
        launch(k_bin_lds<RT, true, true, LPP>, kThreads);
      else if (vc.rowQ >= 0)
        launch(k_bin_lds<RT, false, true, LPP>, kThreads);
      else
        launch(k_bin_lds<RT, true, false, LPP>, kThreads);
    });
  });
  return hipGetLastError();
}

hipError_t launch_group_bin_form(const GroupLaunch& G, int kind, hipStream_t st) {
  const GroupSlice& S = G.kind[kind];
  by_bool(G.f32 != 0, [&](auto f) {
    using RT = typename std::conditional<decltype(f)::value, float, double>::type;
    by_lpp(S.lpp, [&](auto l) {
      constexpr int LPP = decltype(l)::value;
      auto launch = [&](auto kern, int threads) {
        hipLaunchKernelGGL(kern, dim3(S.bin_total), dim3(threads), 0, st, G);
      };
      if (S.form == BIN_PIPE && kind == GK_QU)
        launch(k_group_bin_pipe<RT, GK_QU, LPP>, kPipeThreads);
      else if (S.form == BIN_PIPE)
        launch(k_group_bin_pipe<RT, GK_TQU, LPP>, kPipeThreads);
      else if (kind == GK_T)
        launch(k_group_bin_lds<RT, GK_T, LPP>, kThreads);
      else if (kind == GK_QU)
        launch(k_group_bin_lds<RT, GK_QU, LPP>, kThreads);
      else
        launch(k_group_bin_lds<RT, GK_TQU, LPP>, kThreads);
    });
  });
  return hipGetLastError();
}

}  // namespace dst
