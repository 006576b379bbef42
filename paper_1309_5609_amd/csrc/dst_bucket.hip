// One-shot binning of a timeline into per-pixel sums, hits and weight blocks
// without global atomics (dst_pixel_setup, dst_bin, dst_baseline_reduce,
// dst_residual).
//
// Pixels are dealt to buckets round robin, 64 neighbouring pixels at a time (fewer
// where the map has no 256 such groups).  k_bucket_fill splits the timeline into chunks, one
// workgroup each: it sums stretches of consecutive samples on one pixel
// ("runs") and writes each run's record into the chunk's own range,
// ordered by bucket, with the bucket offsets beside it.  k_bucket_sum, one
// workgroup per bucket, walks its segment of every chunk, adds the records in
// LDS and finishes its pixels there: validity, block inverse, map.  The
// timeline is read once and a run costs one record write and read, where the
// atomic form reads it twice (hits and blocks first, the sums after) and pays
// up to seven device-scope atomics per run.  Measured against it: map of 30
// days FP32 at N_side 256 10.8 -> 1.7 ms (k_bucket_fill 0.29 ms per 2^25
// samples, about 1 GB moved, and k_bucket_sum 0.15 ms), of 6 hours at N_side
// 64 79 -> 42 us of kernels.  k_bucket_fill is bound by HBM traffic and its
// FP64 angle functions, k_bucket_sum by the latency of its short segments.
//
// Coarse maps and long stays on one pixel put many records into few buckets, and
// into few LDS places of them.  There the groups are smaller, a pixel's sums are
// kept in up to 64 copies, and the stretch of a wavefront's lanes that stay on
// one pixel is one record.  30 M samples T/q/u FP64 without these, with them, and
// by the atomic form: stays of 5000 samples on 48 pixels 36.7, 0.27 and 3.6 ms,
// 48 pixels at random 28.7, 1.2 and 122 ms, one pixel 36.9, 0.35 and 33.8 ms.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cmath>
#include <cstdint>
#include <type_traits>

#include "dst_bucket.h"
#include "dst_device.h"
#include "dst_trig.h"

namespace dst {
namespace {

using dev::kBlock;
using dev::kWaves;
using dev::lane_id;
using dev::load4;
using dev::next_lane;
using dev::prev_lane;
using dev::qu_block_inverse;

constexpr int kMaxLogG = 6;       // at most 64 pixels dealt together
constexpr int kMaxLogC = 6;       // at most 64 copies of a pixel's sums
constexpr int kMinLogB = 8;       // at least 256 buckets: one workgroup of k_bucket_sum per CU
constexpr int kMaxLogB = 11;      // at most 2048 buckets (their counters share LDS in k_bucket_fill)
constexpr int kSumBlock = 1024;  // (at most bucket_pix)
// Samples whose records are held at once: 1 GiB of them at most with equal q/u
// weights, 1.75 GiB with block sums (64 M samples there: 1.43 ms, 1.50 in pieces
// of 1 GiB).
constexpr int64_t kPiece = (int64_t)1 << 25;

// Most pixels of a bucket: what LDS holds of hits and sums (28 bytes a pixel
// with equal q/u weights, 52 with block sums).  Large buckets make long
// segments: 30 days at N_side 256 took 1.71 ms with 3072 pixels, 1.88 with
// 1536.
constexpr int bucket_pix(bool blk) { return blk ? 1536 : 3072; }
bool has_blocks(const View& v) { return v.rowQ >= 0 && v.w[1] != v.w[2]; }

// Record of a run: local pixel | (samples << 16) | (kBadAngle if an angle is
// not finite), then the sums of its data terms.
constexpr uint32_t kBadAngle = 0x80000000u;
struct alignas(16) Rec3 {
  uint32_t key;
  uint32_t pad;
  double x[3];
};
struct alignas(16) Rec1 {
  uint32_t key;
  uint32_t pad;
  double x[1];
};
template <bool HQ, bool DATA>
struct RecOf {
  using type = Rec3;
};
template <>
struct RecOf<false, true> {
  using type = Rec1;
};
template <bool HQ>
struct RecOf<HQ, false> {
  using type = uint32_t;
};

// A lane's four consecutive samples as runs: start[k] says that sample k heads
// a run this lane records.  A run that goes on into the next lane and ends
// there is recorded by the lane where it starts (gives: this lane's first
// stretch belongs to the previous lane; takes: the next lane's to this one);
// longer ones are recorded in pieces.
// Where half of the lanes at least lie, whole, on the pixel of a whole lane before
// them (joined), such a stretch is one record, of its first lane.
struct QuadRuns {
  bool brk[4];  // sample k on another pixel than sample k - 1 (brk[0] true)
  bool start[4];
  bool takes;
  unsigned long long goes_on;  // lanes whose stretch began before them (0: none are joined)
};
// JOIN: false where no group of the wavefront is known to have joined lanes.
template <bool JOIN>
__device__ __forceinline__ QuadRuns quad_runs(const int (&p)[4]) {
  QuadRuns q;
  q.brk[0] = true;
#pragma unroll
  for (int k = 1; k < 4; ++k) q.brk[k] = p[k] != p[k - 1];
  const int lane = lane_id();
  const int before = prev_lane(p[3]);
  const bool same = lane > 0 && p[0] >= 0 && before == p[0];
  const bool whole = !(q.brk[1] || q.brk[2] || q.brk[3]);
  const bool gives = same && !whole;
  const int from_next = next_lane((int)gives);  // on every lane: a lane masked off by a branch gives no data
  q.takes = lane < 63 && from_next != 0;
#pragma unroll
  for (int k = 0; k < 4; ++k) q.start[k] = q.brk[k] && p[k] >= 0;
  q.start[0] = q.start[0] && !gives;
  q.goes_on = 0;
  if (JOIN) {
    const unsigned long long wholes = __ballot(whole), on = __ballot(same) & wholes & wholes << 1;
    if (__popcll(on) >= 32) {
      q.goes_on = on;
      if (on >> lane & 1ull) q.start[0] = false;
    }
  }
  return q;
}

// x[k] (k a run start) becomes the sum over the run.
template <typename T>
__device__ __forceinline__ void quad_sums(const QuadRuns& q, T (&x)[4]) {
  T first = x[3];  // sum over this lane's first stretch
#pragma unroll
  for (int k = 2; k >= 0; --k) first = q.brk[k + 1] ? x[k] : x[k] + first;
  const T more = next_lane(first);
  if (q.takes) x[3] += more;
#pragma unroll
  for (int k = 2; k >= 0; --k)
    if (!q.brk[k + 1]) x[k] += x[k + 1];
}

// Joined lanes: n and x[j][0] of a stretch's first lane become the sums over it.
template <int N>
__device__ __forceinline__ void join_sums(const QuadRuns& q, int& n, double (&x)[N][4]) {
  const int lane = lane_id();
  const unsigned long long ends = lane < 63 ? ~q.goes_on >> (lane + 1) : 0ull;
  const int end = ends ? lane + __ffsll(ends) : 64;  // first lane past this lane's stretch
#pragma unroll 1
  for (int off = 1; off < 64; off <<= 1) {
    const bool in = lane + off < end;
    const int m = __shfl_down(n, off, 64);
    n += in ? m : 0;
#pragma unroll
    for (int j = 0; j < N; ++j) {
      const double o = __shfl_down(x[j][0], off, 64);
      x[j][0] += in ? o : 0.0;
    }
  }
}

// One chunk [lo, hi) per workgroup.  DATA: the data sums of x = tod + bsign F
// base (either may be NULL) as T: w_T x; q/u: the rotated, weighted pair.
// Four consecutive samples per lane: 16-byte loads, and the run sums inside a
// lane are plain additions (a sum across lanes for every 64 samples took
// twice the vector instructions: 0.47 ms against 0.29 per 2^25 samples).
// EQ: equal q/u weights, whose QU block is w h times the unit matrix, so no
// block sums are kept (a non-finite angle is flagged instead: it makes the
// block NaN and so invalid); else rec2 holds each run's three block sums.
template <typename PT, typename TT, bool HT, bool HQ, bool DATA, bool EQ>
__global__ void __launch_bounds__(kBlock) k_bucket_fill(View v, const TT* __restrict__ tod,
                                                        const double* __restrict__ base, double bsign, int64_t t_lo,
                                                        int64_t t_hi, int64_t chunk, int log_b, int log_g,
                                                        uint16_t* __restrict__ off,
                                                        typename RecOf<HQ, DATA>::type* __restrict__ rec,
                                                        double* __restrict__ rec2, int* __restrict__ err) {
  using Rec = typename RecOf<HQ, DATA>::type;
  __shared__ uint32_t cur[1 << kMaxLogB];
  __shared__ uint32_t wsum[kWaves];
  const int lane = lane_id(), wave = threadIdx.x >> 6;
  const int B = 1 << log_b;
  const uint32_t bmask = (uint32_t)B - 1u;
  const int64_t lo = t_lo + (int64_t)blockIdx.x * chunk;
  const int span = (int)(min(lo + chunk, t_hi) - lo);
  const int groups = (span + 255) / 256;  // of 256 samples, four per lane
  const int32_t* pix = v.pix + lo;
  for (int b = threadIdx.x; b < B; b += kBlock) cur[b] = 0;
  __syncthreads();
  auto load = [&](const auto* a, int i, auto none, auto& o) {
    if (i + 4 <= span) {
      load4(a + i, o);
    } else {
#pragma unroll
      for (int k = 0; k < 4; ++k) o[k] = i + k < span ? a[i + k] : none;
    }
  };
  // runs per bucket
  bool bad = false, joined = false;
  int ahead[4];
  load(pix, 256 * wave + 4 * lane, -1, ahead);
  for (int g = wave; g < groups; g += kWaves) {
    int p[4];
#pragma unroll
    for (int k = 0; k < 4; ++k) {
      p[k] = ahead[k];
      if (p[k] >= v.n_pix) {
        bad = true;
        p[k] = -1;
      }
    }
    load(pix, 256 * (g + kWaves) + 4 * lane, -1, ahead);
    const QuadRuns q = quad_runs<true>(p);
    joined |= q.goes_on != 0;
#pragma unroll
    for (int k = 0; k < 4; ++k)
      if (q.start[k]) atomicAdd(&cur[((uint32_t)p[k] >> log_g) & bmask], 1u);
  }
  if (__ballot(bad) != 0ull && lane == 0) atomicOr(err, 1);
  __syncthreads();
  // bucket offsets (exclusive scan; each thread takes B / kBlock consecutive buckets)
  {
    const int per = B > kBlock ? B / kBlock : 1;
    const int b0 = threadIdx.x * per;
    uint32_t mine = 0;
    for (int k = 0; k < per; ++k)
      if (b0 + k < B) mine += cur[b0 + k];
    uint32_t incl = mine;
    for (int d = 1; d < 64; d <<= 1) {
      const uint32_t o = __shfl_up(incl, d, 64);
      if (lane >= d) incl += o;
    }
    if (lane == 63) wsum[wave] = incl;
    __syncthreads();
    uint32_t at = incl - mine;
    for (int w = 0; w < wave; ++w) at += wsum[w];
    uint16_t* o = off + (int64_t)blockIdx.x * (B + 1);
    for (int k = 0; k < per; ++k) {
      if (b0 + k >= B) break;
      const uint32_t n = cur[b0 + k];
      cur[b0 + k] = at;
      o[b0 + k] = (uint16_t)at;
      at += n;
      if (b0 + k == B - 1) o[B] = (uint16_t)at;
    }
  }
  __syncthreads();
  // run sums, written at the bucket's next place
  constexpr int ND = DATA ? (HT ? 1 : 0) + (HQ ? 2 : 0) : 0;
  constexpr bool BLK = HQ && !EQ;
  constexpr int N = ND + (BLK ? 3 : 0);
  const PT* psi = static_cast<const PT*>(v.psi) + (HQ ? lo : 0);
  Rec* out = rec + (int64_t)blockIdx.x * chunk;
  double* out2 = BLK ? rec2 + 3 * (int64_t)blockIdx.x * chunk : nullptr;
  const TT* tT = DATA && HT ? tod + v.rowT * v.n_t + lo : nullptr;
  const TT* tq = DATA && HQ ? tod + v.rowQ * v.n_t + lo : nullptr;
  const TT* tu = DATA && HQ ? tod + v.rowU * v.n_t + lo : nullptr;
  const bool has_tod = DATA && tod != nullptr;
  const uint32_t L = (uint32_t)v.L;
  // baseline of the group's first sample, and its place in that baseline
  int64_t gb = 0;
  uint32_t gr = 0;
  if (DATA && base) {
    const int64_t t0 = lo + 256 * wave;
    gb = t0 / v.L;
    gr = (uint32_t)(t0 - gb * v.L);
  }
  struct In {
    int p[4];
    PT ps[4];
    TT xT[4], xq[4], xu[4];
  };
  auto fetch = [&](int g, In& r) {
    const int i = 256 * g + 4 * lane;
    load(pix, i, -1, r.p);
    if (HQ) load(psi, i, PT(0), r.ps);
    if (has_tod) {
      if (HT) load(tT, i, TT(0), r.xT);
      if (HQ) {
        load(tq, i, TT(0), r.xq);
        load(tu, i, TT(0), r.xu);
      }
    }
  };
  In now;
  auto write = [&](int g, auto join) {
    constexpr bool JOIN = decltype(join)::value;
    fetch(g, now);
    int p[4], cnt[4];
    double x[N > 0 ? N : 1][4] = {};
#pragma unroll
    for (int k = 0; k < 4; ++k) p[k] = now.p[k] >= v.n_pix ? -1 : now.p[k];
    double a2[4], sin4[4] = {0.0, 0.0, 0.0, 0.0}, cos4[4] = {0.0, 0.0, 0.0, 0.0};
    double oT[4], oq[4], ou[4];  // offsets of the samples' baselines
    if (DATA && base) {
      // first sample's baseline, and whether all four lie in it
      const uint32_t r = gr + 4u * (uint32_t)lane;
      const uint32_t step = L >= 256u ? (r >= L ? 1u : 0u) : r / L;
      int64_t b = gb + step;
      const bool whole = r - step * L + 4u <= L;
#pragma unroll
      for (int k = 0; k < 4; ++k) {
        if (k > 0 && !whole) b = gb + (r + k) / L;
        b = b < v.n_b ? b : v.n_b - 1;  // past the last sample
        if (k == 0 || !whole) {
          if (HT) oT[k] = bsign * base[v.rowT * v.n_b + b];
          if (HQ) {
            oq[k] = bsign * base[v.rowQ * v.n_b + b];
            ou[k] = bsign * base[v.rowU * v.n_b + b];
          }
        } else {
          oT[k] = oT[0];
          oq[k] = oq[0];
          ou[k] = ou[0];
        }
      }
    }
#pragma unroll
    for (int k = 0; k < 4; ++k) {
      cnt[k] = 1;
      a2[k] = HQ ? 2.0 * (double)now.ps[k] : 0.0;
      if (HQ && EQ && !isfinite(a2[k])) cnt[k] |= 1 << 16;  // (a record holds 259 samples at most)
    }
    if (HQ && (DATA || BLK)) fast_sincos4(a2, sin4, cos4);
#pragma unroll
    for (int k = 0; k < 4; ++k) {
      double xT = 0.0, xq = 0.0, xu = 0.0;
      const double c = cos4[k], s = sin4[k];
      if (DATA) {
        if (has_tod) {
          xT = (double)now.xT[k];
          xq = (double)now.xq[k];
          xu = (double)now.xu[k];
        }
        if (base) {
          xT += oT[k];
          xq += oq[k];
          xu += ou[k];
        }
        if (HT) x[0][k] = v.w[0] * xT;
        if (HQ) {
          const double wq = v.w[1] * xq, wu = v.w[2] * xu;
          x[ND - 2][k] = c * wq - s * wu;
          x[ND - 1][k] = s * wq + c * wu;
        }
      }
      if (BLK) {
        const double wq = v.w[1], wu = v.w[2];
        x[N - 3][k] = wq * c * c + wu * s * s;
        x[N - 2][k] = (wq - wu) * c * s;
        x[N - 1][k] = wq * s * s + wu * c * c;
      }
    }
    const QuadRuns q = quad_runs<JOIN>(p);
    quad_sums(q, cnt);
#pragma unroll
    for (int j = 0; j < N; ++j) quad_sums(q, x[j]);
    if (JOIN && q.goes_on) join_sums(q, cnt[0], x);
#pragma unroll
    for (int k = 0; k < 4; ++k) {
      if (!q.start[k]) continue;
      const uint32_t grp = (uint32_t)p[k] >> log_g;
      const uint32_t local = ((grp >> log_b) << log_g) | ((uint32_t)p[k] & ((1u << log_g) - 1u));
      const uint32_t at = atomicAdd(&cur[grp & bmask], 1u);
      const uint32_t key = local | ((uint32_t)(cnt[k] & 0xffff) << 16) | (cnt[k] >> 16 ? kBadAngle : 0u);
      if constexpr (!DATA) {
        out[at] = key;
      } else if constexpr (!HQ) {
        Rec1 r;
        r.key = key;
        r.pad = 0;
        r.x[0] = x[0][k];
        out[at] = r;
      } else {
        Rec3 r;
        r.key = key;
        r.pad = 0;
        r.x[0] = HT ? x[0][k] : 0.0;
        r.x[1] = x[ND - 2][k];
        r.x[2] = x[ND - 1][k];
        out[at] = r;
      }
      if (BLK) {
#pragma unroll
        for (int j = 0; j < 3; ++j) out2[3 * (int64_t)at + j] = x[N - 3 + j][k];
      }
    }
    if (DATA && base) {
      gr += 256 * kWaves;
      if (gr >= L) {
        const uint32_t n = gr / L;
        gb += n;
        gr -= n * L;
      }
    }
  };
  // (the test for joined lanes in the way of every group: 30 days 1.75 ms, 1.72 without)
  if (joined) {
    for (int g = wave; g < groups; g += kWaves) write(g, std::true_type{});
  } else {
    for (int g = wave; g < groups; g += kWaves) write(g, std::false_type{});
  }
}

// One bucket per workgroup: its records of every chunk added in LDS, carried
// between pieces of a long timeline in acc_hits / acc (unless first / last),
// and after the last piece its pixels' outputs.
template <bool HT, bool HQ, bool DATA, bool EQ>
__global__ void __launch_bounds__(kSumBlock) k_bucket_sum(View v, double rcond_cut, const uint16_t* __restrict__ off,
                                                          const typename RecOf<HQ, DATA>::type* __restrict__ rec,
                                                          const double* __restrict__ rec2, int n_chunks, int64_t chunk,
                                                          int log_b, int log_g, int log_c, int n_local, int first,
                                                          int last,
                                                          uint32_t* __restrict__ acc_hits, double* __restrict__ acc,
                                                          BucketOut o) {
  using Rec = typename RecOf<HQ, DATA>::type;
  constexpr bool BLK = HQ && !EQ;
  constexpr int ND = DATA ? (HT ? 1 : 0) + (HQ ? 2 : 0) : 0;
  constexpr int NA = ND + (BLK ? 3 : 0);
  constexpr int PX = bucket_pix(BLK);
  __shared__ uint32_t hits[PX];
  __shared__ double sum[NA > 0 ? NA : 1][NA > 0 ? PX : 1];
  // neighbouring buckets share cache lines of records: each XCD (workgroup i
  // runs on XCD i mod 8) takes B / 8 neighbours
  const int B = 1 << log_b;
  const int b = (int)((blockIdx.x & 7u) << (log_b - 3) | blockIdx.x >> 3);
  // pixel l's copies are at l << log_c and the places after it; a lane adds into its own
  const int cmask = (1 << log_c) - 1;
  for (int i = threadIdx.x; i < n_local << log_c; i += kSumBlock) {
    const int l = i >> log_c;
    const bool carried = !first && (i & cmask) == 0;
    hits[i] = carried ? acc_hits[(int64_t)b * n_local + l] : 0u;
#pragma unroll
    for (int k = 0; k < NA; ++k) sum[k][i] = carried ? acc[((int64_t)b * NA + k) * n_local + l] : 0.0;
  }
  __syncthreads();
  // A wavefront takes the segments of 64 chunks and deals their records to its
  // lanes as one list: record k belongs to the last segment that starts at or
  // before k.
  __shared__ uint32_t seg_start[kSumBlock / 64][64], seg_at[kSumBlock / 64][64];
  const int lane = lane_id(), wave = threadIdx.x >> 6;
  constexpr int U = 4, W = kSumBlock / 64;
  auto add = [&](const Rec& r, int64_t at) {
    uint32_t key;
    if constexpr (DATA)
      key = r.key;
    else
      key = r;
    const int l = (int)((key & 0xffffu) << log_c) | (lane & cmask);
    atomicAdd(&hits[l], (key >> 16) & 0x7fffu);
    if (HQ && EQ && (key & kBadAngle)) atomicOr(&hits[l], kBadAngle);
    if constexpr (DATA) {
      if constexpr (!HQ) {
        unsafeAtomicAdd(&sum[0][l], r.x[0]);
      } else {
        if (HT) unsafeAtomicAdd(&sum[0][l], r.x[0]);
        unsafeAtomicAdd(&sum[ND - 2][l], r.x[1]);
        unsafeAtomicAdd(&sum[ND - 1][l], r.x[2]);
      }
    }
    if constexpr (BLK) {
#pragma unroll
      for (int k = 0; k < 3; ++k) unsafeAtomicAdd(&sum[NA - 3 + k][l], rec2[3 * at + k]);
    }
  };
  for (int c0 = wave * 64; c0 < n_chunks; c0 += W * 64) {
    const int c = c0 + lane;
    uint32_t i0 = 0, n = 0;
    if (c < n_chunks) {
      const uint16_t* q = off + (int64_t)c * (B + 1) + b;
      i0 = q[0];
      n = q[1] - i0;
    }
    uint32_t incl = n;
    for (int d = 1; d < 64; d <<= 1) {
      const uint32_t o = __shfl_up(incl, d, 64);
      if (lane >= d) incl += o;
    }
    const uint32_t total = __shfl(incl, 63, 64);
    seg_start[wave][lane] = incl - n;
    seg_at[wave][lane] = (uint32_t)c * (uint32_t)chunk + i0 - (incl - n);  // record k of the list at seg_at + k
    __builtin_amdgcn_wave_barrier();
    for (uint32_t k0 = lane; k0 < total; k0 += 64 * U) {
      uint32_t at[U];
      Rec r[U];
#pragma unroll
      for (int u = 0; u < U; ++u) {
        const uint32_t k = k0 + 64 * u;
        int sg = 0;
#pragma unroll
        for (int d = 32; d > 0; d >>= 1)
          if (seg_start[wave][sg + d] <= k) sg += d;
        at[u] = seg_at[wave][sg] + k;
        if (k < total) r[u] = rec[at[u]];
      }
#pragma unroll
      for (int u = 0; u < U; ++u)
        if (k0 + 64 * u < total) add(r[u], at[u]);
    }
    __builtin_amdgcn_wave_barrier();
  }
  __syncthreads();
  for (int h = log_c - 1; h >= 0; --h) {
    for (int i = threadIdx.x; i < n_local << h; i += kSumBlock) {
      const int to = (i >> h << log_c) + (i & ((1 << h) - 1)), from = to + (1 << h);
      const uint32_t x = hits[to], y = hits[from];
      hits[to] = ((x & ~kBadAngle) + (y & ~kBadAngle)) | ((x | y) & kBadAngle);
#pragma unroll
      for (int k = 0; k < NA; ++k) sum[k][to] += sum[k][from];
    }
    __syncthreads();
  }
  for (int pl = threadIdx.x; pl < n_local; pl += kSumBlock) {
    const int l = pl << log_c;
    if (!last) {
      acc_hits[(int64_t)b * n_local + pl] = hits[l];
#pragma unroll
      for (int k = 0; k < NA; ++k) acc[((int64_t)b * NA + k) * n_local + pl] = sum[k][l];
      continue;
    }
    const int64_t p = ((int64_t)(((uint32_t)pl >> log_g) << log_b | (uint32_t)b) << log_g) | (pl & ((1 << log_g) - 1));
    if (p >= v.n_pix) continue;
    const int h = (int)(hits[l] & ~kBadAngle);
    uint8_t f = 0;
    double inv[4] = {0.0, 0.0, 0.0, 0.0};
    const double mII = HT ? v.w[0] * (double)h : 0.0;
    if (HT && h > 0) {
      f |= 1;
      inv[0] = 1.0 / mII;
    }
    double a = 0.0, c = 0.0, d = 0.0;
    if constexpr (HQ) {
      if constexpr (BLK) {
        a = sum[NA - 3][l];
        c = sum[NA - 2][l];
        d = sum[NA - 1][l];
      } else {
        a = d = v.w[1] * (double)h;
        if (hits[l] & kBadAngle) a = c = d = NAN;
      }
      if (h > 0 && qu_block_inverse(a, c, d, rcond_cut, inv + 1)) f |= 2;
    }
    double s[3] = {0.0, 0.0, 0.0};
    if constexpr (DATA) {
      if (HT && (f & 1)) s[0] = sum[0][l];
      if (HQ && (f & 2)) {
        s[1] = sum[ND - 2][l];
        s[2] = sum[ND - 1][l];
      }
    }
    const double m[3] = {inv[0] * s[0], inv[1] * s[1] + inv[2] * s[2], inv[2] * s[1] + inv[3] * s[2]};
    if (o.hits) o.hits[p] = h;
    if (o.valid) o.valid[p] = f;
    if (o.blocks) {
      o.blocks[4 * p + 0] = mII;
      o.blocks[4 * p + 1] = a;
      o.blocks[4 * p + 2] = c;
      o.blocks[4 * p + 3] = d;
    }
    if (o.sum3) {
#pragma unroll
      for (int k = 0; k < 3; ++k) o.sum3[3 * p + k] = s[k];
    }
    if (o.map3) {
#pragma unroll
      for (int k = 0; k < 3; ++k) o.map3[3 * p + k] = m[k];
    }
    if (o.map4) {
      double2* mp = reinterpret_cast<double2*>(o.map4 + 4 * p);
      mp[0] = make_double2(m[0], m[1]);
      mp[1] = make_double2(m[2], 0.0);
    }
  }
}

// Buckets, pixels dealt together, and pixels of each bucket.  Groups of 64 keep
// a scan's neighbours together, and a cache line of the outputs in one workgroup;
// smaller ones (fine) give every bucket of a coarse map some pixels.
struct Deal {
  int log_b, log_g, n_local;
};
Deal deal(int64_t n_pix, bool blk, bool fine) {
  Deal d;
  d.log_g = kMaxLogG;
  while (fine && d.log_g > 0 && (n_pix + ((int64_t)1 << d.log_g) - 1) >> d.log_g < (int64_t)1 << kMinLogB) --d.log_g;
  const int64_t n_groups = (n_pix + ((int64_t)1 << d.log_g) - 1) >> d.log_g;
  auto local = [&]() { return (n_groups + ((int64_t)1 << d.log_b) - 1) >> d.log_b << d.log_g; };
  d.log_b = kMinLogB;
  while (local() > bucket_pix(blk)) ++d.log_b;
  d.n_local = (int)local();
  return d;
}
bool fits(int64_t n_pix, bool blk) { return n_pix <= (int64_t)bucket_pix(blk) << kMaxLogB; }

// Samples per chunk: the records a chunk is writing at a time (all its
// buckets') should stay in L2, which favours short chunks; the segments of
// k_bucket_sum get longer with it.  30 days at N_side 256: 1.79 ms with
// 1024, 1.71 with 2048, 1.87 with 4096, 2.2 with 16384.  Short timelines
// take the smaller chunk to have more workgroups.
constexpr int64_t kChunk = 2048, kShortChunk = 1024;

struct Shape {
  int log_b, log_g, log_c, n_local;
  int64_t chunk, n_chunks;  // samples per chunk, chunks of the timeline
  int n_data, n_blk;        // data and block sums per record
  size_t rec_bytes;
};

Shape shape_of(const View& v, bool data) {
  Shape s;
  // Fine from 256 samples per pixel on: 3072 pixels, a thousand samples 33 us with
  // groups of 64 and 35 with finer ones, 10 M samples 216 and 190.
  const Deal d = deal(v.n_pix, has_blocks(v), v.n_t >> 8 >= v.n_pix);
  s.log_b = d.log_b;
  s.log_g = d.log_g;
  s.n_local = d.n_local;
  s.log_c = 0;
  // Copies: one place per thread at most, and 16 samples per place (a thousand
  // samples 33.7 us with all copies, 31.5 with one; 100,000 of 192 pixels 34 and
  // 74 us).
  while (s.log_c < kMaxLogC && s.n_local << (s.log_c + 1) <= kSumBlock && v.n_pix << (s.log_c + 5) <= v.n_t) ++s.log_c;
  s.chunk = v.n_t >= (int64_t)1 << 22 ? kChunk : kShortChunk;
  s.n_chunks = (v.n_t + s.chunk - 1) / s.chunk;
  const bool ht = v.rowT >= 0, hq = v.rowQ >= 0;
  s.n_data = data ? (ht ? 1 : 0) + (hq ? 2 : 0) : 0;
  s.n_blk = has_blocks(v) ? 3 : 0;
  s.rec_bytes = !data ? sizeof(uint32_t) : (hq ? sizeof(Rec3) : sizeof(Rec1));
  return s;
}

template <typename F>
void by_bool(bool b, F&& f) {
  if (b)
    f(std::true_type{});
  else
    f(std::false_type{});
}

}  // namespace

bool buckets_fit(const View& v) { return fits(v.n_pix, has_blocks(v)); }
bool buckets_fit_any(int64_t n_pix) { return fits(n_pix, true); }

BucketBytes bucket_bytes(const View& v, bool data) {
  const Shape s = shape_of(v, data);
  BucketBytes b;
  b.off = (((size_t)1 << s.log_b) + 1) * sizeof(uint16_t);
  b.rec = (size_t)s.chunk * s.rec_bytes;
  b.rec2 = (size_t)s.chunk * s.n_blk * sizeof(double);
  const size_t px = (size_t)s.n_local << s.log_b;
  b.acc_hits = px * sizeof(uint32_t);
  b.acc = px * (s.n_data + s.n_blk) * sizeof(double);
  b.n_chunks = s.n_chunks;
  b.best_chunks = std::min(s.n_chunks, kPiece / s.chunk);
  return b;
}

BucketReserve bucket_reserve(int64_t n_pix) {
  // One record per pixel in a piece: carrying the sums from piece to piece then
  // moves no more than the records do.
  const int64_t samples = std::max<int64_t>((int64_t)1 << 19, n_pix);
  const size_t chunks = (size_t)((samples + kShortChunk - 1) / kShortChunk);
  BucketReserve r{};
  r.rec = chunks * kShortChunk * sizeof(Rec3);
  r.rec2 = chunks * kShortChunk * 3 * sizeof(double);
  for (bool blk : {false, true}) {
    if (!fits(n_pix, blk)) continue;
    for (bool fine : {false, true}) {
      const Deal d = deal(n_pix, blk, fine);
      const size_t px = (size_t)d.n_local << d.log_b;
      r.off = std::max(r.off, chunks * (((size_t)1 << d.log_b) + 1) * sizeof(uint16_t));
      r.acc_hits = std::max(r.acc_hits, px * sizeof(uint32_t));
      r.acc = std::max(r.acc, px * (blk ? 6 : 3) * sizeof(double));
    }
  }
  return r;
}

hipError_t launch_buckets(const View& v, int psi_f32, const void* tod, int tod_f32, const double* base, double bsign,
                          double rcond_cut, const BucketWork& W, const BucketOut& o, int* err, hipStream_t st) {
  const bool data = tod != nullptr || base != nullptr;
  const Shape s = shape_of(v, data);
  const bool eq = !has_blocks(v);
  for (int64_t c0 = 0; c0 < s.n_chunks; c0 += W.n_chunks) {
    const int n_chunks = (int)std::min(W.n_chunks, s.n_chunks - c0);
    const int64_t t0 = c0 * s.chunk, t1 = std::min(v.n_t, t0 + n_chunks * s.chunk);
    const int first = c0 == 0, last = t1 == v.n_t;
    by_bool(v.rowT >= 0, [&](auto T) {
      by_bool(v.rowQ >= 0, [&](auto Q) {
        by_bool(data, [&](auto D) {
          by_bool(eq, [&](auto E) {
            constexpr bool HT = decltype(T)::value, HQ = decltype(Q)::value, DA = decltype(D)::value,
                           EQ = decltype(E)::value;
            if constexpr ((HT || HQ) && (HQ || EQ)) {
              using Rec = typename RecOf<HQ, DA>::type;
              auto fill = [&](auto pt, auto tt) {
                using PT = decltype(pt);
                using TT = decltype(tt);
                hipLaunchKernelGGL((k_bucket_fill<PT, TT, HT, HQ, DA, EQ>), dim3(n_chunks), dim3(kBlock), 0, st, v,
                                   static_cast<const TT*>(tod), base, bsign, t0, t1, s.chunk, s.log_b, s.log_g, W.off,
                                   static_cast<Rec*>(W.rec), W.rec2, err);
              };
              const bool pf = HQ && psi_f32, tf = DA && tod_f32;
              if (pf && tf)
                fill(float{}, float{});
              else if (pf)
                fill(float{}, double{});
              else if (tf)
                fill(double{}, float{});
              else
                fill(double{}, double{});
              hipLaunchKernelGGL((k_bucket_sum<HT, HQ, DA, EQ>), dim3(1u << s.log_b), dim3(kSumBlock), 0, st, v,
                                 rcond_cut, W.off, static_cast<const Rec*>(W.rec), W.rec2, n_chunks, s.chunk, s.log_b,
                                 s.log_g, s.log_c, s.n_local, first, last, W.acc_hits, W.acc, o);
            }
          });
        });
      });
    });
  }
  return hipGetLastError();
}

}  // namespace dst
