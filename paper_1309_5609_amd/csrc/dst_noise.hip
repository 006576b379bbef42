// Monte Carlo noise on the GPU: white + 1/f timelines with the spectrum of
// Eq. 1 of arXiv:1309.5609, made by filtering white noise in the Fourier
// domain, segment by segment.
//
// * Random bits: Philox4x64-10 (Salmon, Moraes, Dror & Shaw, SC 2011), a
//   counter-based generator: block b of segment j of a stream is the
//   function of counter (b, j, 0, 0) and key (seed, stream), so any sample
//   can be drawn by any thread with no state.
// * Normals: Box-Muller on the top 53 bits of two words,
//   u1 in (0, 1], u2 in [0, 1): sqrt(-2 ln u1) (cos 2 pi u2, sin 2 pi u2).
// * Filter: segments of S = 2^m samples; two real segments travel as the real
//   and imaginary parts of one complex transform (the gain is real and even
//   in frequency, so it acts on each part separately): forward transform, gain
//   sqrt(1 + (f_k / |f|)^alpha) with the zero-frequency bin kept, inverse
//   transform, 1/S.  The last segment is drawn at full length and cut.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cmath>
#include <cstdint>
#include <type_traits>

#include "dst_internal.h"

namespace dst {
namespace {

constexpr uint64_t kM0 = 0xD2E7470EE14C6C93ull, kM1 = 0xCA5A826395121157ull;
constexpr uint64_t kW0 = 0x9E3779B97F4A7C15ull, kW1 = 0xBB67AE8584CAA73Bull;

__device__ __forceinline__ void philox4x64_10(uint64_t (&x)[4], uint64_t k0, uint64_t k1) {
#pragma unroll
  for (int r = 0; r < 10; ++r) {
    if (r > 0) {
      k0 += kW0;
      k1 += kW1;
    }
    const uint64_t hi0 = __umul64hi(kM0, x[0]), lo0 = kM0 * x[0];
    const uint64_t hi1 = __umul64hi(kM1, x[2]), lo1 = kM1 * x[2];
    const uint64_t y0 = hi1 ^ x[1] ^ k0, y2 = hi0 ^ x[3] ^ k1;
    x[0] = y0;
    x[1] = lo1;
    x[2] = y2;
    x[3] = lo0;
  }
}

// Four unit normals of block b of segment seg.
__device__ __forceinline__ void normals4(uint64_t seed, uint64_t stream, uint64_t seg, uint64_t b, double (&z)[4]) {
  uint64_t x[4] = {b, seg, 0ull, 0ull};
  philox4x64_10(x, seed, stream);
  const double scale = 1.1102230246251565e-16;  // 2^-53
#pragma unroll
  for (int p = 0; p < 2; ++p) {
    const double u1 = ((double)(x[2 * p] >> 11) + 1.0) * scale;
    const double u2 = (double)(x[2 * p + 1] >> 11) * scale;
    const double r = sqrt(-2.0 * log(u1));
    double s, c;
    sincos((2.0 * M_PI) * u2, &s, &c);
    z[2 * p] = r * c;
    z[2 * p + 1] = r * s;
  }
}

__device__ __forceinline__ double2 cmul(double2 a, double2 b) {
  return make_double2(a.x * b.x - a.y * b.y, a.x * b.y + a.y * b.x);
}
__device__ __forceinline__ double2 cadd(double2 a, double2 b) { return make_double2(a.x + b.x, a.y + b.y); }
__device__ __forceinline__ double2 csub(double2 a, double2 b) { return make_double2(a.x - b.x, a.y - b.y); }

// ---------------------------------------------------------------- FFT
// In place, in tiles of kElems values held by one workgroup, kPer per thread.
//
// S = R_1 .. R_P C.  Forward, pass p takes every block of length S' = S / (R_1
// .. R_{p-1}) as R = R_p rows of M = S' / R values: the columns' length-R
// transforms, times w_S'^(k q) (column k, row q), stored where they were, so
// that row q is the next pass's block.  The blocks of C contiguous values left
// at the end are transformed whole; bin f = q_1 + R_1 (q_2 + R_2 f') of the
// spectrum sits at place f' of block (q_1, q_2).  The gain is applied there,
// and the inverse transform undoes the passes in the opposite order, so the
// spectrum is never brought into order.  Nothing is stored between drawing
// the normals and the first pass, around the gain, or between the last pass
// and the output: for segments of 2^13 to 2^22 samples a value moves through
// memory five times (three kernels, 80 bytes per complex value with the
// output), up to 2^12 not at all.  (Separate kernels for normals, three passes
// each way between two buffers, and output moved 240 bytes.)  43 M samples
// accumulated, before and now: segments of 2^17 (FP32) 1.49 and 0.61 ms, 2^20
// 1.60 and 0.70, 2^22 2.06 and 0.96; 130 M samples in segments of 2^24 5.9 and
// 2.7 ms.  The first kernel is bound by the generator's integer and FP64
// operations, the others by memory traffic.
//
// Inside a tile: self-sorting stages of radix 8 (and one of 2 or 4) between
// LDS exchanges, the first from and the last to registers.
constexpr int kLogElems = 12;
constexpr int kElems = 1 << kLogElems;  // complex values per workgroup
constexpr int kThreads = 512;
constexpr int kPer = kElems / kThreads;
// Complex values of the buffer (512 MiB): 43 M samples in segments of 2^22 take
// 0.93 ms; with a quarter, which stays in the last-level cache, 1.08 (shorter
// launches), with twice as many 0.93.
constexpr int kLogChunk = 25;
// Largest radix of a column pass: 4 columns (64 bytes) side by side, of which
// the neighbouring tile completes the cache lines.  Segments of 2^22 take 0.93
// ms with one pass of 2^10 and 1.1 with two of 2^5.
constexpr int kLogCol = 10;
static_assert(kPer == 8, "one radix-8 butterfly per thread");

// LDS place of value i of a tile: one value of padding after every eight, so
// that the strided writes of a stage spread over the banks.
__device__ __forceinline__ int pad(int i) { return i + (i >> 3); }
constexpr int kLds = kElems + kElems / 8;

// exp(-2 pi i E / S) from two tables: hi[a] = exp(-2 pi i a 2^h / S), lo[b] =
// exp(-2 pi i b / S); W[i] = exp(-2 pi i i / kElems) serves the tiles.
struct Twiddles {
  const double2* hi;
  const double2* lo;
  const double2* W;
  int h;
  int64_t S;
};
__device__ __forceinline__ double2 twiddle(const Twiddles& t, uint32_t E) {
  E &= (uint32_t)t.S - 1u;
  return cmul(t.hi[E >> t.h], t.lo[E & ((1u << t.h) - 1u)]);
}
template <int DIR>
__device__ __forceinline__ double2 toward(double2 w) {
  return DIR < 0 ? w : make_double2(w.x, -w.y);
}

__global__ void __launch_bounds__(256) k_twiddles(double2* __restrict__ hi, double2* __restrict__ lo,
                                                  double2* __restrict__ W, int h, int m) {
  const int nh = 1 << (m - h), nl = 1 << h;
  for (int i = (int)(blockIdx.x * blockDim.x + threadIdx.x); i < nh + nl + kElems; i += (int)(gridDim.x * blockDim.x)) {
    // angle -2 pi x as sincospi of -2x (exact arguments)
    const double x = i < nh ? (double)i / (double)nh
                            : (i < nh + nl ? (double)(i - nh) / ((double)nh * (double)nl)
                                           : (double)(i - nh - nl) / (double)kElems);
    double s, c;
    sincospi(-2.0 * x, &s, &c);
    (i < nh ? hi[i] : (i < nh + nl ? lo[i - nh] : W[i - nh - nl])) = make_double2(c, s);
  }
}

// w[q] = w_S^(b + q e) (DIR < 0) or its conjugate, from table entries for b, e,
// 2 e and 4 e, at most three products deep.
template <int RAD, int DIR>
__device__ __forceinline__ void powers(const Twiddles& t, uint32_t b, uint32_t e, double2 (&w)[RAD]) {
  w[0] = toward<DIR>(twiddle(t, b));
  w[1] = cmul(w[0], toward<DIR>(twiddle(t, e)));
  if constexpr (RAD >= 4) {
    const double2 s2 = toward<DIR>(twiddle(t, 2 * e));
    w[2] = cmul(w[0], s2);
    w[3] = cmul(w[1], s2);
    if constexpr (RAD == 8) {
      const double2 s4 = toward<DIR>(twiddle(t, 4 * e));
#pragma unroll
      for (int q = 0; q < 4; ++q) w[4 + q] = cmul(w[q], s4);
    }
  }
}

template <int DIR>
__device__ __forceinline__ double2 times_i(double2 a) {  // DIR i a
  return DIR < 0 ? make_double2(a.y, -a.x) : make_double2(-a.y, a.x);
}
template <int RAD, int DIR>
__device__ __forceinline__ void butterfly(double2* v) {
  if constexpr (RAD == 2) {
    const double2 a = v[0];
    v[0] = cadd(a, v[1]);
    v[1] = csub(a, v[1]);
  } else if constexpr (RAD == 4) {
    const double2 t0 = cadd(v[0], v[2]), t1 = csub(v[0], v[2]);
    const double2 t2 = cadd(v[1], v[3]), t3 = times_i<DIR>(csub(v[1], v[3]));
    v[0] = cadd(t0, t2);
    v[1] = cadd(t1, t3);
    v[2] = csub(t0, t2);
    v[3] = csub(t1, t3);
  } else {
    double2 a[4] = {v[0], v[2], v[4], v[6]}, b[4] = {v[1], v[3], v[5], v[7]};
    butterfly<4, DIR>(a);
    butterfly<4, DIR>(b);
    constexpr double h = 0.70710678118654752440;
    const double2 i1 = times_i<DIR>(b[1]), i3 = times_i<DIR>(b[3]);
    b[1] = make_double2(h * (b[1].x + i1.x), h * (b[1].y + i1.y));
    b[2] = times_i<DIR>(b[2]);
    b[3] = make_double2(h * (i3.x - b[3].x), h * (i3.y - b[3].y));
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      v[q] = cadd(a[q], b[q]);
      v[q + 4] = csub(a[q], b[q]);
    }
  }
}

// Stage of span 2^LOGNS of a length-2^LOGR transform in direction DIR: its log
// radix.  The odd stage comes first forward and last backward, so that the
// forward transform ends, and the backward one starts, with the same radix.
template <int LOGR, int DIR>
__host__ __device__ constexpr int log_radix(int log_ns) {
  return LOGR < 3 ? LOGR
                  : (DIR < 0 ? (log_ns == 0 && LOGR % 3 ? LOGR % 3 : 3) : (LOGR - log_ns >= 3 ? 3 : LOGR - log_ns));
}

// Transforms of the tile's 2^(kLogElems - LOGR) columns.  Thread values v[i
// RAD + q]: butterfly i = column c, j with (c, j) = column(i) holds rows j + q
// R / RAD on entry (RAD of the first stage) and on return (of the last).
template <int LOGR>
__device__ __forceinline__ void column(int i, int& c, int& j) {
  const int idx = (int)threadIdx.x + kThreads * i;
  c = idx & ((kElems >> LOGR) - 1);
  j = idx >> (kLogElems - LOGR);
}
template <int LOGR, int DIR, int LOGNS = 0>
__device__ __forceinline__ void fft_tile(double2 (&v)[kPer], double2* L, const double2* __restrict__ W) {
  constexpr int LR = log_radix<LOGR, DIR>(LOGNS), RAD = 1 << LR, LOGTC = kLogElems - LOGR;
#pragma unroll
  for (int i = 0; i < kPer / RAD; ++i) {
    int c, j;
    column<LOGR>(i, c, j);
    if constexpr (LOGNS > 0) {
      // powers s^q of the butterfly's factor: 1, 2 and 4 from the table, the
      // others at most two products deep (table entries for all seven: errors 4.78e-16
      // for 4.94e-16 of the RMS at 512 points, but 43 M samples in segments of 4096
      // 0.82 ms for 0.46)
      const int e = (j & ((1 << LOGNS) - 1)) << (kLogElems - LR - LOGNS);
      double2 w[8];
      w[1] = toward<DIR>(W[e]);
      if constexpr (RAD >= 4) {
        w[2] = toward<DIR>(W[2 * e]);
        w[3] = cmul(w[2], w[1]);
      }
      if constexpr (RAD == 8) {
        w[4] = toward<DIR>(W[4 * e]);
#pragma unroll
        for (int q = 1; q < 4; ++q) w[4 + q] = cmul(w[4], w[q]);
      }
#pragma unroll
      for (int q = 1; q < RAD; ++q) v[i * RAD + q] = cmul(v[i * RAD + q], w[q]);
    }
    butterfly<RAD, DIR>(v + i * RAD);
  }
  if constexpr (LOGNS + LR < LOGR) {
    constexpr int LR2 = log_radix<LOGR, DIR>(LOGNS + LR), RAD2 = 1 << LR2;
    __syncthreads();  // the values of the exchange before are read
#pragma unroll
    for (int i = 0; i < kPer / RAD; ++i) {
      int c, j;
      column<LOGR>(i, c, j);
      const int row = ((j >> LOGNS) << (LOGNS + LR)) + (j & ((1 << LOGNS) - 1));
#pragma unroll
      for (int q = 0; q < RAD; ++q) L[pad(((row + (q << LOGNS)) << LOGTC) + c)] = v[i * RAD + q];
    }
    __syncthreads();
#pragma unroll
    for (int i = 0; i < kPer / RAD2; ++i) {
      int c, j;
      column<LOGR>(i, c, j);
#pragma unroll
      for (int q = 0; q < RAD2; ++q) v[i * RAD2 + q] = L[pad(((j + (q << (LOGR - LR2))) << LOGTC) + c)];
    }
    fft_tile<LOGR, DIR, LOGNS + LR>(v, L, W);
  }
}

// What the first pass draws and the last pass writes.
struct Draw {
  uint64_t seed = 0, stream = 0;
  int64_t p0 = 0, n_seg = 0;  // first segment pair of the chunk, segments in all
  double sigma = 0.0;
};
struct Out {
  void* out = nullptr;
  int64_t n = 0;
  double inv_s = 0.0;
  int accumulate = 0;
};

// Normals 4 b .. 4 b + 3 of pair p (sigma times; imaginary part 0 past n_seg).
__device__ __forceinline__ void draw_pair(const Draw& d, int64_t p, int64_t b, double2 (&z)[4]) {
  const int64_t sa = 2 * (d.p0 + p), sb = sa + 1;
  double za[4], zb[4] = {0.0, 0.0, 0.0, 0.0};
  normals4(d.seed, d.stream, (uint64_t)sa, (uint64_t)b, za);
  if (sb < d.n_seg) normals4(d.seed, d.stream, (uint64_t)sb, (uint64_t)b, zb);
#pragma unroll
  for (int i = 0; i < 4; ++i) z[i] = make_double2(d.sigma * za[i], d.sigma * zb[i]);
}
// Value k of pair p to the timeline.
template <typename OT>
__device__ __forceinline__ void emit(const Out& o, const Draw& d, int64_t S, int64_t p, int64_t k, double2 v) {
  OT* out = static_cast<OT*>(o.out);
  const int64_t ta = 2 * (d.p0 + p) * S + k, tb = ta + S;
  if (ta < o.n) out[ta] = o.accumulate ? (OT)((double)out[ta] + v.x * o.inv_s) : (OT)(v.x * o.inv_s);
  if (tb < o.n) out[tb] = o.accumulate ? (OT)((double)out[tb] + v.y * o.inv_s) : (OT)(v.y * o.inv_s);
}

// Workgroups of one XCD (workgroup i runs on XCD i mod 8) take neighbouring
// tiles, whose rows share cache lines.
__device__ __forceinline__ int64_t tile_of(int64_t n) {
  const int64_t i = blockIdx.x;
  return n % 8 == 0 ? (i & 7) * (n / 8) + (i >> 3) : i;
}

// Column pass of radix 2^LOGR over blocks of length 2^log_s.  FIRST (forward):
// the values are drawn instead of read; LAST (backward): they go to the
// timeline instead.
enum { COL_READ = 0, COL_FIRST = 1, COL_LAST = 2 };
template <int LOGR, int DIR, int MODE, typename OT>
__global__ void __launch_bounds__(kThreads) k_columns(double2* __restrict__ x, int log_s, int64_t n_tiles, Twiddles tw,
                                                      Draw d, Out o) {
  constexpr int LOGTC = kLogElems - LOGR;
  constexpr int LR0 = log_radix<LOGR, DIR>(0), RAD0 = 1 << LR0;
  constexpr int LRZ = DIR < 0 ? log_radix<LOGR, DIR>(LOGR - log_radix<LOGR, 1>(0)) : (LOGR % 3 && LOGR > 3 ? LOGR % 3 : LR0);
  constexpr int RADZ = 1 << LRZ;
  __shared__ double2 L[kLds];
  const int log_m = log_s - LOGR;
  const int64_t g0 = tile_of(n_tiles) << LOGTC;  // first column
  const int64_t blk = g0 >> log_m;
  const uint32_t k0 = (uint32_t)(g0 & (((int64_t)1 << log_m) - 1));
  double2* base = x + (blk << log_s) + k0;
  const uint32_t unit = (uint32_t)(tw.S >> log_s);  // w_S' in units of w_S
  double2 v[kPer];
  if constexpr (MODE == COL_FIRST) {
#pragma unroll
    for (int t = 0; t < kElems / 4 / kThreads; ++t) {
      const int i = 4 * ((int)threadIdx.x + kThreads * t), row = i >> LOGTC, c = i & ((1 << LOGTC) - 1);
      double2 z[4];
      draw_pair(d, blk, (((int64_t)row << log_m) + k0 + c) >> 2, z);
#pragma unroll
      for (int k = 0; k < 4; ++k) L[pad(i + k)] = z[k];
    }
    __syncthreads();
  }
#pragma unroll
  for (int i = 0; i < kPer / RAD0; ++i) {
    int c, j;
    column<LOGR>(i, c, j);
#pragma unroll
    for (int q = 0; q < RAD0; ++q) {
      const int row = j + (q << (LOGR - LR0));
      v[i * RAD0 + q] = MODE == COL_FIRST ? L[pad((row << LOGTC) + c)] : base[((int64_t)row << log_m) + c];
    }
    if constexpr (DIR > 0) {  // undo the forward pass's factors
      const uint32_t k = (k0 + c) * unit;
      double2 w[RAD0];
      powers<RAD0, DIR>(tw, k * j, k << (LOGR - LR0), w);
#pragma unroll
      for (int q = 0; q < RAD0; ++q) v[i * RAD0 + q] = cmul(v[i * RAD0 + q], w[q]);
    }
  }
  fft_tile<LOGR, DIR>(v, L, tw.W);
#pragma unroll
  for (int i = 0; i < kPer / RADZ; ++i) {
    int c, j;
    column<LOGR>(i, c, j);
    if constexpr (DIR < 0) {
      const uint32_t k = (k0 + c) * unit;
      double2 w[RADZ];
      powers<RADZ, DIR>(tw, k * j, k << (LOGR - LRZ), w);
#pragma unroll
      for (int q = 0; q < RADZ; ++q) v[i * RADZ + q] = cmul(v[i * RADZ + q], w[q]);
    }
#pragma unroll
    for (int q = 0; q < RADZ; ++q) {
      const int64_t at = ((int64_t)(j + (q << (LOGR - LRZ))) << log_m) + c;
      if constexpr (MODE == COL_LAST)
        emit<OT>(o, d, tw.S, blk, k0 + at, v[i * RADZ + q]);
      else
        base[at] = v[i * RADZ + q];
    }
  }
}

// The gain of Eq. 1's filter at bin k of a length-S transform:
// sqrt(1 + (f_k / |f|)^alpha), 1 at zero frequency.
struct Gain {
  double fknee = 0.0, alpha = 0.0, df = 0.0;  // df: bin spacing (rate / S); fknee = 0: no filter
};
__device__ __forceinline__ double gain_at(const Gain& G, int64_t k, int64_t S) {
  const int64_t kk = k <= S / 2 ? k : S - k;
  if (kk == 0 || !(G.fknee > 0.0)) return 1.0;
  return sqrt(1.0 + pow(G.fknee / ((double)kk * G.df), G.alpha));
}

// Blocks of 2^LOGR contiguous values: forward transform, gain, backward
// transform.  WHOLE: the block is the whole segment (several pairs per tile),
// drawn here and written to the timeline; else one block (q_1, q_2) of every
// gridDim.y-th pair in turn, so that a thread's gains serve several pairs.
template <int LOGR, bool WHOLE, typename OT>
__global__ void __launch_bounds__(kThreads) k_blocks(double2* __restrict__ x, int log_s, int log_r1, int log_r2,
                                                     int64_t batch, Twiddles tw, Gain G, Draw d, Out o) {
  constexpr int LOGTC = kLogElems - LOGR;
  constexpr int LR = log_radix<LOGR, 1>(0), RAD = 1 << LR;  // last stage forward, first backward
  constexpr int LR0 = log_radix<LOGR, -1>(0), RAD0 = 1 << LR0;
  constexpr int LRZ = LOGR % 3 && LOGR > 3 ? LOGR % 3 : LR, RADZ = 1 << LRZ;
  static_assert(WHOLE || LOGR == kLogElems, "blocks of a longer segment fill a tile");
  __shared__ double2 L[kLds];
  const int64_t S = tw.S;
  const int64_t blk = blockIdx.x;  // WHOLE: tile of pairs
  // bin of place f' of the block: f0 + f' 2^(log_r1 + log_r2)
  const int64_t f0 = WHOLE ? 0 : (blk >> log_r2) + ((blk & (((int64_t)1 << log_r2) - 1)) << log_r1);
  double g[kPer];
  if constexpr (LOGR < kLogElems) {  // each bin's gain once
    double* bins = &L[0].x;
    for (int k = (int)threadIdx.x; k < 1 << LOGR; k += kThreads) bins[k] = gain_at(G, k, S);
    __syncthreads();
#pragma unroll
    for (int i = 0; i < kPer / RAD; ++i) {
      int c, j;
      column<LOGR>(i, c, j);
#pragma unroll
      for (int q = 0; q < RAD; ++q) g[i * RAD + q] = bins[j + (q << (LOGR - LR))];
    }
    __syncthreads();
  } else {
#pragma unroll
    for (int i = 0; i < kPer / RAD; ++i) {
      int c, j;
      column<LOGR>(i, c, j);
#pragma unroll
      for (int q = 0; q < RAD; ++q)
        g[i * RAD + q] = gain_at(G, f0 + ((int64_t)(j + (q << (LOGR - LR))) << (log_r1 + log_r2)), S);
    }
  }
  const int64_t first = WHOLE ? blk << LOGTC : blockIdx.y, step = WHOLE ? batch : gridDim.y;
  for (int64_t p = first; p < batch; p += step) {
    double2* base = x + (p << log_s) + (blk << LOGR);
    double2 v[kPer];
    if constexpr (WHOLE) {
      const int held = (int)min((int64_t)1 << LOGTC, batch - p);  // pairs of the tile
      if (held < 1 << LOGTC) {
        // the last tile, of a short timeline the only one: its segments' draws dealt to all threads, and every bin's
        // gain computed once (a thousand samples in segments of 64: a call 55 -> 32 us; 10 M in segments of 256: 137 -> 105)
        for (int i = (int)threadIdx.x; i < held << (LOGR - 1); i += kThreads) {
          const int c = i % held, h = i / held, b = h >> 1;
          const int64_t seg = 2 * (d.p0 + p + c) + (h & 1);
          double z[4] = {0.0, 0.0, 0.0, 0.0};
          if (seg < d.n_seg) normals4(d.seed, d.stream, (uint64_t)seg, (uint64_t)b, z);
#pragma unroll
          for (int k = 0; k < 4; ++k) {
            double2& to = L[pad(((4 * b + k) << LOGTC) + c)];
            (h & 1 ? to.y : to.x) = d.sigma * z[k];
          }
        }
      } else {
#pragma unroll
        for (int t = 0; t < kElems / 4 / kThreads; ++t) {
          const int i = (int)threadIdx.x + kThreads * t, c = i & ((1 << LOGTC) - 1), b = i >> LOGTC;
          double2 z[4];
          draw_pair(d, p + c, b, z);
#pragma unroll
          for (int k = 0; k < 4; ++k) L[pad(((4 * b + k) << LOGTC) + c)] = z[k];
        }
      }
      __syncthreads();
    }
#pragma unroll
    for (int i = 0; i < kPer / RAD0; ++i) {
      int c, j;
      column<LOGR>(i, c, j);
#pragma unroll
      for (int q = 0; q < RAD0; ++q) {
        const int row = j + (q << (LOGR - LR0));
        v[i * RAD0 + q] = WHOLE ? L[pad((row << LOGTC) + c)] : base[row];
      }
    }
    fft_tile<LOGR, -1>(v, L, tw.W);
#pragma unroll
    for (int k = 0; k < kPer; ++k) v[k] = make_double2(v[k].x * g[k], v[k].y * g[k]);
    fft_tile<LOGR, 1>(v, L, tw.W);
#pragma unroll
    for (int i = 0; i < kPer / RADZ; ++i) {
      int c, j;
      column<LOGR>(i, c, j);
#pragma unroll
      for (int q = 0; q < RADZ; ++q) {
        const int row = j + (q << (LOGR - LRZ));
        if constexpr (!WHOLE)
          base[row] = v[i * RADZ + q];
        else if (p + c < batch)
          emit<OT>(o, d, S, p + c, row, v[i * RADZ + q]);
      }
    }
  }
}

int log2_of(int64_t S) {
  int m = 0;
  while (((int64_t)1 << m) < S) ++m;
  return m;
}

// f(integral_constant<int, n>) for lo <= n <= hi.
template <int LO, int HI, typename F>
void by_int(int n, F&& f) {
  if constexpr (LO <= HI) {
    if (n == LO)
      f(std::integral_constant<int, LO>{});
    else
      by_int<LO + 1, HI>(n, f);
  }
}
template <typename F>
void by_type(int f32, F&& f) {
  if (f32)
    f(float{});
  else
    f(double{});
}

}  // namespace

int64_t noise_twiddle_count(int64_t S) {
  const int m = log2_of(S), h = (m + 1) / 2;
  return ((int64_t)1 << (m - h)) + ((int64_t)1 << h) + kElems;
}

// Pairs filtered at a time: 2^kLogChunk complex values at most, or one pair.
int64_t noise_pairs_per_chunk(int64_t S) {
  const int64_t cap = (int64_t)1 << kLogChunk;
  return S >= cap ? 1 : cap / S;
}

// The buffer holds whole segments only when they are longer than a tile.
int64_t noise_buffer_count(int64_t S) { return S <= kElems ? 1 : noise_pairs_per_chunk(S) * S; }

hipError_t launch_noise(uint64_t seed, uint64_t stream, int64_t n, int64_t S, double rate, double sigma, double fknee,
                        double alpha, void* out, int out_f32, int accumulate, double2* buf, double2* twbuf,
                        hipStream_t st) {
  if (S < 4 || (S & (S - 1))) return hipErrorInvalidValue;
  const int m = log2_of(S), h = (m + 1) / 2;
  Twiddles tw;
  double2 *hi = twbuf, *lo = hi + ((int64_t)1 << (m - h)), *W = lo + ((int64_t)1 << h);
  tw.hi = hi;
  tw.lo = lo;
  tw.W = W;
  tw.h = h;
  tw.S = S;
  hipLaunchKernelGGL(k_twiddles, dim3((unsigned)((noise_twiddle_count(S) + 255) / 256)), dim3(256), 0, st, hi, lo, W,
                     h, m);
  Gain gain;
  if (fknee > 0.0) {
    gain.fknee = fknee;
    gain.alpha = alpha;
    gain.df = rate / (double)S;
  }
  Draw d;
  d.seed = seed;
  d.stream = stream;
  d.n_seg = (n + S - 1) / S;
  d.sigma = sigma;
  Out o;
  o.out = out;
  o.n = n;
  o.inv_s = 1.0 / (double)S;
  o.accumulate = accumulate;
  const int64_t n_pairs = (d.n_seg + 1) / 2;
  if (m <= kLogElems) {
    const int64_t tiles = (n_pairs + (kElems >> m) - 1) / (kElems >> m);
    if (tiles > 0x7fffffff) return hipErrorInvalidValue;
    by_int<2, kLogElems>(m, [&](auto lr) {
      by_type(out_f32, [&](auto ot) {
        hipLaunchKernelGGL((k_blocks<decltype(lr)::value, true, decltype(ot)>), dim3((unsigned)tiles), dim3(kThreads),
                           0, st, nullptr, m, 0, 0, n_pairs, tw, gain, d, o);
      });
    });
    return hipGetLastError();
  }
  // column bits in one pass up to 2^kLogCol, else in two
  const int bits = m - kLogElems;
  const int r1 = bits <= kLogCol ? bits : (bits + 1) / 2, r2 = bits - r1;
  const int64_t chunk = noise_pairs_per_chunk(S);
  for (int64_t p0 = 0; p0 < n_pairs; p0 += chunk) {
    const int64_t np = n_pairs - p0 < chunk ? n_pairs - p0 : chunk;
    const int64_t tiles = np << (m - kLogElems);
    d.p0 = p0;
    by_int<1, kLogCol>(r1, [&](auto lr) {
      hipLaunchKernelGGL((k_columns<decltype(lr)::value, -1, COL_FIRST, double>), dim3((unsigned)tiles),
                         dim3(kThreads), 0, st, buf, m, tiles, tw, d, o);
    });
    if (r2 > 0)
      by_int<1, kLogCol>(r2, [&](auto lr) {
        hipLaunchKernelGGL((k_columns<decltype(lr)::value, -1, COL_READ, double>), dim3((unsigned)tiles),
                           dim3(kThreads), 0, st, buf, m - r1, tiles, tw, d, o);
      });
    // at least 2048 workgroups (two fit a CU), as far as there are pairs
    const unsigned split = (unsigned)std::min<int64_t>(np, bits < 11 ? 1 << (11 - bits) : 1);
    hipLaunchKernelGGL((k_blocks<kLogElems, false, double>), dim3(1u << bits, split), dim3(kThreads), 0, st, buf, m,
                       r1, r2, np, tw, gain, d, o);
    if (r2 > 0)
      by_int<1, kLogCol>(r2, [&](auto lr) {
        hipLaunchKernelGGL((k_columns<decltype(lr)::value, 1, COL_READ, double>), dim3((unsigned)tiles),
                           dim3(kThreads), 0, st, buf, m - r1, tiles, tw, d, o);
      });
    by_int<1, kLogCol>(r1, [&](auto lr) {
      by_type(out_f32, [&](auto ot) {
        hipLaunchKernelGGL((k_columns<decltype(lr)::value, 1, COL_LAST, decltype(ot)>), dim3((unsigned)tiles),
                           dim3(kThreads), 0, st, buf, m, tiles, tw, d, o);
      });
    });
    const hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
  }
  return hipSuccess;
}

}  // namespace dst
