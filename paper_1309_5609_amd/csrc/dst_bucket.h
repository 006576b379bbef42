// One-shot binning by pixel buckets (no global atomics).
#pragma once

#include <hip/hip_runtime.h>

#include <cstdint>

#include "dst_internal.h"

namespace dst {

// Outputs per pixel, any may be NULL: hits, blocks [n_pix][4] (M_II, M_QQ,
// M_QU, M_UU), validity bits, sums [n_pix][3], map M^-1 s [n_pix][3] or
// [n_pix][4].
struct BucketOut {
  int32_t* hits = nullptr;
  double* blocks = nullptr;
  uint8_t* valid = nullptr;
  double* sum3 = nullptr;
  double* map3 = nullptr;
  double* map4 = nullptr;
};

// Work arrays.  The timeline is taken in pieces of n_chunks chunks whose
// records are held at once; acc_hits and acc carry the sums between pieces.
struct BucketWork {
  uint16_t* off = nullptr;
  void* rec = nullptr;
  double* rec2 = nullptr;
  uint32_t* acc_hits = nullptr;
  double* acc = nullptr;
  int64_t n_chunks = 0;
};
// Their sizes in bytes: off, rec, rec2 per chunk; acc_hits, acc in all (read by
// a timeline of several pieces only); the chunks of the whole timeline, and the
// most that are worth holding at once.
struct BucketBytes {
  size_t off, rec, rec2, acc_hits, acc;
  int64_t n_chunks, best_chunks;
};

// Whether the map is small enough for the bucket form (a full N_side 512 sky;
// twice that with equal q/u weights), and whether it is with any weights.
bool buckets_fit(const View& v);
bool buckets_fit_any(int64_t n_pix);
BucketBytes bucket_bytes(const View& v, bool data);
// Sizes in bytes with which any timeline, streams, weights and dtypes on a map
// of up to n_pix pixels (buckets_fit_any) can be binned, in pieces: about 110
// bytes a pixel and 30 MB at least.  Pieces of 2^19 samples, or one per pixel.
struct BucketReserve {
  size_t off, rec, rec2, acc_hits, acc;
};
BucketReserve bucket_reserve(int64_t n_pix);
// s = A^T W x over valid samples, x = tod + bsign F base (either may be NULL;
// both NULL: hits, blocks and validity only).
hipError_t launch_buckets(const View& v, int psi_f32, const void* tod, int tod_f32, const double* base, double bsign,
                          double rcond_cut, const BucketWork& W, const BucketOut& o, int* err, hipStream_t st);

}  // namespace dst
