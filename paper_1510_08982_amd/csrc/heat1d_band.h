// heat1d_band.h -- T steps of Eq.3 applied at once, as a banded matrix on the
// matrix cores (host-side declarations; the kernels are in kernels_band.hip).
//
// T steps of Eq.3 (Section 2) are one linear map: away from the ends every
// point becomes sum_d w_d u_{i+d}, w the coefficients of the T-th power of the
// three-point stencil (r, 1-2r, r).  Those coefficients are the distribution
// of a sum of T independent moves of -1, 0, +1, so they fall off like a
// Gaussian of variance 2 r T: beyond a reach of about 6.3 (FP32) or 9 (FP64)
// standard deviations all of them together are below a sixteenth of a
// rounding of the state.  One pass therefore costs 2 reach + 1 multiply-adds
// per point whatever T is, where stepping costs three instructions per step.
// The Dirichlet ends are exact under the odd extension of the rod about its
// ends (u(-i) = 2 c1 - u(i)), which every step preserves.
#pragma once

#include <hip/hip_runtime.h>
#include <stddef.h>
#include <stdint.h>

namespace heat1d {

// The largest reach of one pass: the tile with its halos and the weights stay
// within the LDS of a workgroup.  Longer runs take several equal passes.
constexpr int kBandMaxReach = 2048;

// Points beyond which the weights of T steps are dropped (at most T): the
// dropped weights sum to at most 2^-28 (FP32) / 2^-57 (FP64).
int band_reach(int dtype, double r, int64_t T);
// The same from a bound that grows with r and with T, and which band_reach never
// exceeds: what room for any r has to be sized for.  (It drops less, 2^-33 and
// 2^-64 at most: runs of many short passes use it.)
int band_reach_bound(int dtype, double r, int64_t T);

// What K steps take off the slowest mode of a Dirichlet rod of N points less its
// ends' line, as a power of e.  (A ring's mean stays; 0.)
__host__ __device__ inline double band_decay(double r, double K, int64_t N, bool ring) {
  return ring ? 0.0 : 9.869604401089358 * r * K / ((double)(N - 1) * (double)(N - 1));
}

// A pass is off by a rounding of the state it reads, whatever it leaves of it, so
// one of a short rod between zero ends (or a gradient's, which always has them) is
// off by e^decay roundings of its result: N = 30, r = 1/2, decay 1 / 4 / 10 / 20: FP64
// 6e-15, 2e-13, 5e-11, 1e-6, FP32 1.4e-6, 3e-5, 8e-3, 130, where steps, which lose a
// little of a little, stay at 2e-15 and 1e-6.  No pass takes off more than this:
// cut so, decays of 2 to 20 come out within 2e-15 to 2e-14 and 4e-7.
constexpr double kBandDecay = 0.6;
// A run of more than this keeps stepping: its passes' errors add up (FP64, N = 100,
// decay 63: 9e-14).
constexpr double kBandDecayRun = 64.0;

// How a run of K steps of N points is cut into passes of at most T steps each.
struct BandRun {
  int64_t passes = 0;
  int64_t T = 0;  // steps of every pass but the last, which takes the rest
};
BandRun band_run(int dtype, double r, int64_t K, int64_t N, bool ring);

constexpr size_t kBandWeightBytes = ((size_t)2 * (kBandMaxReach + 1) * 8 + 16 + 255) / 256 * 256;

// Bytes of scratch (256-byte aligned) of the passes over nrods rods of N points:
// two sets of weights, the flags and a record per tile.
size_t band_scratch_bytes(int64_t N, int64_t nrods);

// One pass of T steps of nrods rods of N points, in -> out.
struct BandPass {
  int dtype = 0;
  const void* in = nullptr;
  void* out = nullptr;
  int64_t N = 0, nrods = 1;
  int64_t T = 0;
  double r = 0, c1 = 0, cN = 0;
  int ring = 0;
  void* scratch = nullptr;
  int slot = 0;        // passes of one run alternate 0, 1 (whose flag is in use)
  int32_t* flag = nullptr;  // raise this flag instead, and keep no records: the
                            // caller does without launch_band_cones, and scratch
                            // needs kBandWeightBytes only
  // z, when not NULL (FP64 only), receives D A^(T-1) applied to the state (D the
  // second difference): K z is du(K)/dr, see heat1d_backward_checkpointed
  void* z = nullptr;
  // dot, when not NULL: dot_scale times the sum of in . dot_with over each
  // tile's inner points, one double per tile (band_tiles per rod)
  const void* dot_with = nullptr;
  double* dot = nullptr;
  double dot_scale = 1.0;
};
bool band_applies(int dtype, int64_t N, int64_t nrods);
int64_t band_tiles(int dtype, int64_t N, int64_t nrods);  // tiles per rod
hipError_t launch_band_weights(const BandPass& p, hipStream_t s);
hipError_t launch_band_pass(const BandPass& p, hipStream_t s);
hipError_t launch_band_cones(const BandPass& p, hipStream_t s);

// What the tiles of a rod need of it, gathered by the workgroup that computes its
// weights: a tile then waits for two loads in turn before its first point, not five.
struct BandSlot {
  int64_t off, N;
  double c1, cN;
  int32_t H, woff;  // H < 0: the rod is stepped
};
constexpr size_t kBandSlotBytes = sizeof(BandSlot);

// Rods of uneven length, step count and r: tiles of kBandBatchTile points, one
// workgroup each.  A rod that decays by more than kBandDecay, which is known when
// its r is, has kBandBatchStep points at most and is stepped by a wavefront.  All pointers are device memory.
constexpr int kBandBatchTile = 2048;
constexpr int kBandBatchStep = 512;
struct BandItem {
  int32_t slot;  // index into rods / woff
  int32_t tile;
};
struct BandBatch {
  int dtype = 0;
  const void* in = nullptr;
  void* out = nullptr;
  const int64_t* offsets = nullptr;
  const double* r = nullptr;
  const double* c1 = nullptr;
  const double* cN = nullptr;
  const int32_t* K = nullptr;
  const BandItem* items = nullptr;  // a rod's tiles one after the other
  const int32_t* rods = nullptr;    // of each slot
  void* slot = nullptr;             // slots x kBandSlotBytes, written by the run
  const int32_t* woff = nullptr;    // slots + 1: where a slot's weights start
  void* w = nullptr;
  int32_t* flag = nullptr;
  void* rec = nullptr;              // 8 bytes per item
  int32_t nitems = 0, nslots = 0;
  int32_t hmax = 0;                 // the longest reach that woff leaves room for
  bool short_rods = false;          // some rod may decay by more than kBandDecay
};
hipError_t launch_band_batch(const BandBatch& b, hipStream_t s);

}  // namespace heat1d
