// heat1d_strips.h -- the emulated asynchronous run (Eq.4 of Section 3, seeded
// delays) of rods with long subdomains, as strips about the subdomain edges.
// (Host-side declarations; the kernels are in kernels_strips.hip.)
//
// In the emulated mode the delays are a fixed function of the seed, so nothing
// has to be traded between workgroups while a run proceeds: what happens at an
// edge depends on the state around it alone.  Over T steps a point feels
// nothing beyond the reach R of T steps (heat1d_band.h: the weights beyond it
// sum to a sixteenth of a rounding), so
//   * a workgroup that steps the strip [e - W, e + W) about an edge e, whatever
//     it takes for the values outside, has the points within W - R of e right;
//   * points further than R from every edge are those of the synchronous run.
// A stage of T steps is therefore one launch of independent strips with the points between them from one band pass (T steps at
// once), or, where the subdomains are short, strips wide enough to meet
// halfway between the edges.  The last values of each edge pass from stage to
// stage for the delayed reads.
#pragma once

#include <hip/hip_runtime.h>
#include <stddef.h>
#include <stdint.h>

namespace heat1d {

// How a run of K steps is staged in at most `most` stages; stages = 0: not by
// strips.  band: the points between the strips may come from a band pass.
struct StripPlan {
  int64_t stages = 0;
  int64_t T = 0;   // steps of every stage but the last, which takes the rest
  int M = 0;       // points per lane: the strip reaches 56 M to either side
  int cut = 0;     // a strip's own points reach this far from its edge, 0: to
                   // the middle of the subdomains (no band pass)
};
constexpr int kStripMaxDelay = 63;  // the last 64 values are kept
StripPlan strip_plan(int dtype, int64_t N, int P, double r, int64_t K, int d,
                     int64_t most, bool band);

size_t strip_history_bytes(int dtype, int P);

// One stage: steps [k0, k0 + T) from `in` to the strips' own points of `out`.
struct StripStage {
  int dtype = 0;
  const void* in = nullptr;
  void* out = nullptr;
  int64_t N = 0;
  int P = 0, d = 0, sched = 0, ring = 0;
  int64_t k0 = 0, T = 0;
  uint64_t seed = 0;
  double r = 0, c1 = 0, cN = 0;
  int M = 0, cut = 0;
  void* history = nullptr;  // strip_history_bytes
  int32_t* flag = nullptr;  // raised when a point read is not finite
};
hipError_t launch_strips(const StripStage& a, hipStream_t s);

}  // namespace heat1d
