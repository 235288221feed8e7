// kernels_strips.hip -- the emulated asynchronous run of Eq.4 (Section 3) as
// independent strips about the subdomain edges.
//
// Layout: a strip is one workgroup of two wavefronts that overlap about the
// edge e.  Wavefront 0 holds the points [e - 56 M, e + 8 M), wavefront 1 [e - 8 M,
// e + 56 M), lane l of each M consecutive ones, so that the edge lies between
// the last register of one fixed lane and the first of the next whatever the
// partition.  Both step across the edge on their own: the points at their cut
// ends go wrong by one a step, and every 8 M steps (in whole groups of 32) they
// give each other the 8 M points that did not.  One wavefront with the whole
// strip issues a VALU instruction every 6 to 7 clocks, being alone on its SIMD
// (1024 strips, 1024 SIMDs); two share it at under 3 each.
//
// Every neighbour but the two across the edge comes by a DPP wavefront shift.
// The last 64 values of the two edge points lie in LDS, one ring per wavefront
// (so that no barrier is needed); the delays are drawn 32 steps at a time, a
// (step, side) per lane, and a delayed value is read while the step before it is
// computed, so that no step waits for LDS.  A step costs the 3 M arithmetic
// instructions of the lane's points and about ten more.
//
// What bounds it: VALU issue, two wavefronts a SIMD at 1024 strips (3.9 clocks an
// instruction), latency below.  2^24 FP32 points, P = 1024, d = 4, K = 5000: 1.15 ms, of
// which the strips (M = 16) take 1.02 and one band pass the rest, where the persistent
// kernel took 10.8 ms; with one wavefront to a strip they took 1.67 ms.  4096 FP64
// points, P = 16, d = 3, K = 20000: 102 stages of 197 steps, 3.0 ms, from 26 ms.
#include <algorithm>
#include <cmath>

#include "heat1d_band.h"
#include "heat1d_delays.h"
#include "heat1d_device.h"
#include "heat1d_strips.h"

namespace heat1d {

namespace {

template <typename F>
struct StripArgs {
  const F* in;
  F* out;
  F* history;
  int32_t* flag;
  int64_t N;
  int P, d, sched, ring;
  int k0, T;
  uint64_t seed;
  F r, c1, cN;
  int cut;
  int nstrips;
};

// Point q of the rod, or of its continuation: around the ring, or oddly about
// a Dirichlet end (a continuation every step preserves).
template <typename F>
__device__ __forceinline__ F strip_point(const StripArgs<F>& a, int64_t q) {
  const int64_t N = a.N;
  if (a.ring) {
    if (q < 0) q += N;
    else if (q >= N) q -= N;
    return a.in[q];
  }
  if (q <= 0) return q == 0 ? a.c1 : F(2) * a.c1 - a.in[-q];
  if (q >= N - 1) return q == N - 1 ? a.cN : F(2) * a.cN - a.in[2 * (N - 1) - q];
  return a.in[q];
}

__device__ __forceinline__ bool strip_finite(float x) {
  return __builtin_fabsf(x) <= 3.4028234663852886e38f;
}
__device__ __forceinline__ bool strip_finite(double x) {
  return __builtin_fabs(x) <= 1.7976931348623157e308;
}

// First point of subdomain b.
__device__ __forceinline__ int64_t strip_lo(int64_t N, int P, int b) {
  return (int64_t)b * N / P;
}

constexpr int kOver = 8;   // lanes of a wavefront beyond the edge
constexpr int kRing = 64;  // steps of history

// T steps of one wavefront's points; la: the lane of point e-1.  ring[k & 63]
// holds the values of points e-1 and e at step k; table[k & 63][side] where in
// the ring step k reads (bytes).
template <typename F, int M, bool kEdge>
__device__ __forceinline__ void strip_run(F (&u)[M], const StripArgs<F>& a, int b, int lane,
                                          int wave, int la, F (*ring)[2], int (*table)[2],
                                          F (*swap)[kOver * M]) {
  constexpr int kSlot = 2 * (int)sizeof(F);  // bytes of a step in the ring
  const int kend = a.k0 + a.T;
  const int pl = b > 0 ? b - 1 : a.P - 1;    // the subdomain left of the edge
  const int side = lane <= la ? 1 : 0;       // what a lane of this half reads: see draw
  // Every lane writes its edge value at `own` + the step's slot: the two at the
  // edge into the ring, the others behind it (a masked write would make the
  // compiler wait for it).
  const int own = lane == la ? 0
                  : lane == la + 1 ? (int)sizeof(F)
                                   : kRing * kSlot + lane * (int)sizeof(F);
  char* rb = reinterpret_cast<char*>(ring);
  F r = a.r;
  asm("" : "+v"(r));  // VALU instructions with a scalar operand issue at half rate
  // slots of steps kb .. kb+31: lane l draws step kb + l/2, side l & 1; side 0 is
  // point e reading e-1, side 1 point e-1 reading e
  auto draw = [&](int kb) {
    if constexpr (kEdge) {
      const int k = kb + (lane >> 1), sd = lane & 1;
      const int dl = sched_delay(a.sched, a.seed, k, sd ? pl : b, sd, a.P, a.d);
      table[k & (kRing - 1)][sd] =
          (max(k - dl, 0) & (kRing - 1)) * kSlot + sd * (int)sizeof(F);
    }
  };
  F left, right;
  int slot = 0, slot2 = 0;  // of the coming step and the one after it
  F old = F(0);             // what the ring holds for the coming step
  // Step k's reads, given its state's end points of each lane: a delay of 0
  // reads the neighbour's value of this step, which the lane shift brings; an
  // older one was read from the ring while the step before was computed.
  auto handover = [&](int k, F u0, F u1) {
    left = from_lower_lane(u1);
    right = from_upper_lane(u0);
    if constexpr (kEdge) {
      const int now = (k & (kRing - 1)) * kSlot;
      const bool late = slot != now + side * (int)sizeof(F);
      left = late && lane == la + 1 ? old : left;
      right = late && lane == la ? old : right;
      *reinterpret_cast<F*>(rb + now + own) = side ? u1 : u0;
      slot = slot2;
      old = *reinterpret_cast<F*>(rb + slot);
      slot2 = table[(k + 2) & (kRing - 1)][side];
    }
  };
  draw(a.k0);
  draw(a.k0 + 32);
  if constexpr (kEdge) {
    slot = table[a.k0 & (kRing - 1)][side];
    slot2 = table[(a.k0 + 1) & (kRing - 1)][side];
    old = *reinterpret_cast<F*>(rb + slot);
  }
  handover(a.k0, u[0], u[M - 1]);
  constexpr int kSwap = kOver * M / 32;  // groups of 32 steps between two trades
  // whether a trade comes as late as the overlap allows, with a weight that counts
  constexpr bool kAgain = kEdge && 32 * kSwap == kOver * M && kOver * M < 57;
  int since = 0;
  for (int kb = a.k0; kb < kend; kb += 32) {
    const int n = min(32, kend - kb);
    for (int i = 0; i < n; ++i) {
      // the lane's two end points first: their values are what the handover
      // waits for, and it is under way while the inner points follow
      F prev = u[0];
      const F u0 = eq3_step(left, u[0], u[1], r);
      const F u1 = eq3_step(u[M - 2], u[M - 1], right, r);
      handover(kb + i + 1, u0, u1);
      __builtin_amdgcn_sched_barrier(0);
      u[0] = u0;
#pragma unroll
      for (int j = 1; j < M - 1; ++j) {
        const F c = u[j];
        u[j] = eq3_step(prev, c, u[j + 1], r);
        prev = c;
      }
      u[M - 1] = u1;
    }
    // the reads run two steps ahead of the table's half that is replaced here
    draw(kb + 64);
    if (++since == kSwap && kb + 32 < kend) {
      // wavefront 0 takes the points from e on, wavefront 1 those before e
      if (wave == 0 ? (lane > la - kOver && lane <= la) : (lane > la && lane <= la + kOver)) {
        const int o = (wave == 0 ? lane - (la - kOver + 1) : lane - (la + 1)) * M;
#pragma unroll
        for (int j = 0; j < M; ++j) swap[wave][o + j] = u[j];
      }
      __syncthreads();
      if (wave == 0 ? lane > la : lane <= la) {
        const int o = (wave == 0 ? lane - (la + 1) : lane) * M;
#pragma unroll
        for (int j = 0; j < M; ++j) u[j] = swap[1 - wave][o + j];
      }
      since = 0;
      // The handover of this step again, for the points that changed.  Where the trade
      // comes as late as the overlap allows, what lies beyond the cut ends has just
      // reached the edge point of the other side, with r^(8 M), and a delay of 0 and the
      // ring took it: 2^-32 of it at M = 4, where the edge's values are made anew.  (What
      // a delayed read of this step brought is older and stands.  From M = 8 on it is
      // 2^-64, less than the 2^-57 that is dropped elsewhere.)
      bool stands = kEdge;
      if constexpr (kAgain) {
        const int now = ((kb + 32) & (kRing - 1)) * kSlot;
        stands = table[(kb + 32) & (kRing - 1)][side] != now + side * (int)sizeof(F);
        *reinterpret_cast<F*>(rb + now + own) = side ? u[M - 1] : u[0];
        old = *reinterpret_cast<F*>(rb + slot);
      }
      __syncthreads();
      const F l = from_lower_lane(u[M - 1]), rr = from_upper_lane(u[0]);
      left = stands && lane == la + 1 ? left : l;
      right = stands && lane == la ? right : rr;
    }
  }
}

template <typename F, int M>
__global__ __launch_bounds__(128) void strip_kernel(const StripArgs<F> a) {
  __shared__ F s_ring[2][2 * kRing + kWave / 2][2];  // the ring, then what lanes off the edge write
  __shared__ int s_table[2][kRing][2];
  __shared__ F s_swap[2][kOver * M];
  const int lane = threadIdx.x & (kWave - 1), wave = uniform(threadIdx.x / kWave);
  // edges 1..P-1, with 0 too on a ring; strips that meet halfway also cover
  // the Dirichlet ends, as edges 0 and P with nothing delayed
  const int b = (a.ring || a.cut == 0) ? (int)blockIdx.x : (int)blockIdx.x + 1;
  const bool edge = a.ring || (b > 0 && b < a.P);
  const int64_t N = a.N;
  const int64_t e = strip_lo(N, a.P, b);
  const int la = wave == 0 ? kWave - 1 - kOver : kOver - 1;
  const int64_t g0 = e - (int64_t)(la + 1) * M;
  const int64_t q0 = g0 + lane * M;
  const bool inside = g0 > 0 && g0 + 64 * M < N;

  F u[M];
  if (inside) {
#pragma unroll
    for (int j = 0; j < M; ++j) u[j] = a.in[q0 + j];
  } else {
#pragma unroll
    for (int j = 0; j < M; ++j) u[j] = strip_point(a, q0 + j);
  }
  bool ok = true;
#pragma unroll
  for (int j = 0; j < M; ++j) ok = ok && strip_finite(u[j]);
  if (__any(!ok) && lane == 0) atomicOr(a.flag, 1);

  F* hist = a.history + (int64_t)b * 128;
  F(*ring)[2] = s_ring[wave];
  if (edge && a.k0 > 0) {
    ring[lane][0] = hist[2 * lane];
    ring[lane][1] = hist[2 * lane + 1];
  }
  // Wavefront 0 replaces the history when it is done, which a stage of few steps is
  // before any exchange has made it wait for the other one's reads above.
  __syncthreads();
  if (edge) strip_run<F, M, true>(u, a, b, lane, wave, la, ring, s_table[wave], s_swap);
  else strip_run<F, M, false>(u, a, b, lane, wave, la, ring, s_table[wave], s_swap);
  if (edge && wave == 0) {
    hist[2 * lane] = ring[lane][0];
    hist[2 * lane + 1] = ring[lane][1];
  }
  // the strip's own points
  int64_t lo = e - a.cut, hi = e + a.cut;
  if (a.cut == 0) {
    // as far as halfway to the next edges (around the ring they lie beyond 0 and N)
    const int64_t prev = b > 0 ? strip_lo(N, a.P, b - 1)
                               : (a.ring ? strip_lo(N, a.P, a.P - 1) - N : -e);
    const int64_t next = b < a.P ? strip_lo(N, a.P, b + 1) : e;
    lo = b == 0 && !a.ring ? 0 : prev + (e - prev) / 2;
    hi = b == a.P ? N : e + (next - e) / 2;
  }
  // wavefront 0 writes those before the edge, wavefront 1 the others
  if (wave == 0) hi = e;
  else lo = e;
  const int plo = (int)(lo - g0), phi = (int)(hi - g0);
  if (inside) {
    store_points<F, M>(u, a.out, q0, lane * M, plo, phi, false);
    return;
  }
#pragma unroll
  for (int j = 0; j < M; ++j) {
    const int p = lane * M + j;
    int64_t q = g0 + p;
    if (p < plo || p >= phi) continue;
    if (a.ring) q = q < 0 ? q + N : (q >= N ? q - N : q);
    F v = u[j];
    if (!a.ring && q == 0) v = a.c1;
    if (!a.ring && q == N - 1) v = a.cN;
    a.out[q] = v;
  }
}

// Shortest stage.  A stage takes 7 us or more, the persistent kernel 1.0 to 1.3 us a
// step: 4096 points, d = 4, K = 2000, FP32, subdomains of 6 / 8 / 12 / 16 / 24 points
// (stages of 2, 3, 5, 7 and 11 steps): 2498 / 2335 / 2462 / 2241 / 2447 us there, 5236
// / 3537 / 2416 / 1742 / 1222 as strips; with d = 50, whose reads wait least, 460
// against 567 at 12 points and 442 against 411 at 16 (K = 448).
constexpr int kStripMinSteps = 7;

constexpr int kStripM[] = {4, 5, 6, 7, 8, 10, 12, 14, 16, 18, 20};

template <typename F>
hipError_t strips_launch(const StripStage& p, hipStream_t s) {
  StripArgs<F> a;
  a.in = (const F*)p.in;
  a.out = (F*)p.out;
  a.history = (F*)p.history;
  a.flag = p.flag;
  a.N = p.N;
  a.P = p.P;
  a.d = p.d;
  a.sched = p.sched;
  a.ring = p.ring;
  a.k0 = (int)p.k0;
  a.T = (int)p.T;
  a.seed = p.seed;
  a.r = (F)p.r;
  a.c1 = (F)p.c1;
  a.cN = (F)p.cN;
  a.cut = p.cut;
  a.nstrips = p.ring ? p.P : (p.cut > 0 ? p.P - 1 : p.P + 1);
  const dim3 grid((unsigned)a.nstrips), block(128);
  switch (p.M) {
#define HEAT1D_STRIP(MM) \
  case MM: hipLaunchKernelGGL((strip_kernel<F, MM>), grid, block, 0, s, a); break;
    HEAT1D_STRIP(4)
    HEAT1D_STRIP(5)
    HEAT1D_STRIP(6)
    HEAT1D_STRIP(7)
    HEAT1D_STRIP(8)
    HEAT1D_STRIP(10)
    HEAT1D_STRIP(12)
    HEAT1D_STRIP(14)
    HEAT1D_STRIP(16)
    HEAT1D_STRIP(18)
    HEAT1D_STRIP(20)
#undef HEAT1D_STRIP
    default: return hipErrorInvalidValue;
  }
  return hipGetLastError();
}

}  // namespace

size_t strip_history_bytes(int dtype, int P) {
  return ((size_t)(P + 1) * 128 * (dtype == 0 ? 4 : 8) + 255) / 256 * 256;
}

StripPlan strip_plan(int dtype, int64_t N, int P, double r, int64_t K, int d, int64_t most,
                     bool band) {
  StripPlan best;
  if (d < 1 || d > kStripMaxDelay || P < 2 || K < 1) return best;
  const int64_t sub = N / P, longest = (N + P - 1) / P;
  // Microseconds of a step of a strip of M points per lane while the chip holds
  // two wavefronts a SIMD, of a band pass and of a stage's launches (measured:
  // FP32 0.12 at M = 7, 0.15 at 8, 0.18 at 12, 0.23 at 16; FP64 0.13 at 5 and
  // 0.14 at 7; 10 a stage; a pass over 2^24 FP32 points, reach 220, 0.17 ms).
  const double per_simd = std::max(1.0, std::ceil((P + 1) / 1024.0));
  const double step0 = dtype == 0 ? 0.06 : 0.07, step1 = dtype == 0 ? 0.0105 : 0.012;
  double cost = 1e300;
  for (int m : kStripM) {
    const int64_t half = (int64_t)(kWave - kOver) * m;
    if (half + 2 > N - 1) continue;
    for (int cover = band ? 0 : 1; cover < 2; ++cover) {
      // the longest stage whose reach the strip and the subdomains allow
      const int64_t reach =
          std::min((sub - 2) / 2, cover ? half - (longest + 1) / 2 - 1 : half / 2);
      if (reach < 2 || (!cover && reach > kBandMaxReach)) continue;
      int64_t lo = 0, hi = K + 1;  // reach of lo steps fits, of hi steps does not (or is not asked)
      while (hi - lo > 1) {
        const int64_t mid = lo + (hi - lo) / 2;
        (band_reach_bound(dtype, r, mid) <= reach ? lo : hi) = mid;
      }
      if (lo < kStripMinSteps) continue;
      const int64_t stages = (K + lo - 1) / lo, T = (K + stages - 1) / stages;
      if (stages > most) continue;
      const int64_t R = band_reach_bound(dtype, r, T);
      double c = (double)K * per_simd * (step0 + step1 * m) + (double)stages * 10.0;
      if (!cover)
        c += (double)stages * (10.0 + (double)N * (2.0 * R + 200.0) * (dtype == 0 ? 1.5e-8 : 3e-8));
      if (c < cost) {
        cost = c;
        best.stages = stages;
        best.T = T;
        best.M = m;
        best.cut = cover ? 0 : (int)R;
      }
    }
  }
  return best;
}

hipError_t launch_strips(const StripStage& a, hipStream_t s) {
  return a.dtype == 0 ? strips_launch<float>(a, s) : strips_launch<double>(a, s);
}

}  // namespace heat1d
