// kernels_band.hip -- T steps of Eq.3 (Section 2) in one pass: the T-step
// operator, a banded Toeplitz matrix, applied on the matrix cores.
//
// Layout of one product.  16 consecutive outputs are a column of D, 16 such
// columns (256 consecutive outputs) one MFMA tile: D[i][n] = y[16 n + i].  With
// B[k][n] = x[16 n + k - Hp] (Hp = the reach rounded up to 16) every column
// multiplies the same A[i][k] = w(k - Hp - i): the matrix operand is the same
// for every tile of the rod, is read from one row of weights in LDS, and no
// element of x is rearranged.  K runs over the 2 Hp + 16 points that a column
// reads.  The state lies in LDS padded by 16 bytes per 16 points, so that the
// 64 lanes of a 16-byte read (16 columns, 4 quarters of a 16-point chunk) take
// all 64 banks once.  The accumulators leave each lane with 4 consecutive
// outputs: 16-byte stores (FP64: two), each cache line written whole.
//
// What bounds it: FP32 (FP64) matrix rate, 2 Hp + 16 multiply-adds per point,
// and below a reach of about 60 points the copy of the state.  One rod of 2^26
// FP32 points, K = 2000, r = 0.25 (Hp = 192): 0.455 ms, where eight passes of the
// autotuned wide register tiles took 5.8 ms; the products alone need 0.35 ms at
// the rate of large matrix products (154 TFLOP/s) and the copy 0.10 ms.  4096 FP64
// points, K = 20000: 16 us, from 8.3 ms on one compute unit.
#include <cmath>
#include <algorithm>

#include "heat1d_band.h"
#include "heat1d_device.h"
#include "heat1d_rod.h"

namespace heat1d {

typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef double f64x4 __attribute__((ext_vector_type(4)));

template <typename F> struct Band;
template <> struct Band<float> {
  using Acc = f32x4;
  using Sum = f64x4;
  static constexpr int pad = 4;  // elements of padding per 16 points
  // chunks (of 16 terms) whose sum is formed in FP32 before it is added to the
  // whole, which is kept in FP64: one running FP32 sum of all terms rounds a
  // hundred times at the size of the result (3.5e-7 of it against 64 bits on
  // the 2^26-point rod, where stepping has 0.9e-7)
  static constexpr int group = 4;
  static __device__ __forceinline__ Acc mma(float a, float b, Acc c) {
    return __builtin_amdgcn_mfma_f32_16x16x4f32(a, b, c, 0, 0, 0);
  }
  // the output that row i of A stands for: lane group g holds rows 4g..4g+3
  static __device__ __forceinline__ int row(int i) { return i; }
};
template <> struct Band<double> {
  using Acc = f64x4;
  using Sum = f64x4;
  static constexpr int pad = 2;
  static constexpr int group = 1 << 20;  // one running sum
  static __device__ __forceinline__ Acc mma(double a, double b, Acc c) {
    return __builtin_amdgcn_mfma_f64_16x16x4f64(a, b, c, 0, 0, 0);
  }
  // lane group g holds rows g, g+4, g+8, g+12 of the FP64 product
  static __device__ __forceinline__ int row(int i) { return 4 * (i & 3) + (i >> 2); }
};

constexpr int kBandTile = 256;    // outputs of one MFMA tile
// Tiles of 256 outputs a wavefront of the largest blocks: in FP32 4 leave room for
// five wavefronts a SIMD where 8, which read each weight half as often, leave three
// (N = 2^26, K = 2000 491 -> 455 us, on uniform noise 549 -> 538; N = 2^22, K = 300
// 37.0 -> 35.2 us); 3, and FP64 with other counts, were within noise.
constexpr int kBandLarge = 4;
constexpr int kStepWeights = 64;  // runs whose weights are stepped

// Record of the points of a tile that are not finite: first and last of them,
// counted from the tile's first point (first > last: none).
struct BandRec {
  int first, last;
};

struct BandScratch {
  void* w;       // two sets of kBandMaxReach + 1 weights
  int* flag;     // [slot]: some point was not finite
  BandRec* rec;  // one per tile
};

static BandScratch band_scratch(void* scratch) {
  BandScratch s;
  s.w = scratch;
  s.flag = (int*)((char*)scratch + (size_t)2 * (kBandMaxReach + 1) * 8);
  s.rec = (BandRec*)(s.flag + 4);
  return s;
}

size_t band_scratch_bytes(int64_t N, int64_t nrods) {
  const size_t head = (size_t)2 * (kBandMaxReach + 1) * 8 + 4 * 4;
  const size_t recs = (size_t)nrods * ((N + kBandTile - 1) / kBandTile) * sizeof(BandRec);
  return (head + recs + 255) / 256 * 256;
}

// Bernstein's bound for a sum of T independent moves of variance 2 r, none
// longer than 1: P(|sum| >= h) <= 2 exp(-h^2 / (2 (2 r T + h/3))).  `need` is
// ln 2 plus the bits to be dropped: 28 (FP32) or 57 (FP64), a sixteenth of a
// rounding of the state, for all dropped weights together.  The sum cannot
// exceed T.
template <typename F>
constexpr double kBandNeed = (sizeof(F) == 4 ? 29.0 : 58.0) * 0.6931471805599453;

template <typename F>
__host__ __device__ __forceinline__ int band_bound_of(double r, double T) {
  const double third = kBandNeed<F> / 3.0;
  const double h = third + sqrt(third * third + 2.0 * kBandNeed<F> * (2.0 * r * T));
  return (int)(h < T ? h + 1.0 : T);
}

// Where the tail is nearly that of the normal law (its tilt t = h/V of variance
// V = 2 r T is small), less is enough: the weights beyond h are at most
// exp(-h^2 / (2V) (1 - h^2 / (12 V^2) ..)) p / (1 - exp(-t)), p the largest weight
// of the tilted law, 0.627 / sqrt(V) at most (0.399 where V is large).  The bound
// above drops 2^-33..-37 where 2^-28 is meant, this one 2^-29..-30 (FP64 2^-58.4
// for 2^-57; weights computed exactly, r from 0.01 to 1/2, T from 70 to 5000),
// with 5 to 8 % fewer weights: N = 2^26, r = 1/4, K = 2000, FP32 590 -> 564 us on
// uniform noise, N = 2^25 FP64 723 -> 698 us.
template <typename F>
__host__ __device__ __forceinline__ int band_reach_of(double r, double T) {
  const int bound = band_bound_of<F>(r, T);
  const double V = 2.0 * r * T;
  const double t = sqrt(2.0 * kBandNeed<F> / V);
  if (!(t <= 0.6)) return bound;
  const double saved = log(sqrt(V) * (1.0 - exp(-0.9 * t)) / 0.627);
  const double need = kBandNeed<F> - (saved > 0.0 ? saved : 0.0);
  const double h = sqrt(2.0 * V * need) * (1.0 + need / (8.0 * V)) + 2.0;
  return h < (double)bound ? (int)h : bound;
}

int band_reach(int dtype, double r, int64_t T) {
  const double t = (double)std::min<int64_t>(T, (int64_t)1 << 52);
  return dtype == 0 ? band_reach_of<float>((double)(float)r, t) : band_reach_of<double>(r, t);
}

int band_reach_bound(int dtype, double r, int64_t T) {
  const double t = (double)std::min<int64_t>(T, (int64_t)1 << 52);
  return dtype == 0 ? band_bound_of<float>((double)(float)r, t) : band_bound_of<double>(r, t);
}

BandRun band_run(int dtype, double r, int64_t K, int64_t N, bool ring) {
  BandRun b;
  if (K <= 0) return b;
  int64_t T = K;
  if (band_reach(dtype, r, K) > kBandMaxReach) {
    int64_t lo = 1, hi = K;  // reach(lo) <= max < reach(hi)
    while (hi - lo > 1) {
      const int64_t mid = lo + (hi - lo) / 2;
      (band_reach(dtype, r, mid) <= kBandMaxReach ? lo : hi) = mid;
    }
    T = lo;
  }
  if (const double all = band_decay(r, (double)T, N, ring); all > kBandDecay)
    T = std::max<int64_t>(1, (int64_t)((double)T * kBandDecay / all));
  b.passes = (K + T - 1) / T;
  b.T = (K + b.passes - 1) / b.passes;
  return b;
}

// Weights w[d], d = d0, d0 + step, ... <= H, of T steps (lap: of the second
// difference of T-1 steps), by one workgroup.  With g(t) = 1 - 4 r sin^2(t/2),
// the symbol of one step, w_d is the d-th Fourier coefficient of g^T, and the
// trapezoidal sum over M >= 2 H + 2 angles gives w_d + w_{M-d} + ..., whose
// other terms lie beyond the reach.  |g|^T is exp(T log|g|) with the logarithm
// taken of 1 - x, x small, so its relative error does not grow with T where it
// matters.  As a function of the angle it is as narrow as the weights are wide:
// about 30 of the M/2 angles at each end have |g|^T above 1e-24 (the low ones,
// and for r near 1/2 those near the alternating mode), and only those are
// summed.
template <typename F>
__device__ __forceinline__ void band_weights(F* w, int H, double T, double r, bool lap, int d0,
                                             int step, double* s_g, double* s_c) {
  const double steps = lap ? T - 1.0 : T;
  if (T <= kStepWeights) {
    // a few steps: step a unit value (weights that are zero come out as zero)
    double *cur = s_g, *nxt = s_c;
    const int t = (int)steps, d = threadIdx.x;
    if (d < kStepWeights + 2) cur[d] = d == 0 ? 1.0 : 0.0;
    for (int k = 0; k < t + (lap ? 1 : 0); ++k) {
      __syncthreads();
      if (d < kStepWeights + 1) {
        const double c = cur[d], l2 = (d == 0 ? cur[1] : cur[d - 1]) + cur[d + 1] - 2.0 * c;
        nxt[d] = k < t ? __builtin_fma(r, l2, c) : l2;
      }
      if (d == kStepWeights + 1) nxt[d] = 0.0;
      double* was = cur;
      cur = nxt;
      nxt = was;
    }
    __syncthreads();
    if (d0 == 0 && d <= H) w[d] = (F)cur[d];
    return;
  }
  const int M = (2 * H + 2 + 15) / 16 * 16, half = M / 2;
  const bool neg = fmod(steps, 2.0) != 0.0;  // an odd power
  // g^steps <= exp(-steps a), a = 4 r sin^2; |g|^steps <= exp(-steps b), b = 2 - a
  const double lim = steps > 0.0 ? 56.0 / steps : 4.0;
  const double la = lim / (4.0 * r), lb = (lim - (2.0 - 4.0 * r)) / (4.0 * r);
  const int jlow = la >= 0.5 ? half : min(half, (int)(asin(sqrt(la)) * 0.3183098861837907 * M) + 2);
  const int jhigh = la >= 0.5 ? half + 1
                    : lb <= 0.0 ? half + 1
                    : max(jlow + 1, half - (int)(asin(sqrt(min(lb, 1.0))) * 0.3183098861837907 * M) - 2);
  for (int j = threadIdx.x; j <= half; j += blockDim.x) {
    const double x = (double)j / (double)M;
    s_c[j] = cospi(2.0 * x);
    if (j > jlow && j < jhigh) continue;
    const double s = sinpi(x), c = cospi(x);
    const double a = 4.0 * r * s * s;
    const double b = (2.0 - 4.0 * r) + 4.0 * r * c * c;  // 2 - a
    double g = a <= 1.0 ? exp(steps * log1p(-a)) : exp(steps * log1p(-b));
    if (steps == 0.0) g = 1.0;
    if (a > 1.0 && neg) g = -g;
    if (lap) g *= -4.0 * s * s;
    s_g[j] = (j == 0 || j == half) ? g : 2.0 * g;
  }
  __syncthreads();
  // At r = 1/2 the high angles mirror the low ones, w_d is 0 where T - d is odd and
  // twice the low sum elsewhere: the zeros are exact, and what errs is one sum, not
  // the mean of two (a ring of 14816 points, T = 3746: 2e-15 against 5e-16).
  const bool mirror = !lap && r == 0.5 && jhigh <= half;
  for (int d = d0 + threadIdx.x; d <= H; d += step) {
    double sum = 0.0;
    int k = 0;  // j d mod M
    for (int j = 0; j <= jlow; ++j) {
      sum = __builtin_fma(s_g[j], s_c[k > half ? M - k : k], sum);
      k += d;
      if (k >= M) k -= M;
    }
    if (mirror) {
      sum = fmod(steps + (double)d, 2.0) != 0.0 ? 0.0 : 2.0 * sum;
    } else {
      k = (int)(((int64_t)jhigh * d) % M);
      for (int j = jhigh; j <= half; ++j) {
        sum = __builtin_fma(s_g[j], s_c[k > half ? M - k : k], sum);
        k += d;
        if (k >= M) k -= M;
      }
    }
    // The sum is off by some 1e-17 whatever the weight is.  The weights of steps are
    // means of means, none is negative, and a state without negative points keeps none.
    w[d] = (F)(lap ? sum / (double)M : fmax(sum / (double)M, 0.0));
  }
}

// A launch of its own (a few microseconds) and not part of every tile, which
// would spend a tenth of its time on them.
template <typename F>
__global__ __launch_bounds__(256) void band_weights_kernel(F* w, int* flag, int H, double T,
                                                           double r) {
  __shared__ double s_g[kBandMaxReach + 16], s_c[kBandMaxReach + 16];
  if (blockIdx.x == 0 && blockIdx.y == 0 && threadIdx.x < 2) flag[threadIdx.x] = 0;
  band_weights<F>(w + (blockIdx.y == 1 ? kBandMaxReach + 1 : 0), H, T, r, blockIdx.y == 1,
                  (int)blockIdx.x * 256, (int)gridDim.x * 256, s_g, s_c);
}

// One rod of a pass.
template <typename F>
struct BandRod {
  const F* in;
  F* out;        // may be NULL
  F* z;          // kTwo only
  const F* w;    // w[0..H]
  const F* w2;   // kTwo only
  int64_t N;
  int H, Hp;     // Hp: H rounded up to 16
  F c1, cN;      // end values as the product takes them (0 for one that is not finite)
  F e1, eN;      // end values
  bool ring;
  bool straight; // the ends' line is subtracted before and added after the product
};

template <typename F>
__host__ __device__ __forceinline__ bool band_finite(F x) {
  return __builtin_fabs((double)x) <= (sizeof(F) == 4 ? 3.4028234663852886e38
                                                      : 1.7976931348623157e308);
}

template <typename F>
__host__ __device__ __forceinline__ void band_ends(BandRod<F>& a, F c1, F cN) {
  a.e1 = c1;
  a.eN = cN;
  a.c1 = band_finite(c1) ? c1 : F(0);
  a.cN = band_finite(cN) ? cN : F(0);
  a.straight = !a.ring && a.N - 1 < a.Hp + 16;
}

// The straight line between the ends, in double.
template <typename F>
__device__ __forceinline__ double band_line(const BandRod<F>& a, int64_t i) {
  return (double)a.c1 + ((double)a.cN - (double)a.c1) * ((double)i / (double)(a.N - 1));
}

// Point q of the rod as the product reads it, q outside [0, N) included: the
// ring wraps; Dirichlet rods continue oddly about each end.  A rod no longer
// than the reach, where several images of an end are read, is first freed of
// the line between its ends (which every step preserves), so that the images
// do not grow.
template <typename F>
__device__ __forceinline__ F band_point(const BandRod<F>& a, int64_t q) {
  const int64_t N = a.N;
  if (a.ring) {
    q %= N;
    return a.in[q < 0 ? q + N : q];
  }
  if (a.straight) {
    const int64_t P = 2 * (N - 1);
    q %= P;
    if (q < 0) q += P;
    if (q == 0 || q == N - 1) return F(0);
    return q < N - 1 ? (F)((double)a.in[q] - band_line(a, q))
                     : (F)(band_line(a, P - q) - (double)a.in[P - q]);
  }
  if (q <= 0) return q == 0 ? a.c1 : F(2) * a.c1 - a.in[-q];
  if (q >= N - 1) return q == N - 1 ? a.cN : F(2) * a.cN - a.in[2 * (N - 1) - q];
  return a.in[q];
}

// A quarter of band_point(a, q) in double, which no finite state takes out of range
// (an image is up to three times the largest value), and of the line.
template <typename F>
__device__ __forceinline__ double band_line_quarter(const BandRod<F>& a, int64_t i) {
  const double c1 = 0.25 * (double)a.c1, cN = 0.25 * (double)a.cN;
  return c1 + (cN - c1) * ((double)i / (double)(a.N - 1));
}
template <typename F>
__device__ double band_point_quarter(const BandRod<F>& a, int64_t q) {
  const int64_t N = a.N;
  if (a.straight) {
    const int64_t P = 2 * (N - 1);
    q %= P;
    if (q < 0) q += P;
    if (q == 0 || q == N - 1) return 0.0;
    return q < N - 1 ? 0.25 * (double)a.in[q] - band_line_quarter(a, q)
                     : band_line_quarter(a, P - q) - 0.25 * (double)a.in[P - q];
  }
  if (q <= 0) return q == 0 ? 0.25 * (double)a.c1 : 0.5 * (double)a.c1 - 0.25 * (double)a.in[-q];
  if (q >= N - 1)
    return q == N - 1 ? 0.25 * (double)a.cN
                      : 0.5 * (double)a.cN - 0.25 * (double)a.in[2 * (N - 1) - q];
  return 0.25 * (double)a.in[q];
}

// The value a step reads at point j of the rod.
template <typename F>
__device__ __forceinline__ F band_value(const BandRod<F>& a, int64_t j) {
  if (!a.ring && j == 0) return a.e1;
  if (!a.ring && j == a.N - 1) return a.eN;
  return a.in[j];
}

template <typename Sum, typename Acc>
__device__ __forceinline__ void band_add(Sum& s, const Acc& x) {
#pragma unroll
  for (int e = 0; e < 4; ++e) s[e] += (double)x[e];
}

// Blocks are dealt to the 8 XCDs in turn: give each XCD a run of consecutive
// tiles, whose halos overlap, so that its L2 holds them.
__device__ __forceinline__ int band_block(int b, int n) {
  const int x = b & 7, q = n >> 3, rem = n & 7;
  return x * q + (x < rem ? x : rem) + (b >> 3);
}

// The tile of NT*WO*256 points from t0 on of one rod, by one workgroup: WO
// wavefronts hold NT MFMA tiles of outputs each, WS wavefronts share the K
// range of one such set and add their sums in LDS.  dot: see BandPass.
template <typename F, int NT, int WO, int WS, bool kTwo>
__device__ __forceinline__ void band_tile(const BandRod<F>& a, int64_t t0, BandRec* rec, int* flag,
                                          const F* dot_with, double* dot, double dot_scale,
                                          F* xs) {
  using B = Band<F>;
  using Acc = typename B::Acc;
  using Sum = typename B::Sum;
  using VT = typename Vec<F>::T;
  constexpr int V = Vec<F>::n;
  constexpr int kThreads = WO * WS * kWave;
  constexpr int kStride = 16 + B::pad;  // of 16 points in LDS
  constexpr int kOut = NT * WO * kBandTile;
  __shared__ int s_first, s_last, s_lost;
  __shared__ double s_dot[WO * WS];
  const int span = kOut + 2 * a.Hp;            // points of the tile with its halos
  F* wl = xs + span / 16 * kStride;            // weights, w(d) at d + Hp + 15
  const int tid = threadIdx.x, lane = tid & (kWave - 1), wave = uniform(tid / kWave);
  const int64_t N = a.N;

  if (tid == 0) {
    s_first = 0x7fffffff;
    s_last = -1;
    s_lost = 0;
  }
  for (int j = tid; j < 2 * a.Hp + 32; j += kThreads) {
    int d = j - a.Hp - 15;
    d = d < 0 ? -d : d;
    wl[j] = d <= a.H ? a.w[d] : F(0);
    if constexpr (kTwo) wl[2 * a.Hp + 32 + j] = d <= a.H ? a.w2[d] : F(0);
  }
  __syncthreads();

  // the state, with zeros for points that are not finite: what they reach is
  // written by band_cone
  const int64_t q0 = t0 - a.Hp;  // rod point of xs[0]
  const bool aligned = ((uintptr_t)(a.in + q0) & 15u) == 0;
  // only points up to the reach past the end are read by outputs that exist
  const int64_t qend = N + a.Hp;
  for (int p = tid * V; p < span; p += kThreads * V) {
    const int64_t q = q0 + p;
    VT v;
    F* pv = reinterpret_cast<F*>(&v);
    if (q > 0 && q + V < N && !a.straight && aligned) {
      v = *reinterpret_cast<const VT*>(a.in + q);
    } else {
#pragma unroll
      for (int e = 0; e < V; ++e) pv[e] = q + e < qend ? band_point(a, q + e) : F(0);
    }
    bool ok = true;
#pragma unroll
    for (int e = 0; e < V; ++e) ok = ok && band_finite(pv[e]);
    // an end value that is not finite entered as 0: it is found here
    if (!a.ring && ((q <= 0 && q + V > 0) || (q <= N - 1 && q + V > N - 1)))
      ok = ok && band_finite(a.e1) && band_finite(a.eN);
    if (!ok) {
#pragma unroll
      for (int e = 0; e < V; ++e) {
        const bool own = p + e >= a.Hp && p + e < a.Hp + kOut && q + e < N;
        const bool bad = own && !band_finite(band_value(a, q + e));
        if (!band_finite(pv[e])) {
          pv[e] = F(0);
          s_lost = 1;
        }
        if (bad) {
          atomicMin(&s_first, (int)(q + e - t0));
          atomicMax(&s_last, (int)(q + e - t0));
        }
      }
    }
    *reinterpret_cast<VT*>(xs + p + (p >> 4) * B::pad) = v;
  }
  __syncthreads();
  if (tid == 0) {
    if (rec != nullptr) *rec = BandRec{s_first, s_last};
    // (an image of a finite point that is out of range counts too)
    if (s_last >= 0 || s_lost) atomicOr(flag, 1);
  }

  const int n = lane & 15, g = lane >> 4;
  const int wo = wave / WS, ws = wave % WS;
  const int chunks = a.Hp / 8 + 1;
  const int cb = chunks * ws / WS, ce = chunks * (ws + 1) / WS;
  const F* xl = xs + (wo * NT * 16 + n) * kStride + 4 * g;
  const F* wa = wl + 4 * g + 15 - B::row(n);
  Sum acc[NT] = {};
  Sum acc2[kTwo ? NT : 1] = {};
  // wavefronts past the end of the rod have nothing to write
  if (t0 + wo * NT * kBandTile < N) {
    for (int c = cb; c < ce;) {
      Acc part[NT] = {};
      Acc part2[kTwo ? NT : 1] = {};
      const int end = ce - c < B::group ? ce : c + B::group;
      for (; c < end; ++c) {
        F wv[4], wv2[4], x[NT][4];
#pragma unroll
        for (int e = 0; e < 4; ++e) wv[e] = wa[16 * c + e];
        if constexpr (kTwo) {
#pragma unroll
          for (int e = 0; e < 4; ++e) wv2[e] = wa[2 * a.Hp + 32 + 16 * c + e];
        }
#pragma unroll
        for (int t = 0; t < NT; ++t) {
          const F* px = xl + (16 * t + c) * kStride;
#pragma unroll
          for (int e = 0; e < 4; e += V) {
            const VT v = *reinterpret_cast<const VT*>(px + e);
            const F* pv = reinterpret_cast<const F*>(&v);
#pragma unroll
            for (int k = 0; k < V; ++k) x[t][e + k] = pv[k];
          }
        }
#pragma unroll
        for (int e = 0; e < 4; ++e) {
#pragma unroll
          for (int t = 0; t < NT; ++t) {
            part[t] = B::mma(wv[e], x[t][e], part[t]);
            if constexpr (kTwo) part2[t] = B::mma(wv2[e], x[t][e], part2[t]);
          }
        }
      }
#pragma unroll
      for (int t = 0; t < NT; ++t) {
        band_add(acc[t], part[t]);
        if constexpr (kTwo) band_add(acc2[t], part2[t]);
      }
    }
  }
  // dL/dr: in . dot_with over this tile's points, in double; a point that is
  // not finite makes it NaN, as it makes every term it reaches
  double part = 0.0;
  if (dot != nullptr) {
    for (int p = tid; p < kOut; p += kThreads) {
      const int64_t q = t0 + p;
      if (q > 0 && q < N - 1) {
        const int x = a.Hp + p;
        part += (double)xs[x + (x >> 4) * B::pad] * (double)dot_with[q];
      }
    }
    if (s_last >= 0) part = __builtin_nan("");
  }
  if constexpr (WS > 1) {
    __syncthreads();  // every wavefront is done with the state
    Sum* sums = reinterpret_cast<Sum*>(xs);
    constexpr int kSets = kTwo ? 2 * NT : NT;
    if (ws > 0) {
#pragma unroll
      for (int t = 0; t < NT; ++t) {
        sums[((wo * (WS - 1) + ws - 1) * kSets + t) * kWave + lane] = acc[t];
        if constexpr (kTwo)
          sums[((wo * (WS - 1) + ws - 1) * kSets + NT + t) * kWave + lane] = acc2[t];
      }
    }
    __syncthreads();
    if (ws == 0) {
      for (int o = 0; o < WS - 1; ++o) {
#pragma unroll
        for (int t = 0; t < NT; ++t) {
          acc[t] += sums[((wo * (WS - 1) + o) * kSets + t) * kWave + lane];
          if constexpr (kTwo)
            acc2[t] += sums[((wo * (WS - 1) + o) * kSets + NT + t) * kWave + lane];
        }
      }
    }
  }
  if (dot != nullptr) {
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) part += __shfl_xor(part, o);
    if (lane == 0) s_dot[wave] = part;
    __syncthreads();
    if (tid == 0) {
      for (int i = 1; i < WO * WS; ++i) part += s_dot[i];
      *dot = dot_scale * part;
    }
  }
  if (ws != 0) return;
  F* dst = a.out;
  F* zst = kTwo ? a.z : nullptr;
  const bool st_aligned = dst != nullptr && ((uintptr_t)(dst + t0) & 15u) == 0;
  const bool z_aligned = kTwo && ((uintptr_t)(zst + t0) & 15u) == 0;
#pragma unroll
  for (int t = 0; t < NT; ++t) {
    const int64_t q = t0 + (wo * NT + t) * kBandTile + 16 * n + 4 * g;
    if (q >= N) continue;
    F y[4], y2[4];
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      y[e] = (F)acc[t][e];
      if constexpr (kTwo) y2[e] = (F)acc2[t][e];
    }
    const bool inner = a.ring ? q + 4 <= N : (q > 0 && q + 4 < N && !a.straight);
    if (!inner && !a.ring) {
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        if (a.straight) y[e] = (F)((double)acc[t][e] + band_line(a, q + e));
        if (q + e == 0) y[e] = a.e1;
        if (q + e == N - 1) y[e] = a.eN;
        if constexpr (kTwo)
          if (q + e == 0 || q + e == N - 1) y2[e] = F(0);
      }
    }
    if (dst != nullptr) {
#pragma unroll
      for (int e = 0; e < 4; e += V) {
        if (st_aligned && q + e + V <= N) {
          VT v;
          F* pv = reinterpret_cast<F*>(&v);
#pragma unroll
          for (int k = 0; k < V; ++k) pv[k] = y[e + k];
          *reinterpret_cast<VT*>(dst + q + e) = v;
        } else {
#pragma unroll
          for (int k = 0; k < V; ++k)
            if (q + e + k < N) dst[q + e + k] = y[e + k];
        }
      }
    }
    if constexpr (kTwo) {
#pragma unroll
      for (int e = 0; e < 4; e += V) {
        if (z_aligned && q + e + V <= N) {
          VT v;
          F* pv = reinterpret_cast<F*>(&v);
#pragma unroll
          for (int k = 0; k < V; ++k) pv[k] = y2[e + k];
          *reinterpret_cast<VT*>(zst + q + e) = v;
        } else {
#pragma unroll
          for (int k = 0; k < V; ++k)
            if (q + e + k < N) zst[q + e + k] = y2[e + k];
        }
      }
    }
  }
}

// Where a point is not finite the band product says nothing: stepping spreads
// it one point a step each way, NaN inside the cone (the step subtracts an
// infinity from itself) and, at exactly T steps' distance, the infinity itself.
// Writes those cones into the tile of kout points at index `tile` of one rod
// with `tiles` of them (rec: one record each).  And where an image of a point about
// an end (or the point less the ends' line) is out of the type's range though the
// state is not, as 2 c1 - u with c1 = 1e38 and u = -2e38: the product took 0 for it,
// and the points that it reaches are summed here from quarters.
template <typename F>
__device__ void band_cone(const BandRod<F>& a, int64_t tile, int64_t tiles, int kout,
                          const BandRec* rec, int64_t T) {
  const int64_t N = a.N;
  for (int p = threadIdx.x; p < kout; p += blockDim.x) {
    const int64_t i = tile * kout + p;
    if (i >= N || (!a.ring && (i == 0 || i == N - 1))) continue;
    // nearest point that is not finite on each side, at most T (or once around
    // the ring) away
    int64_t dist[2] = {T + 1, T + 1};
    F val[2] = {F(0), F(0)};
    for (int side = 0; side < 2; ++side) {
      int64_t tk = tile, from = i, gone = 0;  // gone: points from i to `from`
      while (gone <= T && gone < N) {
        const int64_t lo = tk * kout, hi = min(N, lo + kout) - 1;
        const BandRec rk = rec[tk];
        if (rk.last >= 0) {
          int64_t j = from;
          if (side == 0) {
            while (j >= lo + rk.first && band_finite(band_value(a, j))) --j;
            if (j < lo + rk.first) j = -1;
          } else {
            while (j <= lo + rk.last && band_finite(band_value(a, j))) ++j;
            if (j > lo + rk.last) j = -1;
          }
          if (j >= 0) {
            dist[side] = gone + (side == 0 ? from - j : j - from);
            val[side] = band_value(a, j);
            break;
          }
        }
        gone += side == 0 ? from - lo + 1 : hi - from + 1;
        tk += side == 0 ? -1 : 1;
        if (tk < 0 || tk >= tiles) {
          if (!a.ring) break;
          tk = tk < 0 ? tiles - 1 : 0;
        }
        from = side == 0 ? min(N, (tk + 1) * (int64_t)kout) - 1 : tk * kout;
      }
    }
    const int64_t near = min(dist[0], dist[1]);
    if (near > T) {
      if (a.ring || (!a.straight && i >= a.H && i + a.H <= N - 1)) continue;
      bool lost = false;
      for (int64_t q = i - a.H; q <= i + a.H && !lost; ++q) lost = !band_finite(band_point(a, q));
      if (!lost) continue;
      double sum = 0.0, sum2 = 0.0;
      for (int d = -a.H; d <= a.H; ++d) {
        const double v = band_point_quarter(a, i + d);
        sum = __builtin_fma((double)a.w[d < 0 ? -d : d], v, sum);
        if (a.z != nullptr) sum2 = __builtin_fma((double)a.w2[d < 0 ? -d : d], v, sum2);
      }
      if (a.straight) sum += band_line_quarter(a, i);
      if (a.out != nullptr) a.out[i] = (F)(4.0 * sum);
      if (a.z != nullptr) a.z[i] = (F)(4.0 * sum2);
      continue;
    }
    F y = (F)__builtin_nan("");
    if (near == T) y = (dist[0] == T ? val[0] : F(0)) + (dist[1] == T ? val[1] : F(0));
    if (a.out != nullptr) a.out[i] = y;
    if (a.z != nullptr) a.z[i] = (F)__builtin_nan("");
  }
}

// Equal rods, back to back.
template <typename F>
struct BandArgs {
  BandRod<F> rod;  // the first
  const F* dot_with;
  double* dot;
  double dot_scale;
  int* flag;
  BandRec* rec;
  int tiles;       // per rod
};

template <typename F>
__device__ __forceinline__ BandRod<F> band_rod(const BandArgs<F>& a, int64_t i) {
  BandRod<F> r = a.rod;
  r.in += i * r.N;
  if (r.out != nullptr) r.out += i * r.N;
  if (r.z != nullptr) r.z += i * r.N;
  return r;
}

template <typename F, int NT, int WO, int WS, bool kTwo>
__global__ __launch_bounds__(WO* WS * kWave) void band_kernel(const BandArgs<F> a) {
  extern __shared__ __align__(16) char band_lds[];
  const int block = band_block(blockIdx.x, gridDim.x);
  const int rodi = block / a.tiles;
  const int64_t t0 = (int64_t)(block - rodi * a.tiles) * (NT * WO * kBandTile);
  band_tile<F, NT, WO, WS, kTwo>(band_rod(a, rodi), t0, a.rec != nullptr ? a.rec + block : nullptr,
                                 a.flag,
                                 a.dot != nullptr ? a.dot_with + rodi * a.rod.N : nullptr,
                                 a.dot != nullptr ? a.dot + block : nullptr, a.dot_scale,
                                 reinterpret_cast<F*>(band_lds));
}

// Returns at once when no point was flagged.
template <typename F>
__global__ __launch_bounds__(256) void band_cone_kernel(const BandArgs<F> a, int* next_flag,
                                                        int64_t T, int kout, int64_t blocks) {
  const bool any = *a.flag != 0;
  if (blockIdx.x == 0 && threadIdx.x == 0) *next_flag = 0;
  if (!any) return;
  for (int64_t block = blockIdx.x; block < blocks; block += gridDim.x) {
    const int64_t rodi = block / a.tiles;
    band_cone(band_rod(a, rodi), block - rodi * a.tiles, a.tiles, kout, a.rec + rodi * a.tiles, T);
  }
}

// Outputs of a block.  Large tiles (a weight is read once per 4 products, the
// halos are a twentieth to a tenth of the tile) where they still give every
// CU two blocks and pad a rod by no more than an eighth; else 2048 outputs; else
// 256, eight wavefronts sharing the K range, so that a rod of a few thousand
// points still spreads over the chip.
// Passes that also write z hold twice the sums: half as many tiles.
template <typename F>
static int band_out(int64_t N, int64_t nrods, bool two = false) {
  const int64_t large = (int64_t)kBandLarge / (two ? 2 : 1) * 4 * kBandTile;
  const int64_t nl = (N + large - 1) / large, nm = (N + 2047) / 2048;
  if (nl * nrods >= 512 && nl * large * 8 <= nm * 2048 * 9) return (int)large;
  if (nm * nrods >= 512 && N >= 1024) return 2048;
  return kBandTile;
}

int64_t band_tiles(int dtype, int64_t N, int64_t nrods) {
  const int o = dtype == 0 ? band_out<float>(N, nrods) : band_out<double>(N, nrods);
  return (N + o - 1) / o;
}

bool band_applies(int dtype, int64_t N, int64_t nrods) {
  // a grid of at most 2^32 - 1 threads, 512 in a block
  return band_tiles(dtype, N, nrods) <= (int64_t(1) << 22) / nrods;
}

// The weights of z, a second difference, fall off later in relation to their sum.
static int pass_reach(const BandPass& p) {
  if (p.z == nullptr) return band_reach(p.dtype, p.r, p.T);
  const int h = band_reach(p.dtype, p.r, p.T);
  return std::max(h, std::min(band_reach_bound(p.dtype, p.r, p.T), kBandMaxReach));
}

template <typename F>
static BandArgs<F> band_args(const BandPass& p) {
  const BandScratch s = band_scratch(p.scratch);
  BandArgs<F> a;
  a.rod.in = (const F*)p.in;
  a.rod.out = (F*)p.out;
  a.rod.z = (F*)p.z;
  a.rod.w = (const F*)s.w;
  a.rod.w2 = (const F*)s.w + kBandMaxReach + 1;
  a.rod.N = p.N;
  a.rod.H = pass_reach(p);
  a.rod.Hp = (a.rod.H + 15) / 16 * 16;
  a.rod.ring = p.ring != 0;
  band_ends(a.rod, (F)p.c1, (F)p.cN);
  a.dot_with = (const F*)p.dot_with;
  a.dot = p.dot;
  a.dot_scale = p.dot_scale;
  a.flag = p.flag != nullptr ? p.flag : s.flag + p.slot;
  a.rec = p.flag != nullptr ? nullptr : s.rec;
  const int64_t o = band_out<F>(p.N, p.nrods, p.z != nullptr);
  a.tiles = (int)((p.N + o - 1) / o);
  return a;
}

template <typename F>
static hipError_t band_weights_launch(const BandPass& p, hipStream_t s) {
  const BandScratch b = band_scratch(p.scratch);
  const int H = pass_reach(p);
  if (H > kBandMaxReach) return hipErrorInvalidValue;
  hipLaunchKernelGGL(band_weights_kernel<F>,
                     dim3((unsigned)(H / 256 + 1), p.z != nullptr ? 2 : 1), dim3(256), 0, s,
                     (F*)b.w, b.flag, H, (double)p.T, (double)(F)p.r);
  return hipGetLastError();
}

hipError_t launch_band_weights(const BandPass& p, hipStream_t s) {
  return p.dtype == 0 ? band_weights_launch<float>(p, s) : band_weights_launch<double>(p, s);
}

// LDS of a tile: the padded state with its halos and the weights (or the sums
// of the wavefronts that share a K range).
template <typename F, int NT, int WO, int WS, bool kTwo>
static size_t band_lds_bytes(int Hp) {
  constexpr int kStride = 16 + Band<F>::pad;
  const size_t xs = (size_t)(NT * WO * kBandTile + 2 * Hp) / 16 * kStride;
  size_t lds = (xs + (size_t)(kTwo ? 2 : 1) * (2 * Hp + 32)) * sizeof(F);
  if (WS > 1)
    lds = std::max(lds, (size_t)WO * (WS - 1) * (kTwo ? 2 : 1) * NT * kWave * 4 * 8);
  return lds;
}

template <typename F, int NT, int WO, int WS, bool kTwo>
static hipError_t band_launch(const BandArgs<F>& a, int64_t nrods, hipStream_t s) {
  const size_t lds = band_lds_bytes<F, NT, WO, WS, kTwo>(a.rod.Hp);
  const auto kernel = band_kernel<F, NT, WO, WS, kTwo>;
  if (lds > 65536) {
    const hipError_t e = hipFuncSetAttribute(
        (const void*)kernel, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
    if (e != hipSuccess) return e;
  }
  hipLaunchKernelGGL(kernel, dim3((unsigned)(a.tiles * nrods)), dim3(WO * WS * kWave),
                     (unsigned)lds, s, a);
  return hipGetLastError();
}

template <typename F, bool kTwo>
static hipError_t band_dispatch(const BandPass& p, hipStream_t s) {
  const BandArgs<F> a = band_args<F>(p);
  if (a.rod.H > kBandMaxReach) return hipErrorInvalidValue;
  const int o = band_out<F>(p.N, p.nrods, kTwo);
  if (o == kBandTile) return band_launch<F, 1, 1, 8, kTwo>(a, p.nrods, s);
  if (o == 2048) return band_launch<F, 2, 4, 1, kTwo>(a, p.nrods, s);
  return band_launch<F, kBandLarge / (kTwo ? 2 : 1), 4, 1, kTwo>(a, p.nrods, s);
}

hipError_t launch_band_pass(const BandPass& p, hipStream_t s) {
  if (p.z == nullptr)
    return p.dtype == 0 ? band_dispatch<float, false>(p, s) : band_dispatch<double, false>(p, s);
  return p.dtype == 0 ? hipErrorInvalidValue : band_dispatch<double, true>(p, s);
}

template <typename F>
static hipError_t band_cones(const BandPass& p, hipStream_t s) {
  const BandArgs<F> a = band_args<F>(p);
  const int64_t blocks = (int64_t)a.tiles * p.nrods;
  hipLaunchKernelGGL(band_cone_kernel<F>, dim3((unsigned)std::min<int64_t>(blocks, 1024)),
                     dim3(256), 0, s, a, band_scratch(p.scratch).flag + (1 - p.slot), p.T,
                     band_out<F>(p.N, p.nrods, p.z != nullptr), blocks);
  return hipGetLastError();
}

hipError_t launch_band_cones(const BandPass& p, hipStream_t s) {
  return p.dtype == 0 ? band_cones<float>(p, s) : band_cones<double>(p, s);
}

// ---- rods of uneven length ------------------------------------------------
template <typename F>
struct BandBatchArgs {
  const F* in;
  F* out;
  const int64_t* offsets;
  const double* r;
  const double* c1;
  const double* cN;
  const int32_t* K;
  const BandItem* items;
  const int32_t* rods;
  const int32_t* woff;
  BandSlot* slots;
  F* w;
  int* flag;
  BandRec* rec;
  int nitems;
};

// r of a slot as the run uses it; 0 where the caller's is not a number in
// [0, 1/2] (its rod is then written as NaN).
template <typename F>
__device__ __forceinline__ bool band_batch_r(const BandBatchArgs<F>& a, int rod, double* r) {
  const double x = (double)(F)a.r[rod];
  const bool ok = x >= 0.0 && x <= 0.5;
  *r = ok ? x : 0.0;
  return ok;
}

template <typename F>
__device__ __forceinline__ int band_batch_reach(const BandBatchArgs<F>& a, int slot, double r,
                                                int K) {
  return min(band_reach_of<F>(r, (double)K), a.woff[slot + 1] - a.woff[slot] - 1);
}

template <typename F>
__device__ __forceinline__ BandRod<F> band_batch_rod(const BandBatchArgs<F>& a, int slot) {
  const BandSlot d = a.slots[slot];
  BandRod<F> b;
  b.in = a.in + d.off;
  b.out = a.out + d.off;
  b.z = nullptr;
  b.w = a.w + d.woff;
  b.w2 = nullptr;
  b.N = d.N;
  b.H = d.H;
  b.Hp = (b.H + 15) / 16 * 16;
  b.ring = false;
  band_ends(b, (F)d.c1, (F)d.cN);
  return b;
}

template <typename F>
__global__ __launch_bounds__(256) void band_batch_weights_kernel(const BandBatchArgs<F> a) {
  __shared__ double s_g[kBandMaxReach + 16], s_c[kBandMaxReach + 16];
  const int slot = blockIdx.x, rod = a.rods[slot];
  if (slot == 0 && threadIdx.x == 0) *a.flag = 0;
  double r;
  const bool ok = band_batch_r(a, rod, &r);
  const int64_t N = a.offsets[rod + 1] - a.offsets[rod];
  const bool steps = band_decay(r, (double)a.K[rod], N, false) > kBandDecay && N <= kBandBatchStep;
  const int H = steps ? -1 : band_batch_reach(a, slot, r, a.K[rod]);
  F* w = a.w + a.woff[slot];
  if (!steps) band_weights<F>(w, H, (double)a.K[rod], r, false, 0, 256, s_g, s_c);
  if (threadIdx.x == 0) {
    if (!ok) w[0] = (F)__builtin_nan("");
    a.slots[slot] = BandSlot{a.offsets[rod], N, a.c1[rod], a.cN[rod], H, a.woff[slot]};
  }
}

// K steps of the slots' rods that are stepped, a wavefront each (at most
// kBandBatchStep points, up to eight a lane, neighbours by DPP): the bits of one launch
// per step.  A launch of its own, where a plan has such rods: in the tiles' kernel it
// cost those 0.9 %, and a workgroup a rod, with a barrier a step, up to 2.2 times the
// time (32768 rods of 3 points, K = 5000, FP32: 10.5 ms).
template <typename F>
__global__ __launch_bounds__(256) void band_batch_step_kernel(const BandBatchArgs<F> a, int nslots) {
  const int lane = threadIdx.x & (kWave - 1);
  const int slot = uniform((int)blockIdx.x * 4 + (int)(threadIdx.x / kWave));
  if (slot >= nslots) return;
  const BandRod<F> b = band_batch_rod(a, slot);
  if (b.H >= 0) return;
  const int rod = a.rods[slot], n = uniform((int)b.N), K = uniform(a.K[rod]);
  const F r = (F)a.r[rod];
#define HEAT1D_SHORT(M)                                                                      \
  return rod_resident<F, M, RodSync::kWave>(b.in, b.out, n, K, r, b.e1, b.eN, nullptr, 1, 0, \
                                            lane, false)
  if (n <= kWave) HEAT1D_SHORT(1);
  if (n <= 2 * kWave) HEAT1D_SHORT(2);
  if (n <= 4 * kWave) HEAT1D_SHORT(4);
  HEAT1D_SHORT(8);
#undef HEAT1D_SHORT
}

// With BandSlot (which also saves each tile computing its reach) the rods of the
// benchmark's batch go from 646 to 610 us.
// One tile per workgroup of four wavefronts: 22 thousand tiles for 4096 rods
// of 256 to 65536 points, so the chip stays even to the end without queues.
template <typename F>
__global__ __launch_bounds__(256) void band_batch_kernel(const BandBatchArgs<F> a) {
  extern __shared__ __align__(16) char band_lds[];
  const int i = band_block(blockIdx.x, gridDim.x);
  const BandItem it = a.items[i];
  const BandRod<F> rod = band_batch_rod(a, uniform(it.slot));
  if (rod.H < 0) {
    if (threadIdx.x == 0) a.rec[i] = BandRec{0x7fffffff, -1};
    return;
  }
  band_tile<F, 2, 4, 1, false>(rod, (int64_t)uniform(it.tile) * kBandBatchTile, a.rec + i, a.flag,
                               nullptr, nullptr, 0.0, reinterpret_cast<F*>(band_lds));
}

template <typename F>
__global__ __launch_bounds__(256) void band_batch_cone_kernel(const BandBatchArgs<F> a) {
  if (*a.flag == 0) return;
  for (int i = blockIdx.x; i < a.nitems; i += gridDim.x) {
    const BandItem it = a.items[i];
    const BandRod<F> rod = band_batch_rod(a, it.slot);
    if (rod.H < 0) continue;
    band_cone(rod, it.tile, (rod.N + kBandBatchTile - 1) / kBandBatchTile, kBandBatchTile,
              a.rec + (i - it.tile), (int64_t)a.K[a.rods[it.slot]]);
  }
}

template <typename F>
static hipError_t band_batch(const BandBatch& b, hipStream_t s) {
  BandBatchArgs<F> a;
  a.in = (const F*)b.in;
  a.out = (F*)b.out;
  a.offsets = b.offsets;
  a.r = b.r;
  a.c1 = b.c1;
  a.cN = b.cN;
  a.K = b.K;
  a.items = b.items;
  a.rods = b.rods;
  a.woff = b.woff;
  a.slots = (BandSlot*)b.slot;
  a.w = (F*)b.w;
  a.flag = b.flag;
  a.rec = (BandRec*)b.rec;
  a.nitems = b.nitems;
  hipLaunchKernelGGL(band_batch_weights_kernel<F>, dim3((unsigned)b.nslots), dim3(256), 0, s, a);
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  const size_t lds = band_lds_bytes<F, 2, 4, 1, false>((b.hmax + 15) / 16 * 16);
  if (lds > 65536) {
    e = hipFuncSetAttribute((const void*)band_batch_kernel<F>,
                            hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
    if (e != hipSuccess) return e;
  }
  hipLaunchKernelGGL(band_batch_kernel<F>, dim3((unsigned)b.nitems), dim3(256), (unsigned)lds, s,
                     a);
  e = hipGetLastError();
  if (e != hipSuccess) return e;
  if (b.short_rods) {
    hipLaunchKernelGGL(band_batch_step_kernel<F>, dim3((unsigned)((b.nslots + 3) / 4)), dim3(256),
                       0, s, a, b.nslots);
    e = hipGetLastError();
    if (e != hipSuccess) return e;
  }
  hipLaunchKernelGGL(band_batch_cone_kernel<F>, dim3((unsigned)std::min(b.nitems, 1024)),
                     dim3(256), 0, s, a);
  return hipGetLastError();
}

hipError_t launch_band_batch(const BandBatch& b, hipStream_t s) {
  if (b.hmax > kBandMaxReach || b.nitems < 1) return hipErrorInvalidValue;
  return b.dtype == 0 ? band_batch<float>(b, s) : band_batch<double>(b, s);
}

}  // namespace heat1d
