// heat1d_api.cpp -- the C ABI declared in include/heat1d.h: argument checks,
// plans, workspace layout, kernel choice and the autotuner.  Every step of the
// computation runs in the HIP kernels of kernels_*.hip; this file only decides
// which ones to launch and with what geometry.
#include "heat1d.h"

#include <hip/hip_runtime.h>

#include <algorithm>
#include <cmath>
#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <numeric>
#include <string>
#include <vector>

#include "heat1d_band.h"
#include "heat1d_ensemble.h"
#include "heat1d_launch.h"
#include "heat1d_observe.h"
#include "heat1d_strips.h"
#include "heat1d_weights.h"

using namespace heat1d;

namespace {

// Synchronous runs of at least this many steps take band passes.  A run of K
// steps is three short launches there, 14 us (18 up to K = 64) on up to 2^18
// points; stepping with AUTO's default kernel against that, at K = 64 / 80 / 128,
// in us: 4096 FP32 points 20 / 24 / 37 against 15 / 14 / 14, 2^22 37 / 51 / 73
// against 29 / 27 / 28, 2^26 331 / 475 / 659 against 221 / 219 / 243.  Where one
// workgroup steps a short rod, or the ring's tiles a small FP64 ring, as fast as
// that, the line lies higher: 100 FP32 points 12 / 15 / 23 against 15 / 14 / 14,
// an FP64 ring of 2^18 16 / 22 / 30 against 18 / 14 / 15.  And where thousands of
// rods fill the chip with narrow register tiles (plans of more than 4096 rods),
// FP32 rods of 257 to 1023 points cost a pass a block of eight wavefronts per 256
// points: 16384 rods of 1000 points take 153 / 197 / 306 us stepped, 382 at
// K = 160, against 320 at any.
constexpr int32_t kBandFrom = 64;
int32_t band_from_steps(int dtype, int64_t N, int64_t nrods, bool ring) {
  const bool f32 = dtype == HEAT1D_F32;
  if (f32 && !ring && nrods > 4096 && N > 256 && N < 1024)
    return 16 + 32 * (int32_t)((N + 255) / 256);
  const bool fast = ring ? !f32 : N <= (f32 ? 1024 : 512);
  return fast && N * nrods <= (int64_t(1) << 18) ? 80 : kBandFrom;
}

// The same for the rods of a batch, and for the long rods of an emulated
// asynchronous run: a line of contract, not of speed.  Shorter runs there give the
// bits of one launch per step, which programs compare them with, and that costs
// them: 4096 rods of 256 to 65536 FP32 points, K = 64 / 200 / 447, take 585 / 1166 /
// 2325 us in the queues where passes would take 239 / 250 / 289; an emulated run of
// 2^18 FP32 points, 1024 subdomains, 101 / 261 / 552 against 38 / 56 / 93.
constexpr int32_t kBatchBandFrom = 448;

// FP32 stepping drifts: late in a run the change of a point in one step is a
// few roundings of its value, and they do not average out.  Against 64 bits the
// single-step kernels are off by 1e-6 (noise) to 6e-5 (a smooth profile) of the
// state after K (1 + 0.1 / r) = 6200 steps, and by 2e-4 to 5e-4 at 20000 steps,
// where one pass stays at 2e-7.  FP32 runs beyond that length keep stepping, not
// for speed or accuracy, but because results that programs have from them would
// move by more than 2e-5.
bool fp32_drifts(int dtype, double r, int64_t K) {
  return dtype == HEAT1D_F32 && (double)K * (1.0 + 0.1 / r) > 6200.0;
}

constexpr size_t kAlign = 256;
size_t align_up(size_t x) { return (x + kAlign - 1) / kAlign * kAlign; }
size_t esize(int dtype) { return dtype == HEAT1D_F32 ? 4 : 8; }
int vec_width(int dtype) { return dtype == HEAT1D_F32 ? 4 : 2; }

struct EventPair {
  hipEvent_t a = nullptr, b = nullptr;
};

}  // namespace

struct heat1d_plan_s {
  int64_t N = 0;
  int dtype = 0;
  int64_t nrods = 1;
  heat1d_opts opts{};
  // synchronous kernel choice
  int sync_kernel = HEAT1D_SYNC_TILED;
  int T = 32;
  int M = 32;
  int fuse = 1;  // steps per register sweep on tiles without a rod end
  int tile_waves = 1;  // tiled kernel: wavefronts per tile (1, or 4 / 8 for wide tiles)
  int waves = 16;
  // runs of at least this many steps take band passes (0: none); only plans
  // that leave the synchronous kernel open
  int32_t band_from = 0;
  // asynchronous
  int32_t max_delay = 16;
  int64_t watchdog = int64_t(1) << 22;
  // adjoint
  int32_t ckpt_stride = 0;
  // batched
  bool batched = false;
  std::vector<int64_t> Nh;
  std::vector<int32_t> Kh;
  std::vector<int32_t> by_work;   // rod indices, longest N*K first
  std::vector<int32_t> order[3];  // workgroup, group and wavefront rods
  int64_t t_wave = 0, t_group = 0;  // longest rod of the wavefront / group queues
  int32_t groups = 0;
  int32_t small_first = 0;  // workgroups that start with the group and wavefront queues
  bool tuned = false;       // the batched work order was chosen by timing
  // rods that take a band pass: their tiles, rod indices and weight offsets
  std::vector<BandItem> band_items;
  std::vector<int32_t> band_rods, band_woff;
  int32_t band_hmax = 0;
  bool band_short = false;  // some of them may decay too much for a pass
  // timing of the dominant kernel
  bool timing = false;
  std::vector<EventPair> ev;
  size_t ev_used = 0;
  std::string desc;
};

namespace {

bool r_ok(double r) { return r > 0.0 && r <= 0.5; }

// [a, a+na) and [b, b+nb) share a byte
bool overlaps(const void* a, size_t na, const void* b, size_t nb) {
  const uintptr_t x = (uintptr_t)a, y = (uintptr_t)b;
  return x < y + nb && y < x + na;
}
bool overlaps(const void* a, const void* b, size_t bytes) { return overlaps(a, bytes, b, bytes); }

int hip_status(hipError_t e) {
  if (e == hipSuccess) return HEAT1D_OK;
  if (std::getenv("HEAT1D_DEBUG")) std::fprintf(stderr, "heat1d: HIP error %s\n", hipGetErrorString(e));
  return HEAT1D_EHIP;
}

int num_cus() {
  int dev = 0, n = 0;
  if (hipGetDevice(&dev) != hipSuccess) return 0;
  if (hipDeviceGetAttribute(&n, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess) return 0;
  return n;
}

// Timing helpers: bracket a launch with a pair of events on its stream.
EventPair* timing_begin(heat1d_plan_t p, hipStream_t s) {
  if (!p->timing) return nullptr;
  if (p->ev_used == p->ev.size()) {
    EventPair e;
    if (hipEventCreate(&e.a) != hipSuccess || hipEventCreate(&e.b) != hipSuccess) return nullptr;
    p->ev.push_back(e);
  }
  EventPair* e = &p->ev[p->ev_used++];
  hipEventRecord(e->a, s);
  return e;
}
void timing_end(EventPair* e, hipStream_t s) {
  if (e) hipEventRecord(e->b, s);
}

int smallest_m(int dtype, int64_t need, bool (*supports)(int, int)) {
  for (int m = 1; m <= 64; m *= 2)
    if (supports(dtype, m) && m >= need) return m;
  return 0;
}

void describe(heat1d_plan_t p) {
  char buf[256];
  if (p->batched) {
    std::snprintf(buf, sizeof buf,
                  "batched rods=%zu dtype=%s wg_rods=%zu group_rods=%zu wave_rods=%zu groups=%d "
                  "small_first=%d t_wave=%lld t_group=%lld band_rods=%zu%s",
                  p->Nh.size(), p->dtype == HEAT1D_F32 ? "f32" : "f64", p->order[0].size(),
                  p->order[1].size(), p->order[2].size(), p->groups, p->small_first,
                  (long long)p->t_wave, (long long)p->t_group, p->band_rods.size(),
                  p->tuned ? " tuned" : "");
  } else if (p->sync_kernel == HEAT1D_SYNC_STEP) {
    std::snprintf(buf, sizeof buf, "step N=%lld rods=%lld", (long long)p->N, (long long)p->nrods);
  } else if (p->sync_kernel == HEAT1D_SYNC_RESIDENT) {
    std::snprintf(buf, sizeof buf, "resident N=%lld rods=%lld waves=%d M=%d", (long long)p->N,
                  (long long)p->nrods, p->waves, p->M);
  } else {
    std::snprintf(buf, sizeof buf, "%s N=%lld rods=%lld T=%d M=%d S=%d W=%d",
                  p->sync_kernel == HEAT1D_SYNC_PIPELINED ? "pipelined" : "tiled",
                  (long long)p->N, (long long)p->nrods, p->T, p->M, p->fuse,
                  p->sync_kernel == HEAT1D_SYNC_TILED ? p->tile_waves : 1);
  }
  p->desc = buf;
  if (p->band_from > 0) p->desc += " band_from=" + std::to_string(p->band_from);
}

// Default synchronous choice before any tuning.
void default_sync_choice(heat1d_plan_t p) {
  const int mmax = p->dtype == HEAT1D_F32 ? 64 : 32;
  if (p->N <= 16LL * 64 * mmax && p->nrods <= 4096) {
    p->sync_kernel = HEAT1D_SYNC_RESIDENT;
    p->waves = 16;
    p->M = smallest_m(p->dtype, (p->N + 1023) / 1024, resident_supports);
  } else {
    p->sync_kernel = HEAT1D_SYNC_TILED;
    p->M = p->dtype == HEAT1D_F32 ? 32 : 32;
    p->T = 32;
  }
}

int validate_opts(const heat1d_opts* o, int dtype) {
  if (!o) return HEAT1D_OK;
  if (o->sync_kernel < 0 || o->sync_kernel > HEAT1D_SYNC_PIPELINED) return HEAT1D_EINVAL;
  if (o->depth_t < 0 || o->depth_t > 256) return HEAT1D_EINVAL;
  if (o->waves < 0 || o->waves > 16) return HEAT1D_EINVAL;
  if (o->pts_per_lane < 0 || o->pts_per_lane > 64) return HEAT1D_EINVAL;
  if (o->max_delay < 0 || o->max_delay > 255) return HEAT1D_EINVAL;
  if (o->nsub < 0 || o->watchdog_polls < 0 || o->ckpt_stride < 0 || o->nrods < 0)
    return HEAT1D_EINVAL;
  if (o->fuse_steps != 0 && o->fuse_steps != 1 && o->fuse_steps != 2 && o->fuse_steps != 4 &&
      o->fuse_steps != 8)
    return HEAT1D_EINVAL;
  if (o->jitter < 0 || o->jitter > 65536) return HEAT1D_EINVAL;
  if (o->boundary != HEAT1D_BC_DIRICHLET && o->boundary != HEAT1D_BC_PERIODIC) return HEAT1D_EINVAL;
  if (o->grad_sum != 0 && o->grad_sum != 1) return HEAT1D_EINVAL;
  if (o->delay_schedule < 0 || o->delay_schedule > 2) return HEAT1D_EINVAL;
  (void)dtype;
  return HEAT1D_OK;
}

// Asynchronous geometry: (waves, M) holding ceil(N/P) points per workgroup.
// The fewest wavefronts whose registers hold the subdomain: fewer wavefronts
// mean fewer workgroup barriers per step, and P workgroups must all be
// resident at once.
bool async_geometry(heat1d_plan_t p, int P, int* waves, int* M) {
  const int64_t S = (p->N + P - 1) / P;
  if (p->opts.waves > 0 && p->opts.pts_per_lane > 0) {
    *waves = p->opts.waves;
    *M = p->opts.pts_per_lane;
    return async_supports(p->dtype, *M) && (int64_t)(*waves) * 64 * (*M) >= S;
  }
  for (int w = 1; w <= 16; w *= 2) {
    if (p->opts.waves > 0 && w != p->opts.waves) continue;
    const int64_t need = (S + 64LL * w - 1) / (64LL * w);
    const int m = smallest_m(p->dtype, need, async_supports);
    if (m > 0) {
      *waves = w;
      *M = m;
      return true;
    }
  }
  return false;
}

// Halo ring: P subdomains x 2 edges x Q slots; a slot is one tagged 64-bit
// word per 32 bits of value (one for FP32, two for FP64).
size_t async_ring_bytes(heat1d_plan_t p, int P) {
  const int Q = 2 * p->max_delay + 2;
  const size_t words = p->dtype == HEAT1D_F32 ? 1 : 2;
  return align_up((size_t)P * 2 * Q * words * 8);
}

// Asynchronous workspace: the halo ring, the progress hints and the status
// words, then what a run by strips needs: weights, a flag, the edges' histories
// and a state to alternate with.  The whole of it stays within what the
// allocation-free run has, so that both entry points take the same route: a
// plan whose histories do not fit never runs by strips, one whose state does
// not fit only where a single stage does.
struct AsyncLayout {
  size_t hint_off, err_off, base;          // base: without the strips
  size_t w_off, flag_off, hist_off, ping_off, total;
  bool strips, ping;
};
AsyncLayout async_layout(heat1d_plan_t p, int P) {
  AsyncLayout a{};
  a.hint_off = async_ring_bytes(p, P);
  a.err_off = a.hint_off + align_up((size_t)P * 2 * 4);
  a.base = a.err_off + align_up(2 * 4);
  a.w_off = a.base;
  a.flag_off = a.w_off + kBandWeightBytes;
  a.hist_off = a.flag_off + align_up(4);
  a.ping_off = a.hist_off + strip_history_bytes(p->dtype, P);
  const size_t state = align_up((size_t)p->N * esize(p->dtype));
  a.strips = P >= 2 && p->opts.sync_kernel == HEAT1D_SYNC_AUTO && p->opts.jitter == 0 &&
             band_applies(p->dtype, p->N, 1) && a.ping_off <= kNoAllocScratchBytes;
  a.ping = a.strips && a.ping_off + state <= kNoAllocScratchBytes;
  a.total = a.ping ? a.ping_off + state : (a.strips ? a.ping_off : a.base);
  return a;
}

// The periodic ring runs in the ensemble entry points (runs and their adjoint),
// heat1d_run_sync / heat1d_autotune_sync / heat1d_run_sync_observed and the
// asynchronous run; every other entry point is written for the Dirichlet rod.
bool periodic(heat1d_plan_t p) { return p->opts.boundary == HEAT1D_BC_PERIODIC; }

int plan_nsub(heat1d_plan_t p) {
  if (p->opts.nsub > 0) return p->opts.nsub;
  return (int)std::min<int64_t>(1024, std::max<int64_t>(1, p->N / 16384));
}

// Adjoint layout: checkpoints every S steps (the forward pass writes them),
// the starts of the sub-stretches of one stretch, one lambda buffer, and one
// partial dL/dr sum per (rod, sub-stretch launch, tile), contiguous per rod.
struct AdjLayout {
  int S;
  int64_t nseg;      // stretches
  int64_t nlaunch;   // sub-stretch launches of the whole backward sweep
  TileGeom g;        // forward passes (T = S)
  TileGeom gsub;     // sub-stretch start recomputation (T = stretch_steps(dtype))
  TileGeom gs;       // register-resident sub-stretch kernel
  size_t state_bytes;
  size_t ckpt_off, sub_off, lam_off, part_off, rod_off, total;
};

// The FP64 adjoint by band passes, on plans that name no synchronous kernel (the
// FP32 gradients stay those of the stepped states: dL/dr sums their roundings,
// 3e-7 of it, in double).  All
// the matrices of the run commute: with A the step and D the second difference,
// u(K) = A^K u0 (ends included), lambda(0) = A^K gK and
//   dL/dr = sum_k lambda(k+1) . D u(k) = K gK . (D A^(K-1) u0),
// so the forward pass leaves z = D A^(K-1) u0 (one state) in the workspace in
// place of the checkpoints, and the backward pass is one product and one dot
// product.  z comes from weights of its own, not from differences of u(K),
// whose rounding would be as large as z.
struct BandAdjLayout {
  size_t z_off, ping_off, spare_off, scr_off, part_off, rod_off, total;
};

// Few steps are as fast from the checkpoints: forward and backward together, in
// us, stepped / by passes, at K = 16 / 24 / 32 / 48: 100 points 28/34, 33/34,
// 33/34, 43/34; 4096 rods of 1025 points 105/105, 168/127, 182/128, 265/151;
// 2^22 points 75/76, 119/85, 122/87, 171/102.  Rods of 257 to 1023 points in
// numbers that fill the chip take a block of eight wavefronts per 256 points:
// 4096 of 700 points 66/127, 104/143, 108/145, 152/164 (64: 194/168).
int64_t band_adjoint_from(heat1d_plan_t p) {
  return p->N > 256 && p->N < 1024 && p->nrods >= 512 ? 56 : 24;
}
bool band_adjoint(heat1d_plan_t p, int64_t K) {
  const int64_t from = band_adjoint_from(p);
  // r is known to the calls only: at 1/2 a rod decays fastest.  Passes cut for that
  // are of `from` steps or more, whatever K is.
  return p->dtype == HEAT1D_F64 && p->opts.sync_kernel == HEAT1D_SYNC_AUTO && K >= from &&
         band_applies(p->dtype, p->N, p->nrods) &&
         band_decay(0.5, (double)K, p->N, false) <= kBandDecayRun &&
         band_decay(0.5, 2.0 * (double)from, p->N, false) <= kBandDecay;
}

BandAdjLayout band_adjoint_layout(heat1d_plan_t p, int64_t K) {
  BandAdjLayout a{};
  const size_t st = align_up((size_t)p->N * p->nrods * esize(p->dtype));
  // r = 1/2 reaches furthest and decays fastest: no r takes more passes
  const bool one = band_run(p->dtype, 0.5, K, p->N, false).passes <= 1;
  a.z_off = 0;
  a.ping_off = st;
  a.spare_off = a.ping_off + (one ? 0 : st);
  a.scr_off = a.spare_off + (one ? 0 : st);
  a.part_off = a.scr_off + band_scratch_bytes(p->N, p->nrods);
  a.rod_off = a.part_off +
              align_up((size_t)band_tiles(p->dtype, p->N, p->nrods) * p->nrods * 8);
  a.total = a.rod_off + align_up((size_t)p->nrods * 8);
  return a;
}

AdjLayout adjoint_layout(heat1d_plan_t p, int64_t K) {
  AdjLayout a{};
  const int S2 = stretch_steps(p->dtype);
  // default: about sqrt(K) steps between checkpoints, rounded up to whole
  // sub-stretches so that every sub-stretch but the run's last is full length
  int S = p->ckpt_stride;
  if (S <= 0) {
    S = (int)std::ceil(std::sqrt((double)std::max<int64_t>(K, 1)));
    S = (S + S2 - 1) / S2 * S2;
  }
  S = std::max(1, std::min(S, 480));
  a.S = S;
  a.nseg = K > 0 ? (K + S - 1) / S : 0;
  a.nlaunch = 0;
  for (int64_t j = 0; j < a.nseg; ++j) {
    const int64_t len = std::min<int64_t>(S, K - j * S);
    a.nlaunch += (len + S2 - 1) / S2;
  }
  a.g = tile_geometry(p->dtype, 32, S, p->N);
  a.gsub = tile_geometry(p->dtype, 32, S2, p->N);
  a.gs = stretch_geometry(p->dtype, p->N);
  a.state_bytes = align_up((size_t)p->N * p->nrods * esize(p->dtype));
  const int64_t nsub_max = (S + S2 - 1) / S2;
  a.ckpt_off = 0;
  a.sub_off = a.ckpt_off + (size_t)std::max<int64_t>(a.nseg, 1) * a.state_bytes;
  a.lam_off = a.sub_off + (size_t)std::max<int64_t>(nsub_max - 1, 1) * a.state_bytes;
  a.part_off = a.lam_off + a.state_bytes;
  a.rod_off = a.part_off + align_up((size_t)std::max<int64_t>(a.nlaunch, 1) * p->nrods *
                                    std::max<int64_t>(a.gs.tiles_per_rod, 1) * 8);
  // per-rod dL/dr when the plan reports their sum (opts.grad_sum)
  a.total = a.rod_off + align_up((size_t)p->nrods * 8);
  return a;
}

// Layout of the asynchronous adjoint's workspace: checkpoints u(c S) for the
// stretches c = 0..nck-1, the S-1 states inside one stretch, u(K) when the
// caller passes no uK, two lambda states, the edge records E and LE, the
// partition table, the per-workgroup dL/dr partials and the two end sums.
struct AsyncAdjLayout {
  int S;
  int64_t nck;
  bool tiled;      // register tiles, else one launch per step
  int64_t nparts;  // dL/dr partials: one per workgroup of a step launch or per tile
  size_t state_bytes, rec_bytes;
  size_t ck_off, st_off, fin_off, lam_off, E_off, LE_off, lo_off, part_off, ends_off, ord_off,
      ord_bytes, total;
};

AsyncAdjLayout async_adjoint_layout(heat1d_plan_t p, int64_t K, int P) {
  AsyncAdjLayout a{};
  int64_t S = p->ckpt_stride > 0 ? p->ckpt_stride
                                 : (int64_t)std::ceil(std::sqrt((double)std::max<int64_t>(K, 1)));
  S = std::max<int64_t>(1, std::min<int64_t>(S, std::max<int64_t>(K, 1)));
  a.S = (int)S;
  a.nck = K > 0 ? (K + S - 1) / S : 1;
  a.state_bytes = align_up((size_t)p->N * esize(p->dtype));
  a.rec_bytes = align_up((size_t)(K + 1) * P * 2 * esize(p->dtype));
  a.ck_off = 0;
  a.st_off = a.ck_off + (size_t)a.nck * a.state_bytes;
  a.fin_off = a.st_off + (size_t)(S - 1) * a.state_bytes;
  a.lam_off = a.fin_off + a.state_bytes;
  a.E_off = a.lam_off + 2 * a.state_bytes;
  a.LE_off = a.E_off + a.rec_bytes;
  a.lo_off = a.LE_off + a.rec_bytes;
  a.part_off = a.lo_off + align_up((size_t)(P + 1) * 8);
  const int64_t blocks = async_adjoint_blocks(p->N);
  const int64_t tiles =
      async_tiled_from(p->N, P) > 0 ? async_tiled_tiles(p->dtype, p->N, P) : 0;
  a.tiled = p->opts.sync_kernel != HEAT1D_SYNC_STEP && tiles > 0 && K >= async_tiled_from(p->N, P);
  a.nparts = a.tiled ? tiles : blocks;
  a.ends_off = a.part_off + align_up((size_t)std::max(blocks, tiles) * 8);
  a.ord_off = a.ends_off + align_up(16);
  a.ord_bytes = align_up((size_t)tiles * 4);
  a.total = a.ord_off + 2 * a.ord_bytes;
  return a;
}

// Sync workspace: one state, the other half of the ping-pong pair.
size_t sync_state_bytes(heat1d_plan_t p) {
  return align_up((size_t)p->N * p->nrods * esize(p->dtype));
}

// K steps of nrods rods as band passes (heat1d_band.h): K is cut into equal
// passes that alternate between out and ping (which a single pass does not
// touch); the last one leaves u(K) in out, and D A^(K-1) u0 in z when z is
// given.  dot: K times the partial sums of the input with dot_with.  out may be
// NULL where a single pass only wants z.  scratch: band_scratch_bytes.
int run_band(heat1d_plan_t p, int64_t nrods, const void* in, void* out, double r, double c1,
             double cN, int64_t K, void* ping, void* scratch, void* z, const void* dot_with,
             double* dot, hipStream_t s) {
  BandPass b;
  b.dot_scale = (double)K;
  b.dtype = p->dtype;
  b.r = p->dtype == HEAT1D_F32 ? (double)(float)r : r;
  const BandRun run = band_run(p->dtype, b.r, K, p->N, periodic(p));
  b.N = p->N;
  b.nrods = nrods;
  b.c1 = c1;
  b.cN = cN;
  b.ring = p->opts.boundary == HEAT1D_BC_PERIODIC;
  b.scratch = scratch;
  for (int64_t i = 0; i < run.passes; ++i) {
    const bool last = i + 1 == run.passes;
    const int64_t T = last ? K - i * run.T : run.T;
    b.in = i == 0 ? in : b.out;
    b.out = (run.passes - 1 - i) % 2 == 0 ? out : ping;
    b.z = last ? z : nullptr;
    b.dot = i == 0 ? dot : nullptr;
    b.dot_with = dot_with;
    hipError_t e = hipSuccess;
    if (i == 0 || T != b.T || b.z != nullptr) {
      b.T = T;
      b.slot = 0;  // the weights' launch clears both flags
      e = launch_band_weights(b, s);
    } else {
      b.slot = 1 - b.slot;
    }
    if (e != hipSuccess) return hip_status(e);
    EventPair* ev = timing_begin(p, s);
    e = launch_band_pass(b, s);
    timing_end(ev, s);
    if (e == hipSuccess) e = launch_band_cones(b, s);
    if (e != hipSuccess) return hip_status(e);
  }
  return HEAT1D_OK;
}

// Whether K steps, of a run of `of` steps in all, take band passes: not where they
// would have to be cut, for what they take off the state, below the steps from which
// a pass is faster.
bool takes_band(heat1d_plan_t p, double r, int64_t K, int64_t of, const void* ws) {
  if (p->band_from == 0 || K < p->band_from || ws == nullptr || fp32_drifts(p->dtype, r, of))
    return false;
  const bool ring = periodic(p);
  return band_decay(r, (double)of, p->N, ring) <= kBandDecayRun &&
         band_run(p->dtype, r, K, p->N, ring).T >= p->band_from;
}

int run_sync_impl(heat1d_plan_t p, const void* u0, void* uK, double r, double c1, double cN,
                  int64_t K, void* ws, hipStream_t s, int kernel, int T, int M, int waves,
                  int fuse) {
  const int64_t N = p->N, B = p->nrods;
  if (periodic(p)) {
    // the ring (Section 5.3): no end values; one launch per step or ring tiles
    if (K == 0)
      return hip_status(hipMemcpyAsync(uK, u0, (size_t)N * B * esize(p->dtype),
                                       hipMemcpyDeviceToDevice, s));
    const bool step = kernel == HEAT1D_SYNC_STEP;
    const bool wide = !step && waves > 1;  // ring tiles of `waves` wavefronts
    const TileGeom g = ring_geometry(p->dtype, wide ? M * waves : M, T, N);
    if (!step && g.tiles_per_rod <= 0) return HEAT1D_EINVAL;
    const int64_t passes = step ? K : (K + T - 1) / T;
    for (int64_t i = 0; i < passes; ++i) {
      const int steps = step ? 1 : (int)std::min<int64_t>(T, K - i * T);
      const void* in = (i == 0) ? u0 : (((passes - i) % 2 == 0) ? uK : ws);
      void* out = ((passes - 1 - i) % 2 == 0) ? uK : ws;
      EventPair* e = timing_begin(p, s);
      hipError_t err =
          step   ? launch_sync_step(p->dtype, in, out, N, B, r, c1, cN, s, true)
          : wide ? launch_sync_wide_ring(p->dtype, g, M, waves, in, out, N, B, steps, r, fuse, s)
                 : launch_sync_ring(p->dtype, g, in, out, N, B, steps, r, fuse, s);
      timing_end(e, s);
      if (err != hipSuccess) return hip_status(err);
    }
    return HEAT1D_OK;
  }
  if (K == 0) return hip_status(launch_impose_ends(p->dtype, u0, uK, N, B, c1, cN, s));
  if (kernel == HEAT1D_SYNC_RESIDENT) {
    EventPair* e = timing_begin(p, s);
    hipError_t err = launch_sync_resident(p->dtype, M, waves, u0, uK, N, B, K, r, c1, cN, s);
    timing_end(e, s);
    return hip_status(err);
  }
  if (kernel == HEAT1D_SYNC_STEP) {
    for (int64_t i = 0; i < K; ++i) {
      const void* in = (i == 0) ? u0 : (((K - i) % 2 == 0) ? uK : ws);
      void* out = ((K - 1 - i) % 2 == 0) ? uK : ws;
      EventPair* e = timing_begin(p, s);
      hipError_t err = launch_sync_step(p->dtype, in, out, N, B, r, c1, cN, s);
      timing_end(e, s);
      if (err != hipSuccess) return hip_status(err);
    }
    return HEAT1D_OK;
  }
  if (kernel == HEAT1D_SYNC_TILED && waves > 1) {
    // wide tiles: `waves` wavefronts per tile
    const TileGeom gw = tile_geometry(p->dtype, M * waves, T, N);
    if (gw.tiles_per_rod <= 0) return HEAT1D_EINVAL;
    const int64_t passes = (K + T - 1) / T;
    for (int64_t i = 0; i < passes; ++i) {
      const int steps = (int)std::min<int64_t>(T, K - i * T);
      const void* in = (i == 0) ? u0 : (((passes - i) % 2 == 0) ? uK : ws);
      void* out = ((passes - 1 - i) % 2 == 0) ? uK : ws;
      EventPair* e = timing_begin(p, s);
      hipError_t err =
          launch_sync_wide(p->dtype, gw, M, waves, in, out, N, B, steps, r, c1, cN, fuse, s);
      timing_end(e, s);
      if (err != hipSuccess) return hip_status(err);
    }
    return HEAT1D_OK;
  }
  const TileGeom g = tile_geometry(p->dtype, M, T, N);
  if (g.tiles_per_rod <= 0) return HEAT1D_EINVAL;
  const int64_t passes = (K + T - 1) / T;
  for (int64_t i = 0; i < passes; ++i) {
    const int steps = (int)std::min<int64_t>(T, K - i * T);
    const void* in = (i == 0) ? u0 : (((passes - i) % 2 == 0) ? uK : ws);
    void* out = ((passes - 1 - i) % 2 == 0) ? uK : ws;
    EventPair* e = timing_begin(p, s);
    hipError_t err =
        (kernel == HEAT1D_SYNC_PIPELINED && pipelined_applies(p->dtype, g, in, out, N))
            ? launch_sync_pipelined(p->dtype, g, in, out, N, B, steps, r, c1, cN, fuse, s)
            : launch_sync_tiled(p->dtype, g, in, out, N, B, steps, r, c1, cN, fuse, s);
    timing_end(e, s);
    if (err != hipSuccess) return hip_status(err);
  }
  return HEAT1D_OK;
}

// run_sync_impl with the plan's kernel, or band passes where the plan leaves the
// choice open and the run is long enough: K steps of a run of `of` steps in all.
// ws: heat1d_sync_workspace_bytes.
int run_sync_plan(heat1d_plan_t p, const void* u0, void* uK, double r, double c1, double cN,
                  int64_t K, int64_t of, void* ws, hipStream_t s) {
  if (takes_band(p, r, K, of, ws))
    return run_band(p, p->nrods, u0, uK, r, c1, cN, K, ws, (char*)ws + sync_state_bytes(p),
                    nullptr, nullptr, nullptr, s);
  return run_sync_impl(p, u0, uK, r, c1, cN, K, ws, s, p->sync_kernel, p->T, p->M,
                       p->sync_kernel == HEAT1D_SYNC_TILED ? p->tile_waves : p->waves, p->fuse);
}

// Split the rods of a batched plan into the three queues, each longest N*K
// first: at most t_wave points run on one wavefront, at most t_group on a
// 4-wavefront group, the rest on the whole workgroup.  The thresholds are
// clamped to what each block holds; opts.waves forces the smallest block a rod
// may run on (16: every rod on a whole workgroup, 2..15: no single-wavefront
// rods).
void batched_assign(heat1d_plan_t p, int64_t t_wave, int64_t t_group) {
  t_wave = std::min<int64_t>(std::max<int64_t>(t_wave, 0), batched_wave_capacity(p->dtype));
  t_group = std::min<int64_t>(std::max<int64_t>(t_group, t_wave),
                              batched_group_capacity(p->dtype));
  if (p->opts.waves >= 16) t_wave = t_group = 0;
  else if (p->opts.waves >= 2) t_wave = 0;
  p->t_wave = t_wave;
  p->t_group = t_group;
  for (auto& q : p->order) q.clear();
  for (int32_t b : p->by_work) {
    const int q = p->Nh[b] <= t_wave ? 2 : (p->Nh[b] <= t_group ? 1 : 0);
    p->order[q].push_back(b);
  }
}

// Take the rods of at least kBatchBandFrom steps out of the queues (by_work):
// they run as band passes, in tiles, the most work first.  Room for the weights
// of any r; a rod whose reach could pass kBandMaxReach stays in the queues, and
// so does every rod of a plan that names a block size (opts.waves).
void batched_split_band(heat1d_plan_t p) {
  if (p->opts.waves > 0 || p->opts.sync_kernel != HEAT1D_SYNC_AUTO) return;
  std::vector<int32_t> rest;
  int64_t tiles = 0, w = 0;
  for (int32_t b : p->by_work) {
    const int h = band_reach_bound(p->dtype, 0.5, std::max(p->Kh[b], 1));
    const int64_t nt = (p->Nh[b] + kBandBatchTile - 1) / kBandBatchTile;
    // r is known on the device only, when the rod's place has long been chosen: the
    // line is that of r = 1/2, 5166 steps, whatever r is.  (A line by each rod's r
    // would send rods of small r back to the queues, for results that are further off:
    // a smooth rod, r = 0.05, K = 5000, is 1.0e-4 off there and 4e-7 by a pass.)
    if (p->Kh[b] < kBatchBandFrom || fp32_drifts(p->dtype, 0.5, p->Kh[b]) ||
        h > kBandMaxReach || tiles + nt > (1 << 22) || w + h + 1 > INT32_MAX ||
        (p->Nh[b] > kBandBatchStep && band_decay(0.5, p->Kh[b], p->Nh[b], false) > kBandDecay)) {
      rest.push_back(b);
      continue;
    }
    for (int64_t t = 0; t < nt; ++t)
      p->band_items.push_back({(int32_t)p->band_rods.size(), (int32_t)t});
    p->band_rods.push_back(b);
    p->band_woff.push_back((int32_t)w);
    p->band_hmax = std::max(p->band_hmax, h);
    p->band_short |= band_decay(0.5, p->Kh[b], p->Nh[b], false) > kBandDecay;
    tiles += nt;
    w += h + 1;
  }
  p->band_woff.push_back((int32_t)w);
  p->by_work = rest;
}

// Workgroups that take the group and wavefront queues first: about twice
// those queues' share of the point updates (their rods keep fewer points per
// wavefront busy per step), at most half the grid, all of it when no rod
// needs a whole workgroup.
int batched_rule_small_first(heat1d_plan_t p) {
  double lw[3] = {0, 0, 0};
  for (int q = 0; q < 3; ++q)
    for (int32_t b : p->order[q]) lw[q] += (double)(p->Nh[b] - 2) * (double)p->Kh[b];
  const double small = lw[1] + lw[2], all = lw[0] + small;
  if (p->order[0].empty()) return p->groups;
  if (small <= 0) return 0;
  return std::min(p->groups / 2 > 0 ? p->groups / 2 : 1,
                  (int)std::ceil(p->groups * 2.0 * small / all));
}

}  // namespace

extern "C" {

const char* heat1d_version(void) { return "heat1d 0.2 gfx950"; }

int heat1d_fused_weights(int32_t dtype, double r, int32_t S, double* w) {
  if ((dtype != HEAT1D_F32 && dtype != HEAT1D_F64) || !r_ok(r) || (S != 2 && S != 4 && S != 8) ||
      !w)
    return HEAT1D_EINVAL;
  if (dtype == HEAT1D_F32) {
    const StepWeights<float> sw = step_weights<float>(r, S);
    for (int d = 0; d <= S; ++d) w[d] = sw.w[d];
  } else {
    const StepWeights<double> sw = step_weights<double>(r, S);
    for (int d = 0; d <= S; ++d) w[d] = sw.w[d];
  }
  return HEAT1D_OK;
}

const char* heat1d_strerror(int status) {
  switch (status) {
    case HEAT1D_OK: return "ok";
    case HEAT1D_EINVAL: return "invalid argument";
    case HEAT1D_EUNSUPPORTED: return "unsupported configuration";
    case HEAT1D_EOCCUPANCY: return "persistent kernel cannot keep all workgroups resident";
    case HEAT1D_ETIMEOUT: return "asynchronous kernel watchdog expired";
    case HEAT1D_EHIP: return "HIP runtime error";
    case HEAT1D_ESCRATCH:
      return "run needs more scratch than the fixed allocation-free array holds (4 MiB)";
    default: return "unknown status";
  }
}

int heat1d_plan_create(heat1d_plan_t* out, int64_t N, int32_t dtype, const heat1d_opts* opts) {
  if (!out) return HEAT1D_EINVAL;
  *out = nullptr;
  if (N < 3 || (dtype != HEAT1D_F32 && dtype != HEAT1D_F64)) return HEAT1D_EINVAL;
  if (N > (int64_t(1) << 40)) return HEAT1D_EINVAL;
  if (validate_opts(opts, dtype) != HEAT1D_OK) return HEAT1D_EINVAL;
  heat1d_plan_t p = new heat1d_plan_s();
  p->N = N;
  p->dtype = dtype;
  if (opts) p->opts = *opts;
  p->nrods = p->opts.nrods > 0 ? p->opts.nrods : 1;
  if (p->opts.max_delay > 0) p->max_delay = p->opts.max_delay;
  if (p->opts.watchdog_polls > 0) p->watchdog = p->opts.watchdog_polls;
  p->ckpt_stride = p->opts.ckpt_stride;
  default_sync_choice(p);
  // explicit choices.  On an asynchronous plan (nsub > 0) with no explicit
  // synchronous kernel, waves and pts_per_lane shape the asynchronous kernel
  // only and the synchronous kernel keeps its defaults.
  heat1d_opts o = p->opts;
  if (o.nsub > 0 && o.sync_kernel == HEAT1D_SYNC_AUTO) {
    o.waves = 0;
    o.pts_per_lane = 0;
  }
  if (o.sync_kernel != HEAT1D_SYNC_AUTO) p->sync_kernel = o.sync_kernel;
  if (p->sync_kernel == HEAT1D_SYNC_TILED || p->sync_kernel == HEAT1D_SYNC_PIPELINED) {
    if (o.depth_t > 0) p->T = o.depth_t;
    if (o.pts_per_lane > 0) p->M = o.pts_per_lane;
    else if (p->M == 0 || !tiled_supports(dtype, p->M)) p->M = 32;
    if (!tiled_supports(dtype, p->M)) { delete p; return HEAT1D_EUNSUPPORTED; }
    p->fuse = o.fuse_steps > 0 ? o.fuse_steps : 1;
    const bool wide = p->sync_kernel == HEAT1D_SYNC_TILED && o.waves > 1;
    if (!wide && !fused_supports(dtype, p->M, p->fuse)) { delete p; return HEAT1D_EUNSUPPORTED; }
    if (wide) {
      p->tile_waves = o.waves;
      if (!wide_supports(dtype, p->M, p->fuse, p->tile_waves) ||
          tile_geometry(dtype, p->M * p->tile_waves, p->T, N).tiles_per_rod <= 0) {
        delete p;
        return HEAT1D_EUNSUPPORTED;
      }
    }
    if (tile_geometry(dtype, p->M, p->T, N).tiles_per_rod <= 0) { delete p; return HEAT1D_EINVAL; }
  } else if (p->sync_kernel == HEAT1D_SYNC_RESIDENT && o.boundary != HEAT1D_BC_PERIODIC) {
    if (o.waves > 0) p->waves = o.waves;
    if (o.pts_per_lane > 0) p->M = o.pts_per_lane;
    else p->M = smallest_m(dtype, (N + 64LL * p->waves - 1) / (64LL * p->waves), resident_supports);
    if (p->M == 0 || !resident_supports(dtype, p->M) || (int64_t)p->waves * 64 * p->M < N) {
      delete p;
      return HEAT1D_EUNSUPPORTED;
    }
  }
  if (o.boundary == HEAT1D_BC_PERIODIC && p->sync_kernel != HEAT1D_SYNC_STEP) {
    // the synchronous ring runs one launch per step or ring tiles of one
    // wavefront (narrow) or of opts.waves wavefronts (wide)
    if (o.sync_kernel == HEAT1D_SYNC_RESIDENT || o.sync_kernel == HEAT1D_SYNC_PIPELINED) {
      delete p;
      return HEAT1D_EUNSUPPORTED;
    }
    const bool wide = o.sync_kernel == HEAT1D_SYNC_TILED && o.waves > 1;
    p->sync_kernel = HEAT1D_SYNC_TILED;
    p->tile_waves = wide ? o.waves : 1;
    p->T = o.depth_t > 0 ? o.depth_t : 32;
    p->M = o.pts_per_lane > 0 ? o.pts_per_lane : (dtype == HEAT1D_F32 ? 32 : 16);
    p->fuse = o.fuse_steps > 0 ? o.fuse_steps : 1;
    const bool ok = wide ? wide_supports(dtype, p->M, p->fuse, p->tile_waves)
                         : fused_supports(dtype, p->M, p->fuse);
    if (!ok || ring_geometry(dtype, p->M * p->tile_waves, p->T, N).tiles_per_rod <= 0) {
      delete p;
      return HEAT1D_EUNSUPPORTED;
    }
  }
  // A plan that names no synchronous kernel, tile or sweep leaves the choice to
  // the run's length.
  if (o.sync_kernel == HEAT1D_SYNC_AUTO && o.depth_t == 0 && o.pts_per_lane == 0 &&
      o.waves == 0 && o.fuse_steps == 0 && band_applies(dtype, N, p->nrods))
    p->band_from = band_from_steps(dtype, N, p->nrods, o.boundary == HEAT1D_BC_PERIODIC);
  describe(p);
  *out = p;
  return HEAT1D_OK;
}

int heat1d_plan_batched(heat1d_plan_t* out, int32_t nrods, const int64_t* N_host,
                        const int32_t* K_host, int32_t dtype, const heat1d_opts* opts) {
  if (!out) return HEAT1D_EINVAL;
  *out = nullptr;
  if (nrods < 1 || !N_host || !K_host || (dtype != HEAT1D_F32 && dtype != HEAT1D_F64))
    return HEAT1D_EINVAL;
  if (validate_opts(opts, dtype) != HEAT1D_OK) return HEAT1D_EINVAL;
  if (opts && opts->boundary != HEAT1D_BC_DIRICHLET) return HEAT1D_EUNSUPPORTED;
  const int wave_cap = batched_wave_capacity(dtype);
  const int group_cap = batched_group_capacity(dtype);
  const int wg_cap = batched_wg_capacity(dtype);
  for (int32_t b = 0; b < nrods; ++b) {
    if (N_host[b] < 3 || K_host[b] < 0) return HEAT1D_EINVAL;
    if (N_host[b] > wg_cap) return HEAT1D_EUNSUPPORTED;
  }
  heat1d_plan_t p = new heat1d_plan_s();
  p->batched = true;
  p->dtype = dtype;
  if (opts) p->opts = *opts;
  p->Nh.assign(N_host, N_host + nrods);
  p->Kh.assign(K_host, K_host + nrods);
  p->N = *std::max_element(p->Nh.begin(), p->Nh.end());
  p->by_work.resize(nrods);
  std::iota(p->by_work.begin(), p->by_work.end(), 0);
  std::stable_sort(p->by_work.begin(), p->by_work.end(), [&](int32_t a, int32_t b) {
    return (double)p->Nh[a] * p->Kh[a] > (double)p->Nh[b] * p->Kh[b];
  });
  batched_split_band(p);
  p->groups = std::max(1, num_cus());
  batched_assign(p, wave_cap, group_cap);
  p->small_first = batched_rule_small_first(p);
  describe(p);
  *out = p;
  return HEAT1D_OK;
}

void heat1d_plan_destroy(heat1d_plan_t plan) {
  if (!plan) return;
  for (auto& e : plan->ev) {
    if (e.a) hipEventDestroy(e.a);
    if (e.b) hipEventDestroy(e.b);
  }
  delete plan;
}

const char* heat1d_plan_describe(heat1d_plan_t plan) {
  if (!plan) return "";
  return plan->desc.c_str();
}

size_t heat1d_sync_workspace_bytes(heat1d_plan_t p) {
  if (!p || p->batched) return 0;
  return sync_state_bytes(p) + (p->band_from > 0 ? band_scratch_bytes(p->N, p->nrods) : 0);
}

size_t heat1d_async_workspace_bytes(heat1d_plan_t p) {
  if (!p || p->batched) return 0;
  return async_layout(p, plan_nsub(p)).total;
}

size_t heat1d_adjoint_workspace_bytes(heat1d_plan_t p, int64_t K) {
  if (!p || p->batched || K < 0) return 0;
  // a workspace for K steps also serves fewer, whichever way those go
  const int64_t from = band_adjoint_from(p);
  const bool band = band_adjoint(p, K);
  size_t n = adjoint_layout(p, band ? from - 1 : K).total;
  if (K >= from && band_adjoint(p, from)) n = std::max(n, band_adjoint_layout(p, K).total);
  return n;
}

// Batched workspace: the three queues (int32, 256-byte aligned) and three heads.
namespace {
// Every queue has room for all rods, so the layout does not depend on how the
// rods are split (the autotuner re-splits them in place).
size_t batched_queue_off(heat1d_plan_t p, int q) {
  return (size_t)q * align_up(p->Nh.size() * 4 + 4);
}
// Behind the queues and their heads: the tiles, rods and weight offsets of the
// band passes, their flag, records and weights.
struct BatchedBandLayout {
  size_t items, rods, woff, slot, flag, rec, w, total;
};
BatchedBandLayout batched_band_layout(heat1d_plan_t p) {
  BatchedBandLayout L{};
  L.items = batched_queue_off(p, 3) + align_up(3 * 4);
  L.rods = L.items + align_up(p->band_items.size() * sizeof(BandItem));
  L.woff = L.rods + align_up(p->band_rods.size() * 4);
  L.slot = L.woff + align_up(p->band_woff.size() * 4);
  L.flag = L.slot + align_up(p->band_rods.size() * kBandSlotBytes);
  L.rec = L.flag + align_up(4);
  L.w = L.rec + align_up(p->band_items.size() * 8);
  L.total = L.w + align_up((p->band_woff.empty() ? 0 : (size_t)p->band_woff.back()) *
                           esize(p->dtype));
  return L;
}
}  // namespace

size_t heat1d_batched_workspace_bytes(heat1d_plan_t p) {
  if (!p || !p->batched) return 0;
  return batched_band_layout(p).total;
}

int heat1d_set_timing(heat1d_plan_t plan, int32_t enable) {
  if (!plan) return HEAT1D_EINVAL;
  plan->timing = enable != 0;
  plan->ev_used = 0;
  return HEAT1D_OK;
}

double heat1d_last_kernel_ms(heat1d_plan_t plan, int64_t* launches) {
  if (launches) *launches = 0;
  if (!plan || plan->ev_used == 0) return -1.0;
  double total = 0.0;
  for (size_t i = 0; i < plan->ev_used; ++i) {
    if (hipEventSynchronize(plan->ev[i].b) != hipSuccess) return -1.0;
    float ms = 0.f;
    if (hipEventElapsedTime(&ms, plan->ev[i].a, plan->ev[i].b) != hipSuccess) return -1.0;
    total += ms;
  }
  if (launches) *launches = (int64_t)plan->ev_used;
  const double avg = total / (double)plan->ev_used;
  plan->ev_used = 0;
  return avg;
}

int heat1d_run_sync(heat1d_plan_t p, const void* u0, void* uK, double r, double c1, double cN,
                    int64_t K, void* workspace, void* stream) {
  if (!p || p->batched || !u0 || !uK || !r_ok(r) || K < 0) return HEAT1D_EINVAL;
  if (!std::isfinite(c1) || !std::isfinite(cN)) return HEAT1D_EINVAL;
  const size_t bytes = (size_t)p->N * p->nrods * esize(p->dtype);
  if (overlaps(u0, uK, bytes)) return HEAT1D_EINVAL;
  // the resident kernel needs no workspace, and is what runs when there is none
  const size_t wsb = heat1d_sync_workspace_bytes(p);
  const bool ws_ok = workspace && !overlaps(workspace, wsb, u0, bytes) &&
                     !overlaps(workspace, wsb, uK, bytes);
  if (K > 1 && p->sync_kernel != HEAT1D_SYNC_RESIDENT && !ws_ok) return HEAT1D_EINVAL;
  if (K > INT32_MAX) return HEAT1D_EUNSUPPORTED;
  return run_sync_plan(p, u0, uK, r, c1, cN, K, K, ws_ok ? workspace : nullptr,
                       (hipStream_t)stream);
}

size_t heat1d_observed_workspace_bytes(heat1d_plan_t p) {
  if (!p || p->batched) return 0;
  return align_up(heat1d_sync_workspace_bytes(p)) +
         align_up((size_t)p->N * p->nrods * esize(p->dtype)) +
         align_up((size_t)norm_partials(p->N, p->nrods) * 8);
}

int heat1d_run_sync_observed(heat1d_plan_t p, const void* u0, void* uK, double r, double c1,
                             double cN, int64_t K, int64_t every, double* norms, void* workspace,
                             void* stream) {
  if (!p || p->batched || !u0 || !uK || !norms || !workspace || !r_ok(r) || K < 0 || every < 1)
    return HEAT1D_EINVAL;
  if (!std::isfinite(c1) || !std::isfinite(cN)) return HEAT1D_EINVAL;
  const bool ring = periodic(p);
  if (K > INT32_MAX || p->nrods > 65535) return HEAT1D_EUNSUPPORTED;
  const int64_t N = p->N, B = p->nrods;
  const size_t bytes = (size_t)N * B * esize(p->dtype);
  const int64_t nobs = K / every + 1;
  const size_t nbytes = (size_t)B * nobs * 8;
  const size_t wsb = heat1d_observed_workspace_bytes(p);
  if (overlaps(u0, uK, bytes) || overlaps(workspace, wsb, u0, bytes) ||
      overlaps(workspace, wsb, uK, bytes) || overlaps(norms, nbytes, u0, bytes) ||
      overlaps(norms, nbytes, uK, bytes) || overlaps(norms, nbytes, workspace, wsb))
    return HEAT1D_EINVAL;
  hipStream_t s = (hipStream_t)stream;
  char* ws = (char*)workspace;
  char* extra = ws + align_up(heat1d_sync_workspace_bytes(p));
  double* partials = (double*)(extra + align_up(bytes));
  hipError_t e = launch_state_norms(p->dtype, u0, N, B, c1, cN, partials, norms, nobs, s, !ring);
  if (e != hipSuccess) return hip_status(e);
  const int64_t full = K / every, rem = K % every;
  const int64_t nchunks = full + (rem > 0 ? 1 : 0);
  const int waves = p->sync_kernel == HEAT1D_SYNC_TILED ? p->tile_waves : p->waves;
  if (nchunks == 0)
    return ring ? run_sync_impl(p, u0, uK, r, c1, cN, 0, ws, s, p->sync_kernel, p->T, p->M,
                                waves, p->fuse)
                : hip_status(launch_impose_ends(p->dtype, u0, uK, N, B, c1, cN, s));
  const void* in = u0;
  for (int64_t j = 1; j <= nchunks; ++j) {
    // the buffers alternate so that the last chunk lands in uK
    void* out = ((nchunks - j) % 2 == 0) ? uK : (void*)extra;
    const int64_t steps = j <= full ? every : rem;
    const int st = run_sync_plan(p, in, out, r, c1, cN, steps, K, ws, s);
    if (st != HEAT1D_OK) return st;
    if (j <= full) {
      e = launch_state_norms(p->dtype, out, N, B, c1, cN, partials, norms + j, nobs, s, !ring);
      if (e != hipSuccess) return hip_status(e);
    }
    in = out;
  }
  return HEAT1D_OK;
}

int heat1d_autotune_sync(heat1d_plan_t p, const void* u0, void* uK, double r, int64_t K_probe,
                         void* workspace, void* stream, double* best_ms) {
  if (!p || p->batched || !u0 || !uK || !workspace || !r_ok(r) || K_probe < 1) return HEAT1D_EINVAL;
  const bool ring = periodic(p);
  const size_t bytes = (size_t)p->N * p->nrods * esize(p->dtype);
  const size_t wsb = heat1d_sync_workspace_bytes(p);
  if (overlaps(u0, uK, bytes) || overlaps(workspace, wsb, u0, bytes) ||
      overlaps(workspace, wsb, uK, bytes))
    return HEAT1D_EINVAL;
  hipStream_t s = (hipStream_t)stream;
  struct Cand { int kernel, T, M, waves, fuse; };
  std::vector<Cand> cands;
  if (K_probe <= 4096) cands.push_back({HEAT1D_SYNC_STEP, 0, 0, 0, 1});
  const int Ms32[] = {8, 16, 24, 32, 40, 48, 64};
  const int Ms64[] = {4, 8, 12, 16, 20, 24, 32};
  const int Ts[] = {1, 2, 4, 8, 16, 24, 32, 48, 64, 96, 128, 192, 256};
  // the pipelined kernel needs every buffer of the ping-pong 16-byte aligned
  // and whole vectors per rod (its tile count is checked per candidate)
  const int V = vec_width(p->dtype);
  const bool pipelined_ok = p->N % V == 0 && ((uintptr_t)u0 & 15u) == 0 &&
                            ((uintptr_t)uK & 15u) == 0 && ((uintptr_t)workspace & 15u) == 0;
  for (int i = 0; i < 7; ++i) {
    const int M = p->dtype == HEAT1D_F32 ? Ms32[i] : Ms64[i];
    for (int T : Ts) {
      const TileGeom g = tile_geometry(p->dtype, M, T, p->N);
      const bool narrow = g.tiles_per_rod > 0 && 4 * g.H <= g.L;
      for (int S : {1, 2, 4, 8}) {
        if (p->opts.fuse_steps > 0 ? S != p->opts.fuse_steps : (S > 1 && S > T)) continue;
        if (narrow && fused_supports(p->dtype, M, S)) {
          cands.push_back({HEAT1D_SYNC_TILED, T, M, 0, S});
          if (!ring && pipelined_ok && g.tiles_per_rod >= 2 && p->N > g.L)
            cands.push_back({HEAT1D_SYNC_PIPELINED, T, M, 0, S});
        }
        for (int G : {4, 8}) {
          const TileGeom gw = tile_geometry(p->dtype, G * M, T, p->N);
          if (wide_supports(p->dtype, M, S, G) && gw.tiles_per_rod > 0 && 4 * gw.H <= gw.L)
            cands.push_back({HEAT1D_SYNC_TILED, T, M, G, S});
        }
      }
    }
  }
  for (int w = 1; w <= 16 && !ring; w *= 2) {
    const int64_t need = (p->N + 64LL * w - 1) / (64LL * w);
    const int m = smallest_m(p->dtype, need, resident_supports);
    if (m > 0) cands.push_back({HEAT1D_SYNC_RESIDENT, 0, m, w, 1});
  }
  hipEvent_t a, b;
  if (hipEventCreate(&a) != hipSuccess || hipEventCreate(&b) != hipSuccess) return HEAT1D_EHIP;
  double best = 1e300;
  Cand win = {p->sync_kernel, p->T, p->M,
              p->sync_kernel == HEAT1D_SYNC_TILED ? p->tile_waves : p->waves, p->fuse};
  const bool timing = p->timing;
  p->timing = false;
  int status = HEAT1D_OK;
  for (const Cand& c : cands) {
    // warm-up, then one timed run
    int st = run_sync_impl(p, u0, uK, r, 0.0, 0.0, K_probe, workspace, s, c.kernel, c.T, c.M,
                           c.waves, c.fuse);
    if (st != HEAT1D_OK) { status = st; break; }
    hipEventRecord(a, s);
    st = run_sync_impl(p, u0, uK, r, 0.0, 0.0, K_probe, workspace, s, c.kernel, c.T, c.M, c.waves,
                       c.fuse);
    hipEventRecord(b, s);
    if (st != HEAT1D_OK) { status = st; break; }
    if (hipEventSynchronize(b) != hipSuccess) { status = HEAT1D_EHIP; break; }
    float ms = 0.f;
    hipEventElapsedTime(&ms, a, b);
    if (ms < best) {
      best = ms;
      win = c;
    }
  }
  // Band passes against the best of them, where the plan may take them.  A pass
  // costs nearly the same whatever its steps, stepping a start and so much a step:
  // the line through its times for two step counts says from how many steps on
  // passes are faster, which the probe alone does not (32 steps of 4096 FP64 points
  // are 9 us, 90 are 13, a pass is 15).
  if (status == HEAT1D_OK && p->band_from > 0) {
    // the better of two runs after a warm one, in ms; K < 0: passes of -K steps
    auto timed = [&](int64_t K) {
      double t = 1e300;
      for (int rep = 0; rep < 3 && status == HEAT1D_OK; ++rep) {
        hipEventRecord(a, s);
        status = K > 0 ? run_sync_impl(p, u0, uK, r, 0.0, 0.0, K, workspace, s, win.kernel, win.T,
                                       win.M, win.waves, win.fuse)
                       : run_band(p, p->nrods, u0, uK, r, 0.0, 0.0, -K, workspace,
                                  (char*)workspace + sync_state_bytes(p), nullptr, nullptr,
                                  nullptr, s);
        hipEventRecord(b, s);
        if (status == HEAT1D_OK && hipEventSynchronize(b) != hipSuccess) status = HEAT1D_EHIP;
        float ms = 0.f;
        if (status == HEAT1D_OK) hipEventElapsedTime(&ms, a, b);
        if (rep > 0) t = std::min(t, (double)ms);
      }
      return t;
    };
    const int32_t least = band_from_steps(p->dtype, p->N, p->nrods, ring);
    const double one = timed(least), two = timed(2 * (int64_t)least), pass = timed(-2 * (int64_t)least);
    if (status == HEAT1D_OK) {
      double from = least;
      if (two > one) from = least * std::max(1.0, 1.0 + (pass - one) / (two - one));
      p->band_from = (int32_t)std::min(std::ceil(from), 2147483647.0);
    }
    if (status == HEAT1D_OK && takes_band(p, r, K_probe, K_probe, workspace))
      best = std::min(best, timed(-K_probe));
  }
  hipEventDestroy(a);
  hipEventDestroy(b);
  p->timing = timing;
  if (status != HEAT1D_OK) return status;
  p->sync_kernel = win.kernel;
  if (win.kernel == HEAT1D_SYNC_TILED || win.kernel == HEAT1D_SYNC_PIPELINED) {
    p->T = win.T;
    p->M = win.M;
    p->fuse = win.fuse;
    p->tile_waves = win.kernel == HEAT1D_SYNC_TILED && win.waves > 1 ? win.waves : 1;
  }
  if (win.kernel == HEAT1D_SYNC_RESIDENT) { p->M = win.M; p->waves = win.waves; }
  describe(p);
  if (best_ms) *best_ms = best;
  return HEAT1D_OK;
}

}  // extern "C"

namespace {

// Checks shared by both asynchronous entry points; on success fills the launch
// geometry.  Nothing is enqueued.
int check_async(heat1d_plan_t p, const void* u0, const void* uK, double r, int64_t K, int32_t d,
                int32_t mode, int* P, int* waves, int* M) {
  if (!p || p->batched || !u0 || !uK || !r_ok(r) || K < 0 || d < 0) return HEAT1D_EINVAL;
  if (mode != HEAT1D_ASYNC_EMULATED && mode != HEAT1D_ASYNC_HARDWARE) return HEAT1D_EINVAL;
  if (p->nrods != 1) return HEAT1D_EUNSUPPORTED;
  if (d > p->max_delay) return HEAT1D_EINVAL;
  if (K > INT32_MAX / 2) return HEAT1D_EUNSUPPORTED;
  *P = plan_nsub(p);
  if (*P < 1 || *P > p->N / 2) return HEAT1D_EINVAL;
  // the ring needs two subdomains: with one, nothing is delayed and the run is
  // heat1d_run_sync's periodic iteration
  if (periodic(p) && *P < 2) return HEAT1D_EUNSUPPORTED;
  // the fixed delay schedules are written for the Dirichlet rod
  if (periodic(p) && p->opts.delay_schedule != 0) return HEAT1D_EUNSUPPORTED;
  if (overlaps(u0, uK, (size_t)p->N * esize(p->dtype))) return HEAT1D_EINVAL;
  if (!async_geometry(p, *P, waves, M)) return HEAT1D_EUNSUPPORTED;
  return HEAT1D_OK;
}

// How an asynchronous run goes by strips (stages = 0: it does not).  Emulated
// runs without statistics only, of kBatchBandFrom steps or more.
StripPlan strips_of(heat1d_plan_t p, int P, double r, double c1, double cN, int64_t K, int32_t d,
                    int32_t mode, const int64_t* stats) {
  StripPlan none;
  const AsyncLayout L = async_layout(p, P);
  if (!L.strips || mode != HEAT1D_ASYNC_EMULATED || stats || K < kBatchBandFrom ||
      !std::isfinite(c1) || !std::isfinite(cN))
    return none;
  return strip_plan(p->dtype, p->N, P, r, K, d, L.ping ? K : 1, !fp32_drifts(p->dtype, r, K));
}

int run_strips(heat1d_plan_t p, const StripPlan& sp, const void* u0, void* uK, double r, double c1,
               double cN, int64_t K, int32_t d, uint64_t seed, int P, char* ws,
               const AsyncLayout& L, bool timed, hipStream_t s) {
  BandPass b;
  b.dtype = p->dtype;
  b.N = p->N;
  b.r = p->dtype == HEAT1D_F32 ? (double)(float)r : r;
  b.c1 = c1;
  b.cN = cN;
  b.ring = periodic(p);
  b.scratch = ws + L.w_off;
  b.flag = (int32_t*)(ws + L.flag_off);
  StripStage a;
  a.dtype = p->dtype;
  a.N = p->N;
  a.P = P;
  a.d = d;
  a.sched = p->opts.delay_schedule;
  a.ring = b.ring;
  a.seed = seed;
  a.r = r;
  a.c1 = c1;
  a.cN = cN;
  a.M = sp.M;
  a.cut = sp.cut;
  a.history = ws + L.hist_off;
  a.flag = b.flag;
  for (int64_t i = 0; i < sp.stages; ++i) {
    const int64_t T = std::min<int64_t>(sp.T, K - i * sp.T);
    a.in = i == 0 ? u0 : a.out;
    a.out = (sp.stages - 1 - i) % 2 == 0 ? uK : (void*)(ws + L.ping_off);
    a.k0 = i * sp.T;
    a.T = T;
    hipError_t e = hipSuccess;
    if (sp.cut > 0) {
      // the points away from the edges
      b.in = a.in;
      b.out = a.out;
      if (b.T != T) {
        b.T = T;
        e = launch_band_weights(b, s);
        if (e != hipSuccess) return hip_status(e);
      }
      e = launch_band_pass(b, s);
      if (e != hipSuccess) return hip_status(e);
    }
    EventPair* ev = timed ? timing_begin(p, s) : nullptr;
    e = launch_strips(a, s);
    timing_end(ev, s);
    if (e != hipSuccess) return hip_status(e);
  }
  return HEAT1D_OK;
}

// Enqueue one asynchronous run whose ring, hints and status words sit in `ws`
// (heat1d_async_workspace_bytes(p) bytes, laid out as that call describes).
int run_async_impl(heat1d_plan_t p, const void* u0, void* uK, double r, double c1, double cN,
                   int64_t K, int32_t d, uint64_t seed, int32_t mode, char* ws, int64_t* stats,
                   int P, int waves, int M, bool timed, hipStream_t s) {
  const int Q = 2 * p->max_delay + 2;
  if (async_max_resident_groups(p->dtype, M, waves, Q) < P) return HEAT1D_EOCCUPANCY;
  AsyncLaunch a;
  a.dtype = p->dtype;
  a.M = M;
  a.waves = waves;
  a.in = u0;
  a.out = uK;
  a.N = p->N;
  a.P = P;
  a.K = (int32_t)K;
  a.d = d;
  a.Q = Q;
  a.seed = seed;
  a.mode = mode;
  a.r = r;
  a.c1 = c1;
  a.cN = cN;
  const AsyncLayout L = async_layout(p, P);
  a.ring = ws;
  a.prog = (int32_t*)(ws + L.hint_off);
  a.err = (int32_t*)(ws + L.err_off);
  a.stats = stats;
  a.watchdog = p->watchdog;
  a.remap = (P % 8 == 0 && P >= 16) ? 1 : 0;
  a.jitter = p->opts.jitter;
  a.periodic = periodic(p) ? 1 : 0;
  a.sched = p->opts.delay_schedule;
  char buf[160];
  std::snprintf(buf, sizeof buf, "async N=%lld P=%d waves=%d M=%d d=%d mode=%s%s",
                (long long)p->N, P, waves, M, d, mode == 0 ? "emulated" : "hardware",
                a.periodic ? " ring" : "");
  p->desc = buf;
  const StripPlan sp = strips_of(p, P, r, c1, cN, K, d, mode, stats);
  if (sp.stages > 0) {
    p->desc += " strips=" + std::to_string(sp.stages) + "x" + std::to_string(sp.T) +
               " M=" + std::to_string(sp.M) + " cut=" + std::to_string(sp.cut);
    a.only_if = (int32_t*)(ws + L.flag_off);
  }
  hipError_t e = launch_async_prepare(a, s);
  if (e != hipSuccess) return hip_status(e);
  if (sp.stages > 0) {
    const int rc = run_strips(p, sp, u0, uK, r, c1, cN, K, d, seed, P, ws, L, timed, s);
    if (rc != HEAT1D_OK) return rc;
    // points that are not finite: the whole run again, step by step (the
    // workgroups leave at once where there were none)
    e = launch_async(a, s);
    return e == hipErrorCooperativeLaunchTooLarge ? HEAT1D_EOCCUPANCY : hip_status(e);
  }
  EventPair* ev = timed ? timing_begin(p, s) : nullptr;
  e = launch_async(a, s);
  timing_end(ev, s);
  if (e == hipErrorCooperativeLaunchTooLarge) return HEAT1D_EOCCUPANCY;
  return hip_status(e);
}

}  // namespace

extern "C" {

int heat1d_run_async(heat1d_plan_t p, const void* u0, void* uK, double r, double c1, double cN,
                     int64_t K, int32_t d, uint64_t seed, int32_t mode, void* workspace,
                     int64_t* stats, void* stream) {
  int P = 0, waves = 0, M = 0;
  const int st = check_async(p, u0, uK, r, K, d, mode, &P, &waves, &M);
  if (st != HEAT1D_OK) return st;
  if (!workspace) return HEAT1D_EINVAL;
  const size_t bytes = (size_t)p->N * esize(p->dtype);
  const size_t wsb = heat1d_async_workspace_bytes(p);
  if (overlaps(workspace, wsb, u0, bytes) || overlaps(workspace, wsb, uK, bytes))
    return HEAT1D_EINVAL;
  return run_async_impl(p, u0, uK, r, c1, cN, K, d, seed, mode, (char*)workspace, stats, P, waves,
                        M, true, (hipStream_t)stream);
}

int heat1d_run_async_noalloc(heat1d_plan_t p, const void* u0, void* uK, double r, double c1,
                             double cN, int64_t K, int32_t d, uint64_t seed, int32_t mode,
                             int64_t* stats, int32_t* status, void* stream) {
  int P = 0, waves = 0, M = 0;
  const int st = check_async(p, u0, uK, r, K, d, mode, &P, &waves, &M);
  if (st != HEAT1D_OK) return st;
  if (async_layout(p, P).total > kNoAllocScratchBytes) return HEAT1D_ESCRATCH;
  if (status && (overlaps(status, 4, u0, (size_t)p->N * esize(p->dtype)) ||
                 overlaps(status, 4, uK, (size_t)p->N * esize(p->dtype))))
    return HEAT1D_EINVAL;
  void* ws = nullptr;
  if (async_noalloc_scratch(&ws) != hipSuccess) return HEAT1D_EHIP;
  hipStream_t s = (hipStream_t)stream;
  const int rc = run_async_impl(p, u0, uK, r, c1, cN, K, d, seed, mode, (char*)ws, stats, P,
                                waves, M, false, s);
  if (rc != HEAT1D_OK || !status) return rc;
  const int32_t* err = (const int32_t*)((char*)ws + async_layout(p, P).err_off);
  return hip_status(launch_copy_status(err, status, s));
}

int heat1d_async_status(heat1d_plan_t p, void* workspace, void* stream) {
  if (!p || !workspace) return HEAT1D_EINVAL;
  const int P = plan_nsub(p);
  const char* ws = (const char*)workspace;
  const int32_t* err = (const int32_t*)(ws + async_layout(p, P).err_off);
  int32_t h = 0;
  hipStream_t s = (hipStream_t)stream;
  if (hipMemcpyAsync(&h, err, sizeof h, hipMemcpyDeviceToHost, s) != hipSuccess) return HEAT1D_EHIP;
  if (hipStreamSynchronize(s) != hipSuccess) return HEAT1D_EHIP;
  return h == 0 ? HEAT1D_OK : h;
}

int heat1d_delay_schedule(int32_t P, int64_t K, int32_t d, uint64_t seed, uint8_t* out,
                          void* stream) {
  if (P < 1 || K < 0 || d < 0 || d > 255 || !out) return HEAT1D_EINVAL;
  if (K == 0) return HEAT1D_OK;
  return hip_status(launch_delay_schedule(P, K, d, seed, out, (hipStream_t)stream));
}

}  // extern "C"

namespace {

// heat1d_run_async_ensemble with, when nsnap > 0, the states at the steps
// steps_host[0..nsnap) written to snaps.
int run_ensemble_impl(heat1d_plan_t p, const void* u0, void* uK, double r, double c1, double cN,
                      int64_t K, int32_t d, const uint64_t* seeds, int32_t every, double* norms,
                      const int64_t* steps_host, int32_t nsnap, void* snaps, hipStream_t s) {
  if (!p || p->batched || !u0 || !uK || !seeds || !r_ok(r) || K < 0 || d < 0 || d > 255 ||
      every < 1)
    return HEAT1D_EINVAL;
  if (p->opts.delay_schedule != 0) return HEAT1D_EUNSUPPORTED;  // seeded draws only
  const int64_t E = p->nrods, N = p->N;
  const int64_t P = p->opts.nsub > 0 ? p->opts.nsub : N;
  if (P > N) return HEAT1D_EINVAL;
  if (K > INT32_MAX || N > INT32_MAX || E > INT32_MAX) return HEAT1D_EUNSUPPORTED;
  if (ensemble_lds_bytes(p->dtype, N, P, d) > kEnsembleMaxLds) return HEAT1D_EUNSUPPORTED;
  const size_t bytes = (size_t)N * E * esize(p->dtype);
  const size_t nbytes = (size_t)(K / every + 1) * E * 8;
  if (overlaps(u0, uK, bytes) || overlaps(seeds, (size_t)E * 8, uK, bytes) ||
      (norms && (overlaps(norms, nbytes, u0, bytes) || overlaps(norms, nbytes, uK, bytes) ||
                 overlaps(norms, nbytes, seeds, (size_t)E * 8))))
    return HEAT1D_EINVAL;
  EnsembleLaunch L;
  if (nsnap > 0) {
    if (nsnap > kEnsembleMaxSnaps || !steps_host || !snaps) return HEAT1D_EINVAL;
    for (int32_t j = 0; j < nsnap; ++j) {
      if (steps_host[j] < 0 || steps_host[j] > K) return HEAT1D_EINVAL;
      if (j > 0 && steps_host[j] <= steps_host[j - 1]) return HEAT1D_EINVAL;
      L.snap_steps[j] = (int32_t)steps_host[j];
    }
    const size_t sbytes = (size_t)nsnap * bytes;
    if (overlaps(snaps, sbytes, u0, bytes) || overlaps(snaps, sbytes, uK, bytes) ||
        overlaps(snaps, sbytes, seeds, (size_t)E * 8) ||
        (norms && overlaps(snaps, sbytes, norms, nbytes)))
      return HEAT1D_EINVAL;
    L.snaps = snaps;
    L.nsnap = nsnap;
  }
  L.dtype = p->dtype;
  L.u0 = u0;
  L.uK = uK;
  L.seeds = seeds;
  L.norms = norms;
  L.E = E;
  L.N = (int32_t)N;
  L.P = (int32_t)P;
  L.K = (int32_t)K;
  L.d = d;
  L.every = every;
  L.r = r;
  L.c1 = c1;
  L.cN = cN;
  L.periodic = periodic(p) ? 1 : 0;
  char buf[160];
  std::snprintf(buf, sizeof buf, "ensemble members=%lld N=%lld P=%lld d=%d %s", (long long)E,
                (long long)N, (long long)P, d, L.periodic ? "periodic" : "dirichlet");
  p->desc = buf;
  EventPair* ev = timing_begin(p, s);
  hipError_t e = launch_ensemble(L, s);
  timing_end(ev, s);
  return hip_status(e);
}

}  // namespace

extern "C" {

int heat1d_run_async_ensemble(heat1d_plan_t p, const void* u0, void* uK, double r, double c1,
                              double cN, int64_t K, int32_t d, const uint64_t* seeds,
                              int32_t every, double* norms, void* stream) {
  return run_ensemble_impl(p, u0, uK, r, c1, cN, K, d, seeds, every, norms, nullptr, 0, nullptr,
                           (hipStream_t)stream);
}

int heat1d_run_async_ensemble_snapshots(heat1d_plan_t p, const void* u0, void* uK, double r,
                                        double c1, double cN, int64_t K, int32_t d,
                                        const uint64_t* seeds, int32_t every, double* norms,
                                        const int64_t* steps_host, int32_t nsnap, void* snaps,
                                        void* stream) {
  if (nsnap < 1) return HEAT1D_EINVAL;
  return run_ensemble_impl(p, u0, uK, r, c1, cN, K, d, seeds, every, norms, steps_host, nsnap,
                           snaps, (hipStream_t)stream);
}

size_t heat1d_ensemble_adjoint_workspace_bytes(heat1d_plan_t p, int64_t K) {
  if (!p || p->batched || K < 0) return 0;
  return align_up((size_t)(K + 1) * p->N * p->nrods * esize(p->dtype));
}

int heat1d_run_async_ensemble_adjoint(heat1d_plan_t p, const void* u0, const void* gK, double r,
                                      double c1, double cN, int64_t K, int32_t d,
                                      const uint64_t* seeds, void* uK, void* grad_u0,
                                      double* grad_r, double* grad_c1, double* grad_cN,
                                      void* workspace, void* stream) {
  if (!p || p->batched || !u0 || !gK || !seeds || !grad_u0 || !grad_r || !grad_c1 || !grad_cN ||
      !workspace || !r_ok(r) || K < 0 || d < 0 || d > 255)
    return HEAT1D_EINVAL;
  if (!std::isfinite(c1) || !std::isfinite(cN)) return HEAT1D_EINVAL;
  if (p->opts.delay_schedule != 0) return HEAT1D_EUNSUPPORTED;  // seeded draws only
  const int64_t E = p->nrods, N = p->N;
  const int64_t P = p->opts.nsub > 0 ? p->opts.nsub : N;
  if (P > N) return HEAT1D_EINVAL;
  if (K > INT32_MAX || N > INT32_MAX || E > INT32_MAX) return HEAT1D_EUNSUPPORTED;
  if (ensemble_lds_bytes(p->dtype, N, P, d) > kEnsembleMaxLds ||
      ensemble_adjoint_lds_bytes(p->dtype, N, P, d) > kEnsembleMaxLds ||
      (periodic(p) ? N : N - 2) > 16 * 256)
    return HEAT1D_EUNSUPPORTED;
  const size_t bytes = (size_t)N * E * esize(p->dtype);
  const size_t wsb = heat1d_ensemble_adjoint_workspace_bytes(p, K);
  const size_t sb = (size_t)E * 8;
  struct Buf { const void* p; size_t n; } bufs[] = {
      {u0, bytes}, {gK, bytes}, {uK, uK ? bytes : 0}, {grad_u0, bytes}, {workspace, wsb},
      {seeds, sb}, {grad_r, sb}, {grad_c1, sb}, {grad_cN, sb}};
  const int nb = sizeof(bufs) / sizeof(bufs[0]);
  for (int i = 0; i < nb; ++i)
    for (int j = i + 1; j < nb; ++j) {
      if (bufs[i].n == 0 || bufs[j].n == 0) continue;
      if (i == 0 && j == 1) continue;  // u0 and gK are both read only
      if (overlaps(bufs[i].p, bufs[i].n, bufs[j].p, bufs[j].n)) return HEAT1D_EINVAL;
    }
  hipStream_t s = (hipStream_t)stream;
  EnsembleLaunch F;
  F.dtype = p->dtype;
  F.u0 = u0;
  F.uK = uK;
  F.traj = workspace;
  F.seeds = seeds;
  F.norms = nullptr;
  F.E = E;
  F.N = (int32_t)N;
  F.P = (int32_t)P;
  F.K = (int32_t)K;
  F.d = d;
  F.every = 1;
  F.periodic = periodic(p) ? 1 : 0;
  F.r = r;
  F.c1 = c1;
  F.cN = cN;
  hipError_t e = launch_ensemble(F, s);
  if (e != hipSuccess) return hip_status(e);
  EnsembleAdjointLaunch B;
  B.dtype = p->dtype;
  B.traj = workspace;
  B.gK = gK;
  B.seeds = seeds;
  B.grad_u0 = grad_u0;
  B.grad_r = grad_r;
  B.grad_c1 = grad_c1;
  B.grad_cN = grad_cN;
  B.E = E;
  B.N = (int32_t)N;
  B.P = (int32_t)P;
  B.K = (int32_t)K;
  B.d = d;
  B.periodic = periodic(p) ? 1 : 0;
  B.r = r;
  B.c1 = c1;
  B.cN = cN;
  EventPair* ev = timing_begin(p, s);
  e = launch_ensemble_adjoint(B, s);
  timing_end(ev, s);
  return hip_status(e);
}

size_t heat1d_async_adjoint_workspace_bytes(heat1d_plan_t p, int64_t K) {
  if (!p || p->batched || K < 0) return 0;
  return async_adjoint_layout(p, K, plan_nsub(p)).total;
}

int heat1d_run_async_adjoint(heat1d_plan_t p, const void* u0, const void* gK, double r, double c1,
                             double cN, int64_t K, int32_t d, uint64_t seed, void* uK,
                             void* grad_u0, double* grad_r, double* grad_c1, double* grad_cN,
                             void* workspace, void* stream) {
  if (!p || !u0 || !gK || !grad_u0 || !grad_r || !grad_c1 || !grad_cN || !workspace ||
      !r_ok(r) || K < 0 || d < 0 || d > 255)
    return HEAT1D_EINVAL;
  if (!std::isfinite(c1) || !std::isfinite(cN)) return HEAT1D_EINVAL;
  if (p->batched || p->nrods != 1) return HEAT1D_EUNSUPPORTED;
  const int64_t N = p->N;
  const int P = plan_nsub(p);
  if (P > N) return HEAT1D_EINVAL;
  // the ring needs two subdomains, as heat1d_run_async does
  const bool ring = periodic(p);
  if (ring && (P < 2 || p->opts.delay_schedule != 0)) return HEAT1D_EUNSUPPORTED;
  if (K > INT32_MAX / 2 || N > INT32_MAX) return HEAT1D_EUNSUPPORTED;
  const AsyncAdjLayout L = async_adjoint_layout(p, K, P);
  const size_t bytes = (size_t)N * esize(p->dtype);
  struct Buf { const void* q; size_t n; } bufs[] = {
      {u0, bytes}, {gK, bytes}, {uK, uK ? bytes : 0}, {grad_u0, bytes}, {workspace, L.total},
      {grad_r, 8}, {grad_c1, 8}, {grad_cN, 8}};
  const int nb = sizeof(bufs) / sizeof(bufs[0]);
  for (int i = 0; i < nb; ++i)
    for (int j = i + 1; j < nb; ++j) {
      if (bufs[i].n == 0 || bufs[j].n == 0) continue;
      if (i == 0 && j == 1) continue;  // u0 and gK are both read only
      if (overlaps(bufs[i].q, bufs[i].n, bufs[j].q, bufs[j].n)) return HEAT1D_EINVAL;
    }
  hipStream_t s = (hipStream_t)stream;
  char* ws = (char*)workspace;
  auto ck = [&](int64_t c) { return (void*)(ws + L.ck_off + (size_t)c * L.state_bytes); };
  auto st = [&](int64_t j) { return (void*)(ws + L.st_off + (size_t)j * L.state_bytes); };
  void* fin = uK ? uK : (void*)(ws + L.fin_off);
  void* lam[2] = {ws + L.lam_off, ws + L.lam_off + L.state_bytes};
  const size_t es = esize(p->dtype);
  AsyncAdjStep A;
  A.dtype = p->dtype;
  A.ring = ring ? 1 : 0;
  A.sched = p->opts.delay_schedule;
  A.N = N;
  A.P = P;
  A.K = (int)K;
  A.d = d;
  A.seed = seed;
  A.r = r;
  A.c1 = c1;
  A.cN = cN;
  A.E = ws + L.E_off;
  A.LE = ws + L.LE_off;
  A.lo = (const int64_t*)(ws + L.lo_off);
  A.part = (double*)(ws + L.part_off);
  A.ends = (double*)(ws + L.ends_off);
  A.ord_lock = (const int*)(ws + L.ord_off);
  A.ord_adj = (const int*)(ws + L.ord_off + L.ord_bytes);
  auto rec = [&](void* base, int64_t k) { return (void*)((char*)base + (size_t)k * P * 2 * es); };
  const int S = L.S;
  hipError_t e;
#define HEAT1D_TRY(x) do { e = (x); if (e != hipSuccess) return hip_status(e); } while (0)
  HEAT1D_TRY(launch_async_partition((int64_t*)A.lo, N, P, s));
  HEAT1D_TRY(launch_zero_f64(A.part, L.nparts, s));
  HEAT1D_TRY(launch_zero_f64(A.ends, 2, s));
  // forward: u(0) (ends imposed) is checkpoint 0; inside stretch c the states
  // go to st[0..], the stretch's last step to the next checkpoint (or u(K))
  void* u0s = K > 0 ? ck(0) : fin;
  HEAT1D_TRY(ring ? hipMemcpyAsync(u0s, u0, bytes, hipMemcpyDeviceToDevice, s)
                  : launch_impose_ends(p->dtype, u0, u0s, N, 1, c1, cN, s));
  HEAT1D_TRY(launch_async_edges(p->dtype, u0s, A.E, A.lo, P, N, A.ring, s));
  // Register tiles of up to T steps per launch where every subdomain is
  // long enough and the run has steps for it (ring tiles on a ring;
  // opts.sync_kernel = HEAT1D_SYNC_STEP asks for one launch per step); both give
  // the same values bit for bit.
  const bool tiled = L.tiled;
  const int T = async_tiled_depth();
  if (tiled)
    HEAT1D_TRY(launch_async_tiled_order(A, (int*)A.ord_lock, (int*)A.ord_adj, s));
  // Tiled runs go in segments of T steps, whose transpose needs the state at the
  // segment's start alone.  The places of the checkpoints and of a stretch's
  // states (ck and st are one array) hold those of all segments up to
  // K = T (nck + S - 1), 4096 steps with the default S; beyond that the segments
  // form nst stretches of at most m, the starts of a stretch's later segments
  // replayed from its first.
  const int64_t nseg = (K + T - 1) / T, places = L.nck + S - 1;
  int64_t m = 1;
  while ((nseg + m - 1) / m + m - 1 > places) ++m;
  const int64_t nst = std::max<int64_t>(1, std::min(nseg, places - (m - 1)));
  auto first_seg = [&](int64_t c) { return c * (nseg / nst) + std::min(c, nseg % nst); };
  // the segments [a, b) forward from u(a T) = cur: the state after segment g goes
  // to where(g)
  auto forward = [&](const void* cur, int64_t a, int64_t b, int record, auto where) {
    for (int64_t g = a; g < b; ++g) {
      void* out = where(g);
      const hipError_t f = launch_async_lockstep_tiled(
          A, cur, out, (int)(g * T), (int)std::min<int64_t>(T, K - g * T), record, s);
      if (f != hipSuccess) return f;
      cur = out;
    }
    return hipSuccess;
  };
  for (int64_t c = 0; tiled && c < nst && K > 0; ++c) {
    // earlier stretches pass through the two lambda buffers, unused until the
    // backward sweep; the last one's states stay for it
    const int64_t a = first_seg(c), b = first_seg(c + 1);
    const bool last = c + 1 == nst;
    HEAT1D_TRY(forward(ck(c), a, b, 1, [&](int64_t g) {
      if (g + 1 == b) return last ? fin : ck(c + 1);
      return last ? ck(nst + (g - a)) : lam[g & 1];
    }));
  }
  for (int64_t c = 0; !tiled && c < L.nck && K > 0; ++c) {
    const int64_t k0 = c * S, len = std::min<int64_t>(S, K - k0);
    const void* cur = ck(c);
    for (int64_t j = 1; j <= len; ++j) {
      void* nxt = j < len ? st(j - 1) : (c + 1 < L.nck ? ck(c + 1) : fin);
      HEAT1D_TRY(launch_async_lockstep(A, cur, nxt, (int)(k0 + j - 1), 1, s));
      cur = nxt;
    }
  }
  // backward: lambda(K) = gK, its ends zeroed on the Dirichlet rod; the last
  // stretch's states are still in st, every earlier stretch is replayed from
  // its checkpoint
  void* lK = K > 0 ? lam[K & 1] : grad_u0;
  HEAT1D_TRY(ring ? hipMemcpyAsync(lK, gK, bytes, hipMemcpyDeviceToDevice, s)
                  : launch_impose_ends(p->dtype, gK, lK, N, 1, 0.0, 0.0, s));
  HEAT1D_TRY(launch_async_edges(p->dtype, lK, rec(A.LE, K), A.lo, P, N, A.ring, s));
  const void* lcur = lK;
  for (int64_t c = nst - 1; tiled && c >= 0 && K > 0; --c) {
    const int64_t a = first_seg(c), b = first_seg(c + 1);
    if (c + 1 < nst)
      HEAT1D_TRY(forward(ck(c), a, b - 1, 0, [&](int64_t g) { return ck(nst + (g - a)); }));
    for (int64_t g = b - 1; g >= a; --g) {
      const void* u = g == a ? ck(c) : ck(nst + (g - a) - 1);
      void* lout = g == 0 ? grad_u0 : (lcur == lam[0] ? lam[1] : lam[0]);
      EventPair* ev = timing_begin(p, s);
      e = launch_async_adjoint_tiled(A, lcur, lout, u, (int)(g * T),
                                     (int)std::min<int64_t>(T, K - g * T), s);
      timing_end(ev, s);
      if (e != hipSuccess) return hip_status(e);
      lcur = lout;
    }
  }
  for (int64_t c = L.nck - 1; !tiled && c >= 0 && K > 0; --c) {
    const int64_t k0 = c * S, len = std::min<int64_t>(S, K - k0);
    if (c + 1 < L.nck) {
      const void* cur = ck(c);
      for (int64_t j = 1; j < len; ++j) {
        HEAT1D_TRY(launch_async_lockstep(A, cur, st(j - 1), (int)(k0 + j - 1), 0, s));
        cur = st(j - 1);
      }
    }
    for (int64_t k = k0 + len - 1; k >= k0; --k) {
      const void* uk = k == k0 ? ck(c) : st(k - k0 - 1);
      void* l0 = k == 0 ? grad_u0 : lam[k & 1];
      EventPair* ev = timing_begin(p, s);
      e = launch_async_adjoint_step(A, lam[(k + 1) & 1], l0, uk, (int)k, s);
      timing_end(ev, s);
      if (e != hipSuccess) return hip_status(e);
    }
  }
  HEAT1D_TRY(launch_reduce_partials(A.part, L.nparts, 1, grad_r, s));
  HEAT1D_TRY(launch_async_adjoint_ends(p->dtype, gK, N, A.ends, grad_c1, grad_cN, A.ring, s));
#undef HEAT1D_TRY
  return HEAT1D_OK;
}

int heat1d_batched_prepare(heat1d_plan_t p, void* workspace, void* stream) {
  if (!p || !p->batched || !workspace) return HEAT1D_EINVAL;
  char* ws = (char*)workspace;
  hipStream_t s = (hipStream_t)stream;
  for (int q = 0; q < 3; ++q) {
    if (p->order[q].empty()) continue;
    if (hipMemcpyAsync(ws + batched_queue_off(p, q), p->order[q].data(), p->order[q].size() * 4,
                       hipMemcpyHostToDevice, s) != hipSuccess)
      return HEAT1D_EHIP;
  }
  if (!p->band_items.empty()) {
    const BatchedBandLayout L = batched_band_layout(p);
    if (hipMemcpyAsync(ws + L.items, p->band_items.data(), p->band_items.size() * sizeof(BandItem),
                       hipMemcpyHostToDevice, s) != hipSuccess ||
        hipMemcpyAsync(ws + L.rods, p->band_rods.data(), p->band_rods.size() * 4,
                       hipMemcpyHostToDevice, s) != hipSuccess ||
        hipMemcpyAsync(ws + L.woff, p->band_woff.data(), p->band_woff.size() * 4,
                       hipMemcpyHostToDevice, s) != hipSuccess)
      return HEAT1D_EHIP;
  }
  // the host vectors must stay valid until the copies finish
  if (hipStreamSynchronize(s) != hipSuccess) return HEAT1D_EHIP;
  return HEAT1D_OK;
}

}  // extern "C"

namespace {

int check_batched(heat1d_plan_t p, const void* u0, void* uK, const int64_t* offsets,
                  const double* r, const double* c1, const double* cN, const int32_t* K,
                  void* workspace) {
  if (!p || !p->batched || !u0 || !uK || !offsets || !r || !c1 || !cN || !K || !workspace)
    return HEAT1D_EINVAL;
  int64_t total = 0;
  for (int64_t n : p->Nh) total += n;
  const size_t bytes = (size_t)total * esize(p->dtype);
  const size_t wsb = heat1d_batched_workspace_bytes(p);
  if (overlaps(u0, uK, bytes) || overlaps(workspace, wsb, uK, bytes)) return HEAT1D_EINVAL;
  return HEAT1D_OK;
}

BatchedLaunch batched_args(heat1d_plan_t p, const void* u0, void* uK, const int64_t* offsets,
                           const double* r, const double* c1, const double* cN, const int32_t* K,
                           void* workspace) {
  char* ws = (char*)workspace;
  BatchedLaunch b;
  b.dtype = p->dtype;
  b.in = u0;
  b.out = uK;
  b.offsets = offsets;
  b.r = r;
  b.c1 = c1;
  b.cN = cN;
  b.K = K;
  for (int q = 0; q < 3; ++q) {
    b.order[q] = (const int32_t*)(ws + batched_queue_off(p, q));
    b.count[q] = (int32_t)p->order[q].size();
  }
  b.heads = (int32_t*)(ws + batched_queue_off(p, 3));
  b.groups = p->groups;
  b.small_first = p->small_first;
  return b;
}

// The whole batch: the queues' rods in the persistent kernel, the others as
// band passes.
hipError_t launch_batch(heat1d_plan_t p, const void* u0, void* uK, const int64_t* offsets,
                        const double* r, const double* c1, const double* cN, const int32_t* K,
                        void* workspace, hipStream_t s) {
  char* ws = (char*)workspace;
  hipError_t e = hipSuccess;
  if (!p->band_items.empty()) {
    const BatchedBandLayout L = batched_band_layout(p);
    BandBatch b;
    b.dtype = p->dtype;
    b.in = u0;
    b.out = uK;
    b.offsets = offsets;
    b.r = r;
    b.c1 = c1;
    b.cN = cN;
    b.K = K;
    b.items = (const BandItem*)(ws + L.items);
    b.rods = (const int32_t*)(ws + L.rods);
    b.woff = (const int32_t*)(ws + L.woff);
    b.slot = ws + L.slot;
    b.w = ws + L.w;
    b.flag = (int32_t*)(ws + L.flag);
    b.rec = ws + L.rec;
    b.nitems = (int32_t)p->band_items.size();
    b.nslots = (int32_t)p->band_rods.size();
    b.hmax = p->band_hmax;
    b.short_rods = p->band_short;
    e = launch_band_batch(b, s);
  }
  if (e == hipSuccess && !p->by_work.empty())
    e = launch_batched(batched_args(p, u0, uK, offsets, r, c1, cN, K, workspace), s);
  return e;
}

}  // namespace

extern "C" {

int heat1d_run_batched(heat1d_plan_t p, const void* u0, void* uK, const int64_t* offsets,
                       const double* r, const double* c1, const double* cN, const int32_t* K,
                       void* workspace, void* stream) {
  const int st = check_batched(p, u0, uK, offsets, r, c1, cN, K, workspace);
  if (st != HEAT1D_OK) return st;
  hipStream_t s = (hipStream_t)stream;
  EventPair* e = timing_begin(p, s);
  hipError_t err = launch_batch(p, u0, uK, offsets, r, c1, cN, K, workspace, s);
  timing_end(e, s);
  return hip_status(err);
}

int heat1d_autotune_batched(heat1d_plan_t p, const void* u0, void* uK, const int64_t* offsets,
                            const double* r, const double* c1, const double* cN, const int32_t* K,
                            void* workspace, void* stream, double* best_ms) {
  const int st = check_batched(p, u0, uK, offsets, r, c1, cN, K, workspace);
  if (st != HEAT1D_OK) return st;
  hipStream_t s = (hipStream_t)stream;
  hipEvent_t ev[2] = {nullptr, nullptr};
  if (hipEventCreate(&ev[0]) != hipSuccess || hipEventCreate(&ev[1]) != hipSuccess) {
    if (ev[0]) hipEventDestroy(ev[0]);
    return HEAT1D_EHIP;
  }
  int rc = HEAT1D_OK;
  // time the plan's current split: the better of two runs
  auto time_current = [&](double* ms) -> int {
    if (heat1d_batched_prepare(p, workspace, stream) != HEAT1D_OK) return HEAT1D_EHIP;
    *ms = 1e30;
    for (int rep = 0; rep < 2; ++rep) {
      if (hipEventRecord(ev[0], s) != hipSuccess) return HEAT1D_EHIP;
      if (launch_batch(p, u0, uK, offsets, r, c1, cN, K, workspace, s) != hipSuccess)
        return HEAT1D_EHIP;
      if (hipEventRecord(ev[1], s) != hipSuccess || hipEventSynchronize(ev[1]) != hipSuccess)
        return HEAT1D_EHIP;
      float t = 0.f;
      if (hipEventElapsedTime(&t, ev[0], ev[1]) != hipSuccess) return HEAT1D_EHIP;
      *ms = std::min(*ms, (double)t);
    }
    return HEAT1D_OK;
  };
  const int64_t wcap = batched_wave_capacity(p->dtype), gcap = batched_group_capacity(p->dtype);
  const int64_t was_w = p->t_wave, was_g = p->t_group;
  const int was_sf = p->small_first;
  // 1. the thresholds of the three queues, each with the rule's small_first
  int64_t best_w = p->t_wave, best_g = p->t_group;
  double best = 1e30;
  const int64_t waves_c[] = {0, wcap / 4, wcap / 2, wcap};
  const int64_t groups_c[] = {0, gcap / 4, gcap / 2, gcap};
  for (int64_t tw : waves_c) {
    for (int64_t tg : groups_c) {
      if (tg != 0 && tg <= tw) continue;  // no group queue is the tg = 0 candidate
      batched_assign(p, tw, tg == 0 ? tw : tg);
      if (p->t_wave != tw) continue;      // forced by opts.waves
      p->small_first = batched_rule_small_first(p);
      double ms = 0;
      if ((rc = time_current(&ms)) != HEAT1D_OK) break;
      if (ms < best) {
        best = ms;
        best_w = p->t_wave;
        best_g = p->t_group;
      }
    }
    if (rc != HEAT1D_OK) break;
  }
  // 2. how many workgroups start with the small queues, for the best split
  int best_sf = 0;
  if (rc == HEAT1D_OK) {
    batched_assign(p, best_w, best_g);
    const int rule = batched_rule_small_first(p);
    best_sf = rule;
    const int g = p->groups;
    const int sf_c[] = {rule, 0, g / 8, g / 4, g / 2, g};
    best = 1e30;
    for (int sf : sf_c) {
      p->small_first = sf;
      double ms = 0;
      if ((rc = time_current(&ms)) != HEAT1D_OK) break;
      if (ms < best) {
        best = ms;
        best_sf = sf;
      }
    }
  }
  if (rc == HEAT1D_OK) {
    p->small_first = best_sf;
    p->tuned = true;
  } else {
    batched_assign(p, was_w, was_g);
    p->small_first = was_sf;
  }
  const int up = heat1d_batched_prepare(p, workspace, stream);
  if (rc == HEAT1D_OK) rc = up;
  hipEventDestroy(ev[0]);
  hipEventDestroy(ev[1]);
  describe(p);
  if (best_ms) *best_ms = best;
  return rc;
}

// One pass of `steps` <= T steps of the adjoint's forward and recompute
// passes: fused sweeps on wide tiles where they apply, else the tiled kernel.
static hipError_t adjoint_pass(heat1d_plan_t p, const TileGeom& g, int T, const void* in,
                               void* out, int steps, double r, double c1, double cN,
                               hipStream_t s) {
  const int M = p->dtype == 0 ? 16 : 8, G = 4, S = 4;
  // the persistent pipelined kernel first: on 256 rods of 2^16 FP32 at the
  // depths used here (24, 48) it beats one-shot wide tiles by 15-25%
  const TileGeom gp = tile_geometry(p->dtype, M, T, p->N);
  if (fused_supports(p->dtype, M, S) && gp.tiles_per_rod > 0 &&
      pipelined_applies(p->dtype, gp, in, out, p->N))
    return launch_sync_pipelined(p->dtype, gp, in, out, p->N, p->nrods, steps, r, c1, cN, S, s);
  const TileGeom gw = tile_geometry(p->dtype, M * G, T, p->N);
  if (wide_supports(p->dtype, M, S, G) && gw.tiles_per_rod > 0 && 4 * gw.H <= gw.L &&
      gw.tiles_per_rod * p->nrods <= 0x7fffffffLL)
    return launch_sync_wide(p->dtype, gw, M, G, in, out, p->N, p->nrods, steps, r, c1, cN, S, s);
  return launch_sync_tiled(p->dtype, g, in, out, p->N, p->nrods, steps, r, c1, cN, 1, s);
}

int heat1d_forward_checkpointed(heat1d_plan_t p, const void* u0, void* uK, double r, double c1,
                                double cN, int64_t K, void* workspace, void* stream) {
  if (!p || p->batched || !u0 || !workspace || !r_ok(r) || K < 0) return HEAT1D_EINVAL;
  if (periodic(p)) return HEAT1D_EUNSUPPORTED;
  if (K > INT32_MAX) return HEAT1D_EUNSUPPORTED;
  const bool band = band_adjoint(p, K);
  const AdjLayout L = adjoint_layout(p, K);
  if (!band && L.g.tiles_per_rod <= 0) return HEAT1D_EUNSUPPORTED;
  const size_t bytes = (size_t)p->N * p->nrods * esize(p->dtype);
  const size_t wsb = heat1d_adjoint_workspace_bytes(p, K);
  char* ws = (char*)workspace;
  if (overlaps(ws, wsb, u0, bytes) ||
      (uK && (overlaps(ws, wsb, uK, bytes) || overlaps(u0, uK, bytes))))
    return HEAT1D_EINVAL;
  hipStream_t s = (hipStream_t)stream;
  const int64_t N = p->N, B = p->nrods;
  if (band) {
    const BandAdjLayout Z = band_adjoint_layout(p, K);
    const bool one = band_run(p->dtype, r, K, N, false).passes <= 1;
    return run_band(p, B, u0, uK || one ? uK : ws + Z.spare_off, r, c1, cN, K, ws + Z.ping_off,
                    ws + Z.scr_off, ws + Z.z_off, nullptr, nullptr, s);
  }
  hipError_t e = launch_impose_ends(p->dtype, u0, ws + L.ckpt_off, N, B, c1, cN, s);
  if (e != hipSuccess) return hip_status(e);
  if (K == 0) {
    if (uK) return hip_status(launch_impose_ends(p->dtype, u0, uK, N, B, c1, cN, s));
    return HEAT1D_OK;
  }
  for (int64_t j = 0; j < L.nseg; ++j) {
    const int steps = (int)std::min<int64_t>(L.S, K - j * L.S);
    const void* in = ws + L.ckpt_off + j * L.state_bytes;
    void* out = (j + 1 < L.nseg) ? (void*)(ws + L.ckpt_off + (j + 1) * L.state_bytes)
                                 : (uK ? uK : (void*)(ws + L.lam_off));
    EventPair* ev = timing_begin(p, s);
    e = adjoint_pass(p, L.g, L.S, in, out, steps, r, c1, cN, s);
    timing_end(ev, s);
    if (e != hipSuccess) return hip_status(e);
  }
  return HEAT1D_OK;
}

int heat1d_backward_checkpointed(heat1d_plan_t p, const void* gK, double r, double c1, double cN,
                                 int64_t K, void* grad_u0, double* grad_r, void* workspace,
                                 void* stream) {
  if (!p || p->batched || !gK || !grad_u0 || !grad_r || !workspace || !r_ok(r) || K < 0)
    return HEAT1D_EINVAL;
  if (periodic(p)) return HEAT1D_EUNSUPPORTED;
  if (K > INT32_MAX) return HEAT1D_EUNSUPPORTED;
  const bool band = band_adjoint(p, K);
  const AdjLayout L = adjoint_layout(p, K);
  if (!band &&
      (L.g.tiles_per_rod <= 0 || L.gs.tiles_per_rod <= 0 || L.gsub.tiles_per_rod <= 0))
    return HEAT1D_EUNSUPPORTED;
  const size_t bytes = (size_t)p->N * p->nrods * esize(p->dtype);
  const size_t wsb = heat1d_adjoint_workspace_bytes(p, K);
  char* ws = (char*)workspace;
  const size_t gb = (size_t)(p->opts.grad_sum ? 1 : p->nrods) * 8;
  if (overlaps(gK, grad_u0, bytes) || overlaps(ws, wsb, gK, bytes) ||
      overlaps(ws, wsb, grad_u0, bytes) || overlaps(grad_r, gb, ws, wsb) ||
      overlaps(grad_r, gb, gK, bytes) || overlaps(grad_r, gb, grad_u0, bytes))
    return HEAT1D_EINVAL;
  hipStream_t s = (hipStream_t)stream;
  const int64_t N = p->N, B = p->nrods;
  const int S2 = stretch_steps(p->dtype);
  if (band) {
    const BandAdjLayout Z = band_adjoint_layout(p, K);
    double* part = (double*)(ws + Z.part_off);
    const int st = run_band(p, B, gK, grad_u0, r, 0.0, 0.0, K, ws + Z.ping_off, ws + Z.scr_off,
                            nullptr, ws + Z.z_off, part, s);
    if (st != HEAT1D_OK) return st;
    const int64_t tiles = band_tiles(p->dtype, N, B);
    // one sum over all tiles, or one for each rod
    return hip_status(p->opts.grad_sum ? launch_reduce_partials(part, tiles * B, 1, grad_r, s)
                                       : launch_reduce_partials(part, tiles, B, grad_r, s));
  }
  double* partials = (double*)(ws + L.part_off);
  if (K == 0) {
    hipError_t e = launch_impose_ends(p->dtype, gK, grad_u0, N, B, 0.0, 0.0, s);
    if (e != hipSuccess) return hip_status(e);
    // a sum over no sub-stretches writes 0
    return hip_status(launch_reduce_partials(partials, 0, p->opts.grad_sum ? 1 : B, grad_r, s));
  }
  const void* lam_in = gK;
  int64_t q = 0;  // sub-stretch launches issued so far
  for (int64_t j = L.nseg - 1; j >= 0; --j) {
    const int64_t len1 = std::min<int64_t>(L.S, K - j * L.S);
    const int64_t nsub = (len1 + S2 - 1) / S2;
    const char* ck = ws + L.ckpt_off + j * L.state_bytes;
    // starts of the sub-stretches 1..nsub-1 of this stretch
    for (int64_t i = 1; i < nsub; ++i) {
      const void* in = (i == 1) ? (const void*)ck : (const void*)(ws + L.sub_off + (i - 2) * L.state_bytes);
      void* out = ws + L.sub_off + (i - 1) * L.state_bytes;
      hipError_t e = adjoint_pass(p, L.gsub, S2, in, out, S2, r, c1, cN, s);
      if (e != hipSuccess) return hip_status(e);
    }
    for (int64_t i = nsub - 1; i >= 0; --i) {
      const int len = (int)std::min<int64_t>(S2, len1 - i * S2);
      const void* ustart = (i == 0) ? (const void*)ck : (const void*)(ws + L.sub_off + (i - 1) * L.state_bytes);
      void* lam_out = ((L.nlaunch - 1 - q) % 2 == 0) ? grad_u0 : (void*)(ws + L.lam_off);
      EventPair* ev = timing_begin(p, s);
      StretchArgs sa;
      sa.u_start = ustart;
      sa.lam_in = lam_in;
      sa.lam_out = lam_out;
      sa.N = N;
      sa.nrods = B;
      sa.len = len;
      sa.r = r;
      sa.c1 = c1;
      sa.cN = cN;
      sa.partials = partials;
      sa.part_stride = L.nlaunch * L.gs.tiles_per_rod;
      sa.part_off = q * L.gs.tiles_per_rod;
      hipError_t e = launch_adjoint_stretch(p->dtype, L.gs, sa, s);
      timing_end(ev, s);
      if (e != hipSuccess) return hip_status(e);
      lam_in = lam_out;
      ++q;
    }
  }
  double* per_rod = p->opts.grad_sum ? (double*)(ws + L.rod_off) : grad_r;
  hipError_t e = launch_reduce_partials(partials, L.nlaunch * L.gs.tiles_per_rod, B, per_rod, s);
  if (e == hipSuccess && p->opts.grad_sum) e = launch_reduce_partials(per_rod, B, 1, grad_r, s);
  return hip_status(e);
}

namespace {
// Layout of the end-gradient workspace: w, the zero start, the ping-pong
// state of its run, then the dot-product partials.
struct EndsLayout {
  size_t w_off, z_off, ping_off, part_off, rod_off, scr_off, total;
};
EndsLayout ends_layout(heat1d_plan_t p) {
  EndsLayout L{};
  const size_t st = align_up((size_t)p->N * esize(p->dtype));
  L.w_off = 0;
  L.z_off = st;
  L.ping_off = 2 * st;
  L.part_off = 3 * st;
  L.rod_off = L.part_off + align_up((size_t)2 * norm_partials(p->N, p->nrods) * 8);
  // per-rod dL/dc1 and dL/dcN when the plan reports their sums (opts.grad_sum)
  L.scr_off = L.rod_off + 2 * align_up((size_t)p->nrods * 8);
  L.total = L.scr_off + band_scratch_bytes(p->N, 1);
  return L;
}
}  // namespace

size_t heat1d_adjoint_ends_workspace_bytes(heat1d_plan_t p) {
  if (!p || p->batched) return 0;
  return ends_layout(p).total;
}

int heat1d_adjoint_ends(heat1d_plan_t p, const void* gK, double r, int64_t K, double* grad_c1,
                        double* grad_cN, void* workspace, void* stream) {
  if (!p || p->batched || !gK || !grad_c1 || !grad_cN || !workspace || !r_ok(r) || K < 0)
    return HEAT1D_EINVAL;
  if (periodic(p)) return HEAT1D_EUNSUPPORTED;
  if (K > INT32_MAX || p->nrods > 65535) return HEAT1D_EUNSUPPORTED;
  const EndsLayout L = ends_layout(p);
  const size_t bytes = (size_t)p->N * p->nrods * esize(p->dtype);
  const size_t sb = (size_t)(p->opts.grad_sum ? 1 : p->nrods) * 8;
  if (overlaps(workspace, L.total, gK, bytes) || overlaps(workspace, L.total, grad_c1, sb) ||
      overlaps(workspace, L.total, grad_cN, sb) || overlaps(grad_c1, sb, grad_cN, sb) ||
      overlaps(gK, bytes, grad_c1, sb) || overlaps(gK, bytes, grad_cN, sb))
    return HEAT1D_EINVAL;
  hipStream_t s = (hipStream_t)stream;
  char* ws = (char*)workspace;
  // w = u(K) of one rod from a zero interior with c1 = 1, cN = 0: by linearity
  // of Eq.3 in (u0, c1, cN) it is du(K)/dc1, and its mirror image is du(K)/dcN
  hipError_t e = launch_zero(ws + L.z_off, L.ping_off - L.z_off, s);
  if (e != hipSuccess) return hip_status(e);
  heat1d_plan_s one = *p;
  one.nrods = 1;
  one.timing = false;
  // one rod fills few CUs, so the run is bound by launches and per-step
  // latency: 64-step passes over short (8 points per lane) tiles measured
  // fastest for a 2^16-point rod; smaller tiles for short rods, else steps
  int kern = HEAT1D_SYNC_STEP, T = 1, M = 4;
  if (tile_geometry(p->dtype, 8, 64, p->N).tiles_per_rod > 0) {
    kern = HEAT1D_SYNC_TILED, T = 64, M = 8;
  } else if (tile_geometry(p->dtype, 4, 32, p->N).tiles_per_rod > 0) {
    kern = HEAT1D_SYNC_TILED, T = 32, M = 4;
  }
  // By passes beyond two launches of 64 steps: 100 FP64 points, K = 64 / 128 / 200,
  // 29 / 33 / 42 us stepped, 36 by passes; from 2^21 points on it is the state's
  // traffic that counts: 2^22 points, K = 64 / 96, 67 / 89 us stepped, 71 / 77 by passes.
  const int64_t from = p->N >= (int64_t(1) << 21) ? 80 : 129;
  const int st =
      band_adjoint(&one, K) && band_run(p->dtype, r, K, p->N, false).T >= from
          ? run_band(&one, 1, ws + L.z_off, ws + L.w_off, r, 1.0, 0.0, K, ws + L.ping_off,
                     ws + L.scr_off, nullptr, nullptr, nullptr, s)
          : run_sync_impl(&one, ws + L.z_off, ws + L.w_off, r, 1.0, 0.0, K, ws + L.ping_off, s,
                          kern, T, M, 1, 1);
  if (st != HEAT1D_OK) return st;
  double* g1 = grad_c1;
  double* gN = grad_cN;
  if (p->opts.grad_sum) {
    g1 = (double*)(ws + L.rod_off);
    gN = (double*)(ws + L.rod_off + align_up((size_t)p->nrods * 8));
  }
  EventPair* ev = timing_begin(p, s);
  e = launch_mirror_dots(p->dtype, gK, ws + L.w_off, p->N, p->nrods, (double*)(ws + L.part_off),
                         g1, gN, s);
  timing_end(ev, s);
  if (e == hipSuccess && p->opts.grad_sum) {
    e = launch_reduce_partials(g1, p->nrods, 1, grad_c1, s);
    if (e == hipSuccess) e = launch_reduce_partials(gN, p->nrods, 1, grad_cN, s);
  }
  return hip_status(e);
}

int heat1d_adjoint(heat1d_plan_t p, const void* u0, const void* gK, double r, double c1, double cN,
                   int64_t K, void* grad_u0, double* grad_r, void* uK, void* workspace,
                   void* stream) {
  int st = heat1d_forward_checkpointed(p, u0, uK, r, c1, cN, K, workspace, stream);
  if (st != HEAT1D_OK) return st;
  return heat1d_backward_checkpointed(p, gK, r, c1, cN, K, grad_u0, grad_r, workspace, stream);
}

}  // extern "C"
