"""GPU parity of the band passes (many steps of Eq.3 applied at once on the
matrix cores) against the FP64 oracle: sizes around the tiles and the reach,
rods shorter than the reach (several images of the ends), rings shorter than
it, stacked rods whose starts are not 16-byte aligned, several passes; and
the cones of points that are not finite against one launch per step."""
import numpy as np
import pytest
import torch

import oracle
import workloads
from paper_1510_08982_amd import abi
from paper_1510_08982_amd.heat import AdjointPlan, AsyncPlan, BatchedPlan, SyncPlan
from _helpers import normwise, tol_for, torch_dtype, np_dtype, print_case

pytestmark = pytest.mark.gpu
DEV = "cuda"
RING = abi.HEAT1D_BC_PERIODIC


def dev(x, dt):
    return torch.from_numpy(np.ascontiguousarray(x, dtype=np_dtype(dt))).to(DEV)


def reference(u0, r, c1, cN, K, ring):
    if not ring:
        return oracle.sync(u0, r, c1, cN, K)
    return oracle.async_ensemble(u0, r, 0.0, 0.0, K, 1, 0, [1], every=K, periodic=True)[0][0]


CASES = [  # (N, nrods, K, r)
    (3, 1, 64, 0.5), (4, 3, 1000, 0.05), (100, 2, 1000, 0.5), (100, 1, 65, 0.37),
    (255, 1, 300, 0.25), (256, 1, 301, 0.5), (257, 3, 64, 0.45), (1000, 1, 30000, 0.5),
    (2047, 1, 512, 0.3), (2049, 2, 513, 0.3), (4096, 1, 20000, 0.4), (5003, 3, 777, 0.499),
    (5001, 600, 100, 0.5),           # 2048 outputs a block, odd rod starts
    (8192 * 3 + 5, 200, 64, 0.41),   # the largest blocks
    (100, 1, 400000, 0.5),           # several passes, every image of the ends
    (20000, 1, 90000, 0.5),          # several passes
]


def steps(dt, K, r):
    """FP32 runs of this length keep stepping."""
    return dt == "f32" and K * (1 + 0.1 / r) > 6200


@pytest.mark.parametrize("ring", [False, True])
@pytest.mark.parametrize("N,B,K,r,dt", [(*c, dt) for c in CASES for dt in ("f32", "f64")
                                        if not steps(dt, c[2], c[3])])
def test_band_passes_match_oracle(N, B, K, r, dt, ring):
    f = np_dtype(dt)
    rng = np.random.default_rng(N + K)
    u0 = workloads.as_dtype(rng.uniform(-1, 1, (B, N)), f)
    r, c1, cN = (workloads.as_dtype(x, f) for x in (r, 0.75, -0.5))
    plan = SyncPlan(N, torch_dtype(dt), nrods=B, boundary=RING if ring else 0)
    print_case(test="band", dt=dt, N=N, B=B, K=K, r=r, ring=ring, plan=plan.describe())
    assert "band_from=" in plan.describe()
    got = plan.run(dev(u0.reshape(-1), dt), r, c1, cN, K).cpu().numpy().reshape(B, N)
    for b in sorted({0, B // 2, B - 1}):
        ref = reference(u0[b], r, c1, cN, K, ring)
        err = normwise(got[b], ref)
        print(f"  rod {b}: normwise error {err:.3e}")
        assert err <= tol_for(dt)
        if not ring:
            assert got[b][0] == f(c1) and got[b][-1] == f(cN)


@pytest.mark.parametrize("ring", [False, True])
@pytest.mark.parametrize("dt", ["f32", "f64"])
@pytest.mark.parametrize("N,B,K,bad", [
    (5000, 1, 100, {2500: np.nan}), (5000, 1, 100, {50: np.inf, 3000: -np.inf}),
    (700, 3, 64, {1: np.inf, 600: np.nan, 699: np.nan}),   # an end's own value does not count
    (3000, 2, 128, {1000: np.inf, 1256: -np.inf, 2000: np.inf}),  # cones that just meet
    (300, 1, 200, {10: np.nan}), (40, 1, 64, {20: np.inf}), (9000, 1, 64, {8900: -np.inf}),
])
def test_points_that_are_not_finite_spread_as_steps_spread_them(N, B, K, bad, dt, ring):
    """Stepping carries a NaN or an infinity one point a step: outside that cone
    the run is the one with any finite value in its place."""
    f = np_dtype(dt)
    rng = np.random.default_rng(N + K)
    u0 = rng.uniform(-1, 1, (B, N)).astype(f)
    for i, v in bad.items():
        u0[B - 1, i] = v
    bc = RING if ring else 0
    print_case(test="cones", dt=dt, N=N, B=B, K=K, bad=bad, ring=ring)
    x = dev(u0.reshape(-1), dt)
    got = SyncPlan(N, torch_dtype(dt), nrods=B, boundary=bc).run(x, 0.4, 0.25, -0.5, K)
    ref = SyncPlan(N, torch_dtype(dt), nrods=B, boundary=bc,
                   sync_kernel=abi.HEAT1D_SYNC_STEP).run(x, 0.4, 0.25, -0.5, K)
    got, ref = got.cpu().numpy(), ref.cpu().numpy()
    assert np.array_equal(np.isnan(got), np.isnan(ref))
    assert np.array_equal(got[np.isinf(ref)], ref[np.isinf(ref)])
    fin = np.isfinite(ref)
    assert np.array_equal(np.isfinite(got), fin)
    if fin.any():
        assert normwise(got[fin], ref[fin]) <= tol_for(dt)


def test_band_passes_replay_in_a_graph():
    N, K = 30001, 500
    plan = SyncPlan(N, torch.float32)
    xs = [torch.randn(N, generator=torch.Generator().manual_seed(i)).to(DEV) for i in range(3)]
    want = [plan.run(x, 0.4, 0.25, -0.5, K).clone() for x in xs]
    x, out = xs[0].clone(), torch.empty(N, device=DEV)
    s = torch.cuda.Stream()
    s.wait_stream(torch.cuda.current_stream())
    g = torch.cuda.CUDAGraph()
    with torch.cuda.stream(s):
        plan.run(x, 0.4, 0.25, -0.5, K, out=out)
        torch.cuda.synchronize()
        with torch.cuda.graph(g, stream=s):
            plan.run(x, 0.4, 0.25, -0.5, K, out=out)
    torch.cuda.current_stream().wait_stream(s)
    for i in (1, 2, 0, 1):
        x.copy_(xs[i])
        g.replay()
        torch.cuda.synchronize()
        assert torch.equal(out, want[i])
        _ = SyncPlan(N, torch.float32).run(xs[2], 0.3, 0.0, 0.0, 64)   # eager work in between
        torch.cuda.synchronize()


@pytest.mark.parametrize("dt", ["f32", "f64"])
def test_batched_band_rods_match_oracle(dt):
    """Rods on both sides of the step count where band passes begin, lengths
    around the tiles, one rod with a NaN."""
    f = np_dtype(dt)
    n = np.array([3, 4, 17, 255, 256, 257, 600, 2047, 2048, 2049, 4100, 9001, 20000, 5000, 1000])
    K = np.array([448, 5000, 447, 449, 900, 5100 if dt == "f32" else 20000, 1, 600, 2000, 447,
                  3000, 500, 700, 460, 448])
    rng = np.random.default_rng(7)
    r = workloads.as_dtype(np.append(rng.uniform(0.05, 0.5, n.size - 2), [0.5, 0.05]), f)
    c1, cN = (workloads.as_dtype(rng.uniform(-1, 1, n.size), f) for _ in range(2))
    off = np.concatenate([[0], np.cumsum(n)]).astype(np.int64)
    u0 = workloads.as_dtype(rng.uniform(-1, 1, int(off[-1])), f)
    print_case(test="batched_band", dt=dt)
    with BatchedPlan(n, K, torch_dtype(dt)) as plan:
        assert "band_rods=12" in plan.describe()
        args = [dev(off, "f64").to(torch.int64)] + [
            torch.from_numpy(np.ascontiguousarray(x)).to(DEV) for x in (r, c1, cN)] + [
            torch.from_numpy(K.astype(np.int32)).to(DEV)]
        got = plan.run(dev(u0, dt), *args).cpu().numpy()
        x = u0.astype(f)
        x[off[11] + 4000] = np.nan
        bad = plan.run(dev(x, dt), *args).cpu().numpy()
    for b in range(n.size):
        sl = slice(off[b], off[b + 1])
        ref = oracle.sync(u0[sl], r[b], c1[b], cN[b], int(K[b]))
        err = normwise(got[sl], ref)
        print(f"  rod {b}: N={n[b]} K={K[b]} normwise error {err:.3e}")
        assert err <= tol_for(dt)
        if b != 11:
            assert np.array_equal(bad[sl], got[sl])
    i = np.arange(n[11])
    assert np.array_equal(np.isnan(bad[off[11]:off[12]]), np.abs(i - 4000) <= K[11])


@pytest.mark.parametrize("N,B,K,r", [(3, 2, 1, 0.5), (100, 3, 400, 0.5), (257, 1, 2, 0.3),
                                     (5001, 2, 700, 0.45), (2048, 300, 65, 0.25),
                                     (300, 1, 150000, 0.5)])
def test_band_adjoint_matches_oracle(N, B, K, r):
    """dL/du0 and dL/dr by band passes (FP64): one step, rods shorter than the
    reach, several rods, several passes; u(K) asked for and not."""
    dt, f = "f64", np.float64
    rng = np.random.default_rng(N + K)
    # a loss whose sum for dL/dr does not cancel: gK against the state's own curvature
    u0, gK = (workloads.as_dtype(rng.uniform(0, 1, (B, N)), f) for _ in range(2))
    r, c1, cN = (workloads.as_dtype(x, f) for x in (r, 0.75, -0.5))
    print_case(test="band_adjoint", dt=dt, N=N, B=B, K=K, r=r)
    plan = AdjointPlan(N, K, torch_dtype(dt), nrods=B)
    x, g = dev(u0.reshape(-1), dt), dev(gK.reshape(-1), dt)
    gu, gr, uK = plan.adjoint(x, g, r, c1, cN, want_uK=True)
    gu2, gr2, _ = plan.adjoint(x, g, r, c1, cN)
    assert torch.equal(gu, gu2) and torch.equal(gr, gr2)
    gu, gr, uK = (t.cpu().numpy() for t in (gu, gr, uK))
    for b in sorted({0, B - 1}):
        sl = slice(b * N, (b + 1) * N)
        rgu, rgr = oracle.adjoint(u0[b], gK[b], r, c1, cN, K)
        line = oracle.sync(u0[b], r, c1, cN, K)
        assert normwise(uK[sl], line) <= tol_for(dt)
        assert normwise(gu[sl], rgu) <= tol_for(dt)
        # the sum's terms are K gK . D A^(K-1) u0: the tolerance on its magnitude
        scale = max(abs(rgr), K * float(np.abs(gK[b]).max()) * float(
            np.abs(np.diff(oracle.sync(u0[b], r, c1, cN, K - 1), 2)).sum()))
        print(f"  rod {b}: dL/dr {gr[b]:.6e}, off {abs(gr[b] - rgr) / scale:.3e}")
        assert abs(gr[b] - rgr) <= tol_for(dt) * scale
        assert gu[sl][0] == 0 and gu[sl][-1] == 0


STRIP_CASES = [  # (dt, N, P, d, K, r): one stage and several, with band passes and without
    ("f64", 4096, 16, 3, 2000, 0.4), ("f32", 4096, 16, 3, 2000, 0.4),
    ("f32", 1 << 18, 16, 16, 5000, 0.45), ("f64", 70001, 13, 4, 900, 0.5),
    ("f32", 70001, 2, 63, 448, 0.3), ("f64", 30011, 9, 1, 3000, 0.45),
    ("f32", 100003, 300, 5, 448, 0.05), ("f64", 20000, 4, 7, 6000, 0.5),
]


@pytest.mark.parametrize("ring", [False, True])
@pytest.mark.parametrize("dt,N,P,d,K,r", STRIP_CASES)
def test_strips_match_oracle(dt, N, P, d, K, r, ring):
    """The emulated asynchronous run as strips about the subdomain edges, every
    point against the oracle; the allocation-free entry point bit for bit."""
    f = np_dtype(dt)
    u0 = workloads.as_dtype(np.random.default_rng(N + K).uniform(-1, 1, N), f)
    r, c1, cN = (workloads.as_dtype(x, f) for x in (r, 1.0, -1.0))
    x = dev(u0, dt)
    with AsyncPlan(N, P, torch_dtype(dt), max_delay=d, periodic=ring) as plan:
        out = plan.run(x, r, c1, cN, K, d, 42)
        print_case(test="strips", dt=dt, N=N, P=P, d=d, K=K, ring=ring, plan=plan.describe())
        assert "strips=" in plan.describe()
        assert plan.status() == abi.HEAT1D_OK
        same = torch.empty_like(out)
        abi.heat1d_run_async_noalloc(plan.handle, x.data_ptr(), same.data_ptr(), r, c1, cN, K, d,
                                     42, abi.HEAT1D_ASYNC_EMULATED, None, None,
                                     torch.cuda.current_stream().cuda_stream)
        assert torch.equal(out, same)
    got = out.cpu().numpy()
    if ring:
        ref = oracle.async_ensemble(u0, r, 0.0, 0.0, K, P, d, [42], every=K, periodic=True)[0][0]
    else:
        ref = oracle.async_emulated(u0, r, c1, cN, K, P, d, 42)
        assert got[0] == f(c1) and got[-1] == f(cN)
    err = normwise(got, ref)
    print(f"  normwise error {err:.3e}")
    assert err <= tol_for(dt)


@pytest.mark.parametrize("dt", ["f32", "f64"])
@pytest.mark.parametrize("sched", [1, 2])
def test_strips_under_fixed_schedules_match_oracle(sched, dt):
    N, P, d, K = 50000, 20, 9, 1500
    f = np_dtype(dt)
    u0 = workloads.as_dtype(np.random.default_rng(3).uniform(-1, 1, N), f)
    r = workloads.as_dtype(0.45, f)
    with AsyncPlan(N, P, torch_dtype(dt), max_delay=d, delay_schedule=sched) as plan:
        got = plan.run(dev(u0, dt), r, 1.0, -1.0, K, d, 42).cpu().numpy()
        print_case(test="strips_sched", dt=dt, sched=sched, plan=plan.describe())
        assert "strips=" in plan.describe()
    ref = oracle.async_emulated(u0, r, 1.0, -1.0, K, P, d, 42, schedule=sched)
    assert normwise(got, ref) <= tol_for(dt)


def test_strips_leave_points_that_are_not_finite_to_the_stepping_run():
    N, P, d, K = 50000, 20, 4, 700
    u0 = np.random.default_rng(3).uniform(-1, 1, N)
    for i in (26000, 30000):   # near an edge (2500-point subdomains) and on one
        u0[i] = np.inf
    x = dev(u0, "f32")
    with AsyncPlan(N, P, torch.float32, max_delay=d) as plan:
        got = plan.run(x, 0.4, 1.0, -1.0, K, d, 42)
        assert "strips=" in plan.describe()
        st = torch.zeros(d + 3, dtype=torch.int64, device=DEV)
        ref = plan.run(x, 0.4, 1.0, -1.0, K, d, 42, stats=st)   # statistics: stepped
        assert "strips=" not in plan.describe()
    assert torch.equal(got.view(torch.int32), ref.view(torch.int32))
