"""GPU parity of the ensemble kernels of short rods (one wavefront steps, up to
four points a lane, up to seven steps of delay) against the oracle: rods at and
beside every multiple of 64 updated points, the last of them past the range, on
both boundaries; delays up to the largest and the first that is past it; runs
that end in the middle of a chunk of eight steps, norms and snapshots between.
Tolerances as in test_gpu_ensemble.py, whose runners these cases use."""
import numpy as np
import pytest
import torch

import oracle
import workloads
from paper_1510_08982_amd.heat import EnsemblePlan
from _helpers import normwise, np_dtype, print_case, tol_for, torch_dtype
from test_gpu_ensemble import check, check_adjoint, run_adjoint_case, run_case, seeds_tensor

pytestmark = pytest.mark.gpu
DEV = "cuda"

CASES = [  # N, P, d, K, every, dtype, ring
    (4, 4, 7, 9, 1, "f64", False), (65, 65, 1, 40, 3, "f32", False), (66, 5, 7, 33, 2, "f64", False),
    (67, 67, 7, 64, 1, "f64", False), (130, 130, 3, 41, 8, "f32", False),
    (131, 2, 5, 47, 1, "f64", False), (195, 64, 7, 39, 5, "f32", False),
    (258, 258, 7, 63, 1, "f64", False), (258, 100, 2, 50, 7, "f32", False),
    (259, 259, 4, 30, 1, "f64", False), (100, 100, 8, 40, 1, "f64", False),
    (4, 2, 7, 9, 1, "f32", True), (63, 63, 7, 40, 1, "f64", True), (64, 64, 2, 33, 3, "f32", True),
    (127, 5, 6, 47, 1, "f64", True), (128, 128, 7, 63, 9, "f64", True),
    (191, 190, 1, 39, 1, "f32", True), (255, 255, 7, 64, 1, "f64", True),
    (256, 32, 3, 41, 1, "f32", True),
]


@pytest.mark.parametrize("N,P,d,K,every,dt,ring", CASES)
def test_short_rods_match_oracle(N, P, d, K, every, dt, ring):
    rng = np.random.default_rng(N * 3 + d + K)
    E = 3
    u0, gK = rng.uniform(-1, 1, (E, N)), rng.uniform(-1, 1, (E, N))
    seeds = rng.integers(0, 2**63 - 1, size=E, dtype=np.int64).astype(np.uint64)
    print_case(test="short_rods", N=N, P=P, d=d, K=K, every=every, dt=dt, ring=ring)
    r, c1, cN = 0.45, (0.0 if ring else 0.75), (0.0 if ring else -0.5)
    f = np_dtype(dt)
    got, gn, ref, rn = run_case(dt, u0, r, c1, cN, K, P, d, seeds, every, periodic=ring)
    check(dt, N, got, gn, ref, rn)
    x = torch.from_numpy(np.ascontiguousarray(u0, dtype=f)).to(DEV)
    steps = sorted({0, 1, K // 2, K - 1})
    with EnsemblePlan(N, E, P, torch_dtype(dt), periodic=ring) as plan:
        uK, _, snaps = plan.run(x, r, c1, cN, K, d, seeds_tensor(seeds), every, snap_steps=steps)
    fu, fr, f1, fN = (workloads.as_dtype(v, f) for v in (u0, r, c1, cN))
    assert np.array_equal(uK.cpu().numpy().astype(np.float64), got)
    for j, k in enumerate(steps):
        want, _ = oracle.async_ensemble(fu, fr, f1, fN, k, P, d, seeds, 1, periodic=ring)
        for e in range(E):
            assert normwise(snaps[e, j].cpu().numpy().astype(np.float64), want[e]) <= tol_for(dt)
    if not ring:
        back = run_adjoint_case(dt, u0, gK, r, c1, cN, K, P, d, seeds)
        check_adjoint(dt, back, back[5])
        return
    with EnsemblePlan(N, E, P, torch_dtype(dt), periodic=True) as plan:
        g = torch.from_numpy(np.ascontiguousarray(gK, dtype=f)).to(DEV)
        gu, gr, g1, gN, _ = plan.adjoint(x, g, r, 0.0, 0.0, K, d, seeds_tensor(seeds))
    for e in range(E):
        rgu, rgr, sc = oracle.async_adjoint_periodic(fu[e], workloads.as_dtype(gK[e], f), fr, K, P,
                                                     d, int(seeds[e]), with_scale=True)
        assert normwise(gu[e].cpu().numpy().astype(np.float64), rgu) <= tol_for(dt)
        assert abs(float(gr[e]) - rgr) <= tol_for(dt) * sc
        assert float(g1[e]) == 0 and float(gN[e]) == 0


@pytest.mark.parametrize("dt", ["f64", "f32"])
def test_short_rods_are_the_longer_ones_bit_for_bit(dt):
    """A rod in the short kernels' range and a longer one past it, alike but for
    their right ends: the points that no end can have reached after K steps."""
    N, K = 200, 40
    rng = np.random.default_rng(1)
    u0 = np.zeros((1, 400))
    u0[0, :N] = rng.uniform(-1, 1, N)
    f = torch_dtype(dt)
    x = torch.from_numpy(u0).to(DEV, f)
    out = []
    for n in (N, 400):
        with EnsemblePlan(n, 1, 1, f) as plan:
            uK, _ = plan.run(x[:, :n].contiguous(), 0.4, 0.25, 0.0, K, 0, seeds_tensor([1]), 1)
        out.append(uK.cpu())
    assert torch.equal(out[0][0, :N - K - 1], out[1][0, :N - K - 1])
