"""Band passes of states near the end of their type's range: an image of a point
about an end (2 c1 - u), or a point less the line between the ends, can be out of
range where the state and every step of it are not.  Against the oracle of the
run scaled into range: Eq.3 is linear, and a power of two changes no rounding."""
import numpy as np
import pytest
import torch

import oracle
import workloads
from paper_1510_08982_amd import abi
from paper_1510_08982_amd.heat import AdjointPlan, AsyncPlan, BatchedPlan, SyncPlan
from _helpers import normwise, np_dtype, print_case, tol_for, torch_dtype

pytestmark = pytest.mark.gpu
DEV = "cuda"
BIG = {"f32": 2.0 ** 127, "f64": 2.0 ** 1023}


def rod(dt, N, seed):
    """u0 in (-1, 0), r and ends, and u0 as the type's largest power of two times it
    (2 c1 - u0 reaches 1.99 times that, just out of range)."""
    f = np_dtype(dt)
    u0 = workloads.as_dtype(np.random.default_rng(seed).uniform(-0.95, 0, N), f)
    r, c1, cN = (workloads.as_dtype(x, f) for x in (0.4, 0.52, 0.55))
    return u0, r, c1, cN, torch.from_numpy((u0 * BIG[dt]).astype(f)).to(DEV)


def scaled(t, dt):
    return t.cpu().numpy().astype(np.float64) / BIG[dt]


@pytest.mark.parametrize("dt", ["f32", "f64"])
@pytest.mark.parametrize("N,B,K", [(100, 1, 1000), (100, 3, 100), (5000, 1, 100), (5000, 2, 1000),
                                   (300, 1, 500), (40000, 20, 200), (100, 1, 60000)])
def test_images_out_of_range(N, B, K, dt):
    if dt == "f32" and K == 60000:
        pytest.skip("FP32 runs of this length keep stepping")
    u0, r, c1, cN, x = rod(dt, N * B, N + K)
    print_case(test="extremes", dt=dt, N=N, B=B, K=K)
    got = scaled(SyncPlan(N, torch_dtype(dt), nrods=B).run(x, r, c1 * BIG[dt], cN * BIG[dt], K), dt)
    for b in {0, B - 1}:
        sl = slice(b * N, (b + 1) * N)
        assert normwise(got[sl], oracle.sync(u0[sl], r, c1, cN, K)) <= tol_for(dt)


@pytest.mark.parametrize("dt", ["f32", "f64"])
def test_images_out_of_range_beside_a_point_that_is_not_finite(dt):
    N, K = 5000, 200
    u0, r, c1, cN, x = rod(dt, N, 1)
    x[300] = float("nan")
    got = SyncPlan(N, torch_dtype(dt)).run(x, r, c1 * BIG[dt], cN * BIG[dt], K)
    want = oracle.sync(u0, r, c1, cN, K)
    i = np.arange(N)
    cone = (np.abs(i - 300) <= K) & (i > 0)
    assert np.array_equal(np.isnan(got.cpu().numpy()), cone)
    assert normwise(scaled(got, dt)[~cone], want[~cone]) <= tol_for(dt)


@pytest.mark.parametrize("dt", ["f32", "f64"])
def test_images_out_of_range_in_a_batch_and_between_strips(dt):
    n, K = np.array([60, 700, 5000]), np.array([500, 600, 700])
    u0, r, c1, cN, x = rod(dt, int(n.sum()), 2)
    off = np.concatenate([[0], np.cumsum(n)]).astype(np.int64)
    with BatchedPlan(n, K, torch_dtype(dt)) as plan:
        assert "band_rods=3" in plan.describe()
        par = [torch.full((3,), v, dtype=torch.float64, device=DEV)
               for v in (r, c1 * BIG[dt], cN * BIG[dt])]
        got = scaled(plan.run(x, torch.from_numpy(off).to(DEV), *par,
                              torch.from_numpy(K.astype(np.int32)).to(DEV)), dt)
    for b in range(3):
        sl = slice(off[b], off[b + 1])
        assert normwise(got[sl], oracle.sync(u0[sl], r, c1, cN, int(K[b]))) <= tol_for(dt)
    N, P, d, K = 50000, 20, 4, 700
    u0, r, c1, cN, x = rod(dt, N, 3)
    with AsyncPlan(N, P, torch_dtype(dt), max_delay=d) as plan:
        got = scaled(plan.run(x, r, c1 * BIG[dt], cN * BIG[dt], K, d, 42), dt)
        assert "strips=" in plan.describe()
    assert normwise(got, oracle.async_emulated(u0, r, c1, cN, K, P, d, 42)) <= tol_for(dt)


def test_gradients_of_states_whose_images_are_out_of_range():
    """dL/dr is linear in u0 and the ends: that of the scaled rod, scaled."""
    N, K, dt = 5000, 300, "f64"
    u0, r, c1, cN, x = rod(dt, N, 4)
    g = torch.from_numpy(np.random.default_rng(5).uniform(0, 2.0 ** -20, N)).to(DEV)
    plan = AdjointPlan(N, K, torch.float64)
    gu, gr, uK = plan.adjoint(x, g, r, c1 * BIG[dt], cN * BIG[dt], want_uK=True)
    rgu, rgr = oracle.adjoint(u0, g.cpu().numpy(), r, c1, cN, K)
    assert normwise(scaled(uK, dt), oracle.sync(u0, r, c1, cN, K)) <= tol_for(dt)
    assert normwise(gu.cpu().numpy(), rgu) <= tol_for(dt)
    scale = K * 2.0 ** -20 * float(np.abs(np.diff(oracle.sync(u0, r, c1, cN, K - 1), 2)).sum())
    assert abs(float(gr) / BIG[dt] - rgr) <= tol_for(dt) * max(abs(rgr), scale)
