"""Band passes where little of the state is left: short rods between zero ends, and
gradients, which always are, lose their slowest mode by e^(r K pi^2 / (N-1)^2).
The tolerance is relative to what is left, as steps keep it.  r has few bits, so that
the oracle's 1 - 2r is exact."""
import math

import numpy as np
import pytest
import torch

import oracle
import workloads
from paper_1510_08982_amd.heat import AdjointPlan, BatchedPlan, SyncPlan
from _helpers import normwise, np_dtype, print_case, tol_for, torch_dtype

pytestmark = pytest.mark.gpu
DEV = "cuda"


def steps_for(decay, N, r):
    return int(decay * (N - 1) ** 2 / (math.pi ** 2 * r))


@pytest.mark.parametrize("dt", ["f32", "f64"])
@pytest.mark.parametrize("N,B,r", [(16, 1, 0.5), (22, 1, 0.25), (30, 3, 0.5), (64, 1, 0.375),
                                   (100, 2, 0.5), (100, 1, 0.0625)])
@pytest.mark.parametrize("decay", [0.55, 0.65, 2, 6, 20, 60, 70])
def test_short_rods_between_zero_ends(decay, N, B, r, dt):
    K = steps_for(decay, N, r)
    if dt == "f32" and K * (1 + 0.1 / r) > 6200:
        pytest.skip("FP32 runs of this length keep stepping")
    u0 = workloads.as_dtype(np.random.default_rng(N + K).uniform(-1, 1, (B, N)), np_dtype(dt))
    x = torch.from_numpy(u0.astype(np_dtype(dt)).reshape(-1)).to(DEV)
    print_case(test="decay", dt=dt, N=N, B=B, K=K, r=r)
    got = SyncPlan(N, torch_dtype(dt), nrods=B).run(x, r, 0.0, 0.0, K).cpu().numpy().reshape(B, N)
    for b in range(B):
        err = normwise(got[b], oracle.sync(u0[b], r, 0.0, 0.0, K))
        print(f"  normwise error {err:.3e}")
        assert err <= tol_for(dt)


@pytest.mark.parametrize("N,B,r", [(4, 1, 0.25), (16, 2, 0.5), (17, 1, 0.25), (30, 3, 0.5),
                                   (100, 1, 0.375), (300, 1, 0.5)])
@pytest.mark.parametrize("decay", [0.3, 1, 8, 30, 66])
def test_fp64_gradients_of_short_rods(decay, N, B, r):
    K = max(1, steps_for(decay, N, r))
    if K > 60000:
        pytest.skip("a long oracle run")
    rng = np.random.default_rng(N + K)
    u0, gK = rng.uniform(0, 1, (B, N)), rng.uniform(0, 1, (B, N))
    print_case(test="decay_adjoint", N=N, B=B, K=K, r=r)
    plan = AdjointPlan(N, K, torch.float64, nrods=B)
    gu, gr, uK = plan.adjoint(*(torch.from_numpy(a.reshape(-1)).to(DEV) for a in (u0, gK)), r, 0.0,
                              0.0, want_uK=True)
    gu, gr, uK = gu.cpu().numpy().reshape(B, N), gr.cpu().numpy(), uK.cpu().numpy().reshape(B, N)
    for b in range(B):
        rgu, rgr = oracle.adjoint(u0[b], gK[b], r, 0.0, 0.0, K)
        assert normwise(gu[b], rgu) <= tol_for("f64")
        assert normwise(uK[b], oracle.sync(u0[b], r, 0.0, 0.0, K)) <= tol_for("f64")
        # all K terms of dL/dr are alike and none cancels: lambda and u are positive, u concave
        assert abs(gr[b] - rgr) <= 1e-11 * abs(rgr)


@pytest.mark.parametrize("dt", ["f32", "f64"])
def test_short_rods_of_a_batch(dt):
    """Rods on both sides of the decay from which their workgroup steps them, bit for
    bit as one launch per step does."""
    f = np_dtype(dt)
    n = np.array([3, 4, 21, 30, 64, 65, 100, 160, 256, 257, 300, 2050])
    K = np.array([448, 500, 600, 4000, 3000, 450, 5000, 5000, 5000, 5166, 700, 900])
    r = np.array([0.5, 0.25, 0.375, 0.125, 0.5, 0.0625, 0.5, 0.5, 0.25, 0.5, 0.375, 0.25])
    off = np.concatenate([[0], np.cumsum(n)]).astype(np.int64)
    u0 = workloads.as_dtype(np.random.default_rng(9).uniform(-1, 1, int(off[-1])), f)
    x = torch.from_numpy(u0.astype(f)).to(DEV)
    z = torch.zeros(n.size, dtype=torch.float64, device=DEV)
    with BatchedPlan(n, K, torch_dtype(dt)) as plan:
        assert f"band_rods={n.size}" in plan.describe()
        got = plan.run(x, torch.from_numpy(off).to(DEV), torch.from_numpy(r).to(DEV), z, z,
                       torch.from_numpy(K.astype(np.int32)).to(DEV))
    stepped = 0
    for b in range(n.size):
        sl = slice(off[b], off[b + 1])
        ref = oracle.sync(u0[sl], r[b], 0.0, 0.0, int(K[b]))
        decay = r[b] * K[b] * math.pi ** 2 / (n[b] - 1) ** 2
        if np.abs(ref).max() > 1e-30:   # (FP32 underflows below that)
            assert normwise(got[sl].cpu().numpy(), ref) <= tol_for(dt), (n[b], K[b], decay)
        if decay > 0.6:
            one = SyncPlan(int(n[b]), torch_dtype(dt), sync_kernel=1).run(x[sl].clone(), float(r[b]),
                                                                          0.0, 0.0, int(K[b]))
            assert torch.equal(got[sl], one)
            stepped += 1
    assert 4 <= stepped <= n.size - 4
