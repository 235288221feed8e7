"""FP32 rods of a batch at small r and thousands of steps: their passes keep the FP32
tolerance against the oracle on a smooth profile, where stepping, which
heat1d_run_sync keeps for such rods, drifts; the two entry points differ by no more
than that drift, and agree within the tolerance where both take passes."""
import numpy as np
import pytest
import torch

import oracle
import workloads
from paper_1510_08982_amd.heat import BatchedPlan, SyncPlan
from _helpers import F32_TOL, normwise, print_case

pytestmark = pytest.mark.gpu


def test_small_r_and_thousands_of_steps():
    f = np.float32
    rods = [(3000, 2000, 0.05), (3000, 5000, 0.05), (4097, 3000, 0.1), (5000, 5166, 0.07),
            (2500, 2000, 0.3), (9001, 4000, 0.45)]
    n, K = np.array([x[0] for x in rods]), np.array([x[1] for x in rods])
    r = workloads.as_dtype(np.array([x[2] for x in rods]), f)
    off = np.concatenate([[0], np.cumsum(n)]).astype(np.int64)
    u0 = np.concatenate([np.cos(3 * np.pi * np.arange(m) / (2 * (m - 1))) ** 2 for m in n])
    u0 = workloads.as_dtype(u0, f)
    x = torch.from_numpy(u0.astype(f)).to("cuda")
    ones, zeros = torch.ones(len(n), dtype=torch.float64, device="cuda"), torch.zeros(
        len(n), dtype=torch.float64, device="cuda")
    with BatchedPlan(n, K, torch.float32) as plan:
        assert f"band_rods={len(n)}" in plan.describe()
        got = plan.run(x, torch.from_numpy(off).to("cuda"), torch.from_numpy(r).to("cuda"), ones,
                       zeros, torch.from_numpy(K.astype(np.int32)).to("cuda")).cpu().numpy()
    for b in range(len(n)):
        sl = slice(off[b], off[b + 1])
        ref = oracle.sync(u0[sl], r[b], 1.0, 0.0, int(K[b]))
        one = SyncPlan(int(n[b]), torch.float32).run(x[sl].clone(), float(r[b]), 1.0, 0.0,
                                                     int(K[b])).cpu().numpy()
        err, sync = normwise(got[sl], ref), normwise(one, ref)
        print_case(test="batched_drift", N=n[b], K=K[b], r=r[b], batch=err, sync=sync)
        assert err <= F32_TOL
        assert normwise(got[sl], one) <= sync + F32_TOL
        if K[b] * (1 + 0.1 / r[b]) <= 6200:   # a pass there too
            assert normwise(got[sl], one) <= F32_TOL
