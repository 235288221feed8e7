"""Gradients through emulated asynchronous runs of few steps, on both sides of the
step counts from which register tiles take them: states and dL/du0 bit for bit
those of one launch per step, dL/dr to the state tolerance times the magnitude
of its terms."""
import numpy as np
import pytest
import torch

from paper_1510_08982_amd import abi
from paper_1510_08982_amd.heat import AsyncPlan
from _helpers import print_case, tol_for, torch_dtype

pytestmark = pytest.mark.gpu
BIG, HUGE = (1 << 18) + 5, (1 << 21) + 3


@pytest.mark.parametrize("ring", [False, True])
@pytest.mark.parametrize("dt,N,sub,K", [
    ("f32", BIG, 144, 5), ("f32", BIG, 144, 6), ("f64", BIG, 200, 3), ("f64", BIG, 200, 4),
    ("f32", BIG, 600, 1), ("f32", BIG, 600, 2), ("f64", BIG, 1100, 1), ("f64", BIG, 1100, 2),
    ("f32", HUGE, 150, 11), ("f32", HUGE, 150, 12), ("f32", HUGE, 599, 7), ("f32", HUGE, 599, 8),
    ("f32", HUGE, 700, 3), ("f32", HUGE, 700, 4), ("f64", 1 << 18, 144, 1), ("f32", BIG, 16, 3),
])
def test_few_steps_are_the_per_step_launches(dt, N, sub, K, ring):
    P, d = N // sub, 4
    gen = torch.Generator(device="cuda").manual_seed(N + K)
    u0, gK = (torch.rand(N, generator=gen, device="cuda", dtype=torch_dtype(dt)) * 2 - 1
              for _ in range(2))
    print_case(test="few_steps", dt=dt, N=N, P=P, K=K, ring=ring)
    c1, cN = (0.0, 0.0) if ring else (0.25, -0.5)
    got = []
    for kernel in (abi.HEAT1D_SYNC_AUTO, abi.HEAT1D_SYNC_STEP):
        with AsyncPlan(N, P, torch_dtype(dt), max_delay=d, periodic=ring,
                       sync_kernel=kernel) as plan:
            got.append([x.cpu() for x in plan.adjoint(u0, gK, 0.37, c1, cN, K, d, 3)])
    (gu, gr, g1, gN, uK), (hu, hr, h1, hN, vK) = got
    assert torch.equal(gu, hu) and torch.equal(uK, vK)
    assert torch.isfinite(gr).all()
    # every term lambda . second difference is at most 1 x 4, by the maximum principle
    assert abs(float(gr) - float(hr)) <= tol_for(dt) * 4 * K * N
    for x, y in ((g1, h1), (gN, hN)):
        assert abs(float(x) - float(y)) <= tol_for(dt) * (1 + 0.37 * K)
