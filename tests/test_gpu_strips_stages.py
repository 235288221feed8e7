"""GPU parity of emulated asynchronous runs as strips in many stages: stages of
few steps, which hand the edges' last values on through memory, with delays up
to the longest that the history serves, and stages in which the two wavefronts
of a strip trade their points just as the wrong ones reach the edge."""
import numpy as np
import pytest
import torch

import oracle
import workloads
from paper_1510_08982_amd import abi
from paper_1510_08982_amd.heat import AsyncPlan
from _helpers import normwise, tol_for, torch_dtype, np_dtype, print_case

pytestmark = pytest.mark.gpu
DEV = "cuda"


def strips_of(plan):
    """(stages, steps of a stage, points per lane) from the plan's description."""
    word = dict(w.split("=", 1) for w in plan.describe().split() if "=" in w)
    stages, T = word["strips"].split("x")
    return int(stages), int(T), int(word["M"])


def run_against_oracle(dt, N, P, d, K, r, ring, u0, c1, cN, plan):
    f = np_dtype(dt)
    x = torch.from_numpy(u0.astype(f)).to(DEV)
    got = plan.run(x, r, c1, cN, K, d, 42).cpu().numpy()
    print_case(test="strips_stages", dt=dt, N=N, P=P, d=d, K=K, ring=ring, plan=plan.describe())
    assert plan.status() == abi.HEAT1D_OK
    if ring:
        ref = oracle.async_ensemble(u0, r, 0.0, 0.0, K, P, d, [42], every=K, periodic=True)[0][0]
    else:
        ref = oracle.async_emulated(u0, r, c1, cN, K, P, d, 42)
    err = normwise(got, ref)
    print(f"  normwise error {err:.3e}")
    assert err <= tol_for(dt)


@pytest.mark.parametrize("ring", [False, True])
@pytest.mark.parametrize("d", [50, 63])
@pytest.mark.parametrize("dt,N,P,K,r", [
    ("f64", 1418, 32, 1000, 0.25), ("f32", 1418, 32, 463, 0.25),  # a last stage of one step
    ("f64", 3000, 70, 461, 0.5), ("f32", 3000, 70, 900, 0.3),
])
def test_short_stages_read_the_history_before_it_is_replaced(dt, N, P, K, r, d, ring):
    f = np_dtype(dt)
    u0 = workloads.as_dtype(np.random.default_rng(N + K).uniform(-1, 1, N), f)
    r = workloads.as_dtype(r, f)
    with AsyncPlan(N, P, torch_dtype(dt), max_delay=d, periodic=ring) as plan:
        run_against_oracle(dt, N, P, d, K, r, ring, u0, 1.0, -1.0, plan)
        stages, T, _ = strips_of(plan)
        assert stages > 2 and T <= 32


@pytest.mark.parametrize("ring", [False, True])
@pytest.mark.parametrize("dt,N,P,d,K,r", [
    ("f64", 20000, 200, 3, 3000, 0.5), ("f64", 12800, 100, 1, 2000, 0.5),
    ("f64", 20000, 100, 3, 5000, 0.5), ("f64", 23000, 100, 16, 2000, 0.5),
    ("f64", 3200, 16, 3, 5000, 0.45), ("f32", 20000, 100, 3, 2000, 0.5),
])
def test_edge_values_are_right_where_four_points_a_lane_trade(dt, N, P, d, K, r, ring):
    """With four points a lane the wavefronts overlap by 32 points and trade
    every 32 steps: at the trade each holds the other's edge point wrong."""
    f = np_dtype(dt)
    # values that do not average out beyond the cut ends
    u0 = workloads.as_dtype(np.random.default_rng(N + K).uniform(0, 1, N), f)
    r = workloads.as_dtype(r, f)
    with AsyncPlan(N, P, torch_dtype(dt), max_delay=d, periodic=ring) as plan:
        run_against_oracle(dt, N, P, d, K, r, ring, u0, 0.0, 1.0, plan)
        _, T, M = strips_of(plan)
        assert M == 4 and T > 32


@pytest.mark.parametrize("ring", [False, True])
@pytest.mark.parametrize("dt,sub,strips", [("f64", 4, False), ("f32", 6, False), ("f32", 15, False),
                                           ("f64", 16, True), ("f32", 17, True)])
def test_stages_of_few_steps_are_left_to_the_persistent_kernel(dt, sub, strips, ring):
    N, d, K = 1000, 4, 500
    f = np_dtype(dt)
    u0 = workloads.as_dtype(np.random.default_rng(sub).uniform(-1, 1, N), f)
    r = workloads.as_dtype(0.45, f)
    with AsyncPlan(N, N // sub, torch_dtype(dt), max_delay=d, periodic=ring) as plan:
        run_against_oracle(dt, N, N // sub, d, K, r, ring, u0, 1.0, -1.0, plan)
        assert ("strips=" in plan.describe()) == strips


@pytest.mark.parametrize("dt,P,sub", [("f32", 5000, 4000), ("f64", 1900, 40)])
def test_runs_that_would_take_strips_are_refused_before_any_launch(dt, P, sub):
    """More subdomains than can be resident at once: the strips would not need that,
    but the kernel behind them does, and the refusal leaves uK alone.  (At 1900 of
    40 FP64 points all can be, and strips run.)"""
    N, d, K = P * sub, 1, 448
    x = torch.zeros(N, device=DEV, dtype=torch_dtype(dt))
    out = torch.full_like(x, 7.0)
    with AsyncPlan(N, P, torch_dtype(dt), max_delay=d) as plan:
        print_case(test="strips_occupancy", dt=dt, N=N, P=P)
        if dt == "f64":
            plan.run(x, 0.4, 0.25, 0.25, K, d, 1, out=out)
            assert strips_of(plan)[0] > 0 and float(out[0]) == 0.25
            return
        with pytest.raises(abi.Heat1dError) as refused:
            plan.run(x, 0.4, 0.25, 0.25, K, d, 1, out=out)
        assert refused.value.status == abi.HEAT1D_EOCCUPANCY
        torch.cuda.synchronize()
        assert bool((out == 7.0).all())
