"""What a short probe of the autotuner leaves to long runs: band passes, whose cost
hardly depends on the steps, from as many steps on as the probe's times say."""
import pytest
import torch

from paper_1510_08982_amd import abi
from paper_1510_08982_amd.heat import SyncPlan
from _helpers import print_case, torch_dtype

pytestmark = pytest.mark.gpu


def band_from(plan):
    words = dict(w.split("=", 1) for w in plan.describe().split() if "=" in w)
    return int(words["band_from"])


@pytest.mark.parametrize("ring", [False, True])
@pytest.mark.parametrize("dt,N,probe", [("f32", 256, 16), ("f32", 256, 64), ("f64", 100, 64),
                                        ("f32", 100000, 64), ("f64", 5000, 500)])
def test_a_short_probe_keeps_passes_for_long_runs(dt, N, probe, ring):
    K = 3000
    x = torch.rand(N, generator=torch.Generator("cuda").manual_seed(N), device="cuda",
                   dtype=torch_dtype(dt))
    bc = abi.HEAT1D_BC_PERIODIC if ring else abi.HEAT1D_BC_DIRICHLET
    plan, plain = (SyncPlan(N, torch_dtype(dt), boundary=bc) for _ in range(2))
    least = band_from(plain)
    for _ in range(2):   # a second probe starts from the same line
        plan.autotune(x, 0.4, probe)
        print_case(test="autotune_band", dt=dt, N=N, probe=probe, plan=plan.describe())
        # a step of the fastest kernel takes a fiftieth of a pass or more at these sizes
        assert least <= band_from(plan) <= 1000
        assert torch.equal(plan.run(x, 0.4, 0.25, -0.5, K), plain.run(x, 0.4, 0.25, -0.5, K))
    named = SyncPlan(N, torch_dtype(dt), boundary=bc, sync_kernel=abi.HEAT1D_SYNC_TILED)
    named.autotune(x, 0.4, probe)   # a plan that names a kernel has no passes
    assert "band_from" not in named.describe()
