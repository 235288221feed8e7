"""A member's run and gradients do not depend on how many members run beside it:
ensembles on both sides of the member counts where the adjoint of short rods
changes its kernels, against the first and last members run by themselves."""
import numpy as np
import pytest
import torch

from paper_1510_08982_amd.heat import EnsemblePlan
from _helpers import print_case, tol_for, torch_dtype

pytestmark = pytest.mark.gpu
DEV = "cuda"


@pytest.mark.parametrize("N,d,dt,ring,members", [
    (193, 3, "f64", True, (2, 512, 513)), (193, 0, "f32", True, (2, 256, 600)),
    (254, 3, "f64", True, (2, 256, 257)), (254, 0, "f64", True, (2, 300)),
    (258, 0, "f64", False, (256, 257)), (258, 7, "f64", False, (512, 513)),
    (258, 0, "f32", False, (512, 513)), (255, 5, "f32", True, (256, 257)),
    (100, 3, "f64", False, (2, 1025)),
])
def test_members_keep_their_bits(N, d, dt, ring, members):
    K, P, f = 41, 32, torch_dtype(dt)
    rng = np.random.default_rng(N + d)
    E = max(members)
    u0, gK = (torch.from_numpy(rng.uniform(-1, 1, (E, N))).to(DEV, f) for _ in range(2))
    seeds = torch.from_numpy(rng.integers(0, 2 ** 63 - 1, E)).to(DEV)
    c1, cN = (0.0, 0.0) if ring else (0.75, -0.5)
    few = [0, 1]
    out = {}
    for n in members:
        pick = torch.tensor(few + list(range(2, n)), device=DEV)
        print_case(test="members", N=N, d=d, dt=dt, ring=ring, members=n)
        with EnsemblePlan(N, n, P, f, periodic=ring) as plan:
            out[n] = [t[few].cpu() for t in plan.adjoint(
                u0[pick].contiguous(), gK[pick].contiguous(), 0.45, c1, cN, K, d,
                seeds[pick].contiguous(), want_uK=True)]
    with EnsemblePlan(N, 2, P, f, periodic=ring) as plan:
        want = [t.cpu() for t in plan.adjoint(u0[:2].contiguous(), gK[:2].contiguous(), 0.45, c1,
                                              cN, K, d, seeds[:2].contiguous(), want_uK=True)]
    for n in members:
        gu, gr, g1, gN, uK = out[n]
        assert torch.equal(gu, want[0]) and torch.equal(uK, want[4])
        # sums in double of at most K N terms, each of at most 4 and 1
        for a, b in zip((gr, g1, gN), want[1:4]):
            assert float((a - b).abs().max()) <= tol_for(dt) * 4 * K * N
