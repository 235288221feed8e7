"""Where the lines between two kernels lie, as a plan reports them: each line was
measured from both sides, and a call must not take the slower one."""
import pytest

from paper_1510_08982_amd import abi

RING = abi.HEAT1D_BC_PERIODIC
F32, F64 = abi.HEAT1D_F32, abi.HEAT1D_F64


def described(N, dtype, opts):
    p = abi.heat1d_plan_create(N, dtype, opts)
    try:
        return dict(w.split("=", 1) for w in abi.heat1d_plan_describe(p).split() if "=" in w)
    finally:
        abi.heat1d_plan_destroy(p)


@pytest.mark.parametrize("N,dtype,rods,ring,steps", [
    # one workgroup, or the ring's tiles, step these as fast up to about 80 steps
    (3, F32, 1, False, 80), (1024, F32, 256, False, 80), (512, F64, 16, False, 80),
    (100, F64, 1, True, 80), (1 << 18, F64, 1, True, 80),
    # beyond them a pass is faster from 64 steps on
    (1025, F32, 1, False, 64), (100, F32, 8192, False, 64), (1000, F32, 1024, False, 64),
    (513, F64, 1, False, 64), (1 << 19, F64, 1, True, 64), (100, F32, 1, True, 64),
    (1 << 26, F32, 1, False, 64),
    # thousands of short rods on narrow tiles, by the blocks of 256 points of a rod
    (256, F32, 4097, False, 64), (257, F32, 4097, False, 80), (700, F32, 16384, False, 112),
    (1000, F32, 16384, False, 144), (1024, F32, 4097, False, 64), (1000, F64, 16384, False, 64),
])
def test_band_passes_begin_where_they_are_faster(N, dtype, rods, ring, steps):
    opts = dict(nrods=rods, boundary=RING if ring else 0)
    assert described(N, dtype, opts)["band_from"] == str(steps)


def adjoint_bytes(N, dtype, opts, steps):
    p = abi.heat1d_plan_create(N, dtype, opts)
    try:
        return [abi.heat1d_adjoint_workspace_bytes(p, K) for K in steps]
    finally:
        abi.heat1d_plan_destroy(p)


@pytest.mark.parametrize("N,rods,first", [
    (21, 1, 24), (100, 4096, 24), (256, 4096, 24), (257, 511, 24), (257, 512, 56),
    (1000, 4096, 56), (1024, 4096, 24), (1 << 20, 1, 24),
])
def test_fp64_adjoint_of_few_steps_keeps_checkpoints(N, rods, first):
    """Below the line a plan's workspace is that of a plan which names a stepping
    kernel; and the workspace of a run serves every shorter one."""
    steps = list(range(0, 130)) + [1000, 10 ** 6]  # the last: steps again on short rods
    auto = adjoint_bytes(N, F64, dict(nrods=rods), steps)
    named = adjoint_bytes(N, F64, dict(nrods=rods, sync_kernel=abi.HEAT1D_SYNC_STEP), steps)
    assert auto[:first] == named[:first] and auto[100] != named[100]
    assert all(a <= b for a, b in zip(auto, auto[1:]))


@pytest.mark.parametrize("N", [3, 10, 20])
def test_fp64_adjoint_of_rods_that_decay_in_a_few_steps_keeps_checkpoints(N):
    steps = [1, 23, 24, 100, 5000]
    assert adjoint_bytes(N, F64, {}, steps) == adjoint_bytes(
        N, F64, dict(sync_kernel=abi.HEAT1D_SYNC_STEP), steps)
