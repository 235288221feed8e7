"""The work that a user of heat1d has it do, as cases that can be timed and checked.

A case is a dict of plain values.  `prepare` makes what a program holds before the call (inputs on
the GPU, drawn from the seed alone, and the plan it keeps), `run` is one pass through the package's
public entry points, `work` counts what a pass cannot do without, and `exact` evaluates the same
outputs in 64 bits with torch alone: the synchronous iteration through the discrete Fourier symbol
of Eq.3, the asynchronous one (Eq.4) step by step with its delays drawn here.
"""
import math

import numpy as np
import torch

from paper_1510_08982_amd import abi
from paper_1510_08982_amd.heat import (AsyncPlan, BatchedPlan, EnsemblePlan, HeatFn, SyncPlan)

DEV = "cuda"
DTYPES = {"f32": torch.float32, "f64": torch.float64}
LARGEST = (1 << 26) * 2000.0  # point updates of the largest synchronous rod


def listed():
    return [
        # the paper's own rod (Section 5), one synchronous run: the smallest call, a few launches
        dict(name="paper_rod_f64", kind="sync", dtype="f64", N=100, K=1000, r=0.5, ring=False,
             tuned=False),
        # the plain method at its small size: one rod of 4096 points, many steps
        dict(name="small_rod_f64", kind="sync", dtype="f64", N=4096, K=20000, r=0.4, ring=False,
             tuned=False),
        # the headline: one rod of 2^26 points, the plan chosen by the autotuner as bench.py does
        dict(name="large_rod_f32", kind="sync", dtype="f32", N=1 << 26, K=2000, r=0.25, ring=False,
             tuned=True),
        # the periodic ring of Section 5.3 in FP64, an odd length, the plan as it comes
        dict(name="odd_ring_f64", kind="sync", dtype="f64", N=3000001, K=1500, r=0.45, ring=True,
             tuned=False),
        # the small rod run asynchronously: 16 subdomains, seeded delays 0..3
        dict(name="small_async_f64", kind="async", dtype="f64", N=4096, P=16, d=3, K=20000, r=0.4,
             mode="emulated"),
        # the large asynchronous rod, its delays replayed from a seed so that a run can be repeated
        dict(name="large_async_f32", kind="async", dtype="f32", N=1 << 24, P=1024, d=4, K=5000,
             r=0.45, mode="emulated"),
        # the same iteration as the hardware times it: halos as stale as they happen to be
        dict(name="hardware_async_f32", kind="async", dtype="f32", N=1 << 20, P=64, d=4, K=3000,
             r=0.45, mode="hardware"),
        # thousands of rods of uneven length, step count and ratio in one launch
        dict(name="ragged_batch_f32", kind="batched", dtype="f32", rods=4096, nmin=256, nmax=65536,
             kmin=500, kmax=5000, lengths=1),
        # an inverse heat problem: loss against a profile, gradients by autograd
        dict(name="heatfn_f32", kind="heatfn", dtype="f32", rods=256, N=1 << 16, K=2000, r=0.3),
        # the paper's ensemble (Fig. 3): 300 members, the norm after every step
        dict(name="paper_ensemble_f64", kind="ensemble", dtype="f64", members=300, N=100, P=100,
             d=3, K=5000, ring=False, every=1),
        # gradients through every member of that ensemble
        dict(name="ensemble_grads_f64", kind="ensemble_grads", dtype="f64", members=300, N=100,
             P=100, d=3, K=5000, ring=False),
        # gradients through the large asynchronous rod
        dict(name="async_grads_f32", kind="async_grads", dtype="f32", N=1 << 24, P=1024, d=4,
             K=5000, r=0.45),
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["sync", "sync", "sync", "async", "async", "batched", "heatfn", "ensemble",
                       "ensemble_grads", "async_grads"])
    dtype = rng.choice(["f32", "f64"])
    r = 0.5 if rng.random() < 0.15 else round(rng.uniform(0.05, 0.5), 6)
    if kind == "sync":
        N = _log(rng, 100, (1 << 26) if dtype == "f32" else (1 << 25))
        K = min(_log(rng, 100, 20000), max(100, int(LARGEST / 4 / N)))
        return dict(kind=kind, dtype=dtype, N=N, K=K, r=r, ring=rng.random() < 0.35,
                    tuned=rng.random() < 0.4)
    if kind in ("async", "async_grads"):
        N = _log(rng, 4096, (1 << 24) if dtype == "f32" else (1 << 22))
        # one workgroup owns a subdomain: a few hundred to 16384 points
        P = min(1024, max(2, _log(rng, max(2, N // 16384), max(2, N // 256))))
        K = min(_log(rng, 500, 20000), max(500, int((1 << 24) * 5000.0 / 2 / N)))
        if kind == "async_grads":
            K = min(K, 5000)
            return dict(kind=kind, dtype=dtype, N=N, P=P, d=rng.randint(1, 16), K=K, r=r)
        return dict(kind=kind, dtype=dtype, N=N, P=P, d=rng.randint(1, 16), K=K, r=r,
                    mode="emulated")
    if kind == "batched":
        nmax = _log(rng, 2000, 65536 if dtype == "f32" else 32768)
        return dict(kind=kind, dtype=dtype, rods=_log(rng, 64, 4096), nmin=256, nmax=nmax,
                    kmin=500, kmax=_log(rng, 1000, 5000), lengths=rng.randint(2, 10 ** 6))
    if kind == "heatfn":
        N = _log(rng, 500, 1 << 20)
        K = _log(rng, 100, 2000)
        rods = min(256, max(1, _log(rng, 1, max(2, (1 << 23) // N))))
        return dict(kind=kind, dtype=dtype, rods=rods, N=N, K=K, r=r)
    N = _log(rng, 20, 200)
    P = N if rng.random() < 0.6 else rng.randint(2, N)
    c = dict(kind=kind, dtype=dtype, members=_log(rng, 8, 512), N=N, P=P, d=rng.randint(1, 4),
             K=_log(rng, 500, 5000), ring=rng.random() < 0.4)
    if kind == "ensemble":
        c["every"] = rng.choice([1, 1, 10, 100])
    return c


# ------------------------------------------------------------------------------------ inputs

def _uniform(gen, n, lo, hi, dtype):
    x = torch.rand(n, generator=gen, dtype=torch.float64, device=DEV)
    return (x.mul_(hi - lo).add_(lo)).to(dtype)


def _seeds(seed, n):
    return torch.from_numpy(np.random.default_rng(seed).integers(0, 2 ** 63 - 1, n))


def _ragged(case, seed):
    """Lengths and step counts (the case's own: a plan is made for them), then r, c1, cN."""
    rng = np.random.default_rng(case["lengths"])
    n = np.rint(np.exp(rng.uniform(math.log(case["nmin"]), math.log(case["nmax"]), case["rods"])))
    n = np.clip(n.astype(np.int64), case["nmin"], case["nmax"])
    K = rng.integers(case["kmin"], case["kmax"] + 1, case["rods"])
    rng = np.random.default_rng(seed)
    return (n, K, rng.uniform(0.05, 0.5, case["rods"]), rng.uniform(-1, 1, case["rods"]),
            rng.uniform(-1, 1, case["rods"]))


def _inputs(case, seed):
    """The arrays and scalars of a case, from the seed alone."""
    gen = torch.Generator(device=DEV).manual_seed(seed)
    dt, kind = DTYPES[case["dtype"]], case["kind"]
    if kind == "sync":
        # sine modes of falling wavelength with a little noise, as the large rod has them
        N = case["N"]
        a = np.random.default_rng(seed).uniform(-1, 1, 8)
        i = torch.arange(N, dtype=torch.float64, device=DEV)
        u = _uniform(gen, N, -0.01, 0.01, torch.float64)
        for j in range(8):
            if 8 ** j < N - 1:
                u.add_(torch.sin(i * (math.pi * 8 ** j * (2 if case["ring"] else 1) / (N - 1))),
                       alpha=float(a[j]))
        return dict(u0=u.to(dt), c1=0.25, cN=-0.5)
    if kind in ("async", "async_grads"):
        s = dict(u0=_uniform(gen, case["N"], -1, 1, dt), c1=1.0, cN=-1.0,
                 seed=int(_seeds(seed, 1)[0]))
        if kind == "async_grads":
            s["gK"] = _uniform(gen, case["N"], -1, 1, dt)
        return s
    if kind == "batched":
        n, K, r, c1, cN = _ragged(case, seed)
        off = np.concatenate([[0], np.cumsum(n)])
        dev = [torch.from_numpy(x).to(DEV) for x in (off, r, c1, cN, K.astype(np.int32))]
        return dict(u0=_uniform(gen, int(off[-1]), -1, 1, dt), n=n, K=K, dev=dev)
    if kind == "heatfn":
        u0 = _uniform(gen, case["rods"] * case["N"], -1, 1, dt)
        # the profile to be met: another draw, smoothed
        t = _uniform(gen, case["rods"] * case["N"], -1, 1, torch.float64)
        t = torch.nn.functional.avg_pool1d(t.view(case["rods"], 1, -1), 65, 1, 32)
        return dict(u0=u0, target=t.reshape(-1).to(dt), c1=0.1, cN=-0.2)
    # the paper's rod (cos^2 profile, ends 1 and 0), each member a little off it
    E, N = case["members"], case["N"]
    i = torch.arange(N, dtype=torch.float64, device=DEV)
    u = torch.cos(i * (3 * math.pi / (2 * (N - 1)))) ** 2
    u = (u + 0.05 * _uniform(gen, E * N, -1, 1, torch.float64).view(E, N)).to(dt)
    s = dict(u0=u.contiguous(), seeds=_seeds(seed, E).to(DEV))
    if kind == "ensemble_grads":
        s["gK"] = _uniform(gen, E * N, -1, 1, dt).view(E, N)
    return s


def prepare(case, seed):
    s = _inputs(case, seed)
    s["case"] = case
    dt, kind = DTYPES[case["dtype"]], case["kind"]
    if kind == "sync":
        bc = abi.HEAT1D_BC_PERIODIC if case["ring"] else abi.HEAT1D_BC_DIRICHLET
        s["plan"] = SyncPlan(case["N"], dt, boundary=bc)
        if case["tuned"]:
            s["plan"].autotune(s["u0"], case["r"], min(512, case["K"]))
    elif kind in ("async", "async_grads"):
        s["plan"] = AsyncPlan(case["N"], case["P"], dt, max_delay=case["d"])
    elif kind == "batched":
        s["plan"] = BatchedPlan(s["n"], s["K"], dt)
    elif kind == "heatfn":
        s["u0"].requires_grad_(True)
        s["par"] = [torch.tensor(x, dtype=torch.float64, device="cpu", requires_grad=True)
                    for x in (case["r"], s["c1"], s["cN"])]
    else:
        s["plan"] = EnsemblePlan(case["N"], case["members"], case["P"], dt, periodic=case["ring"])
    return s


def run(s):
    c, kind = s["case"], s["case"]["kind"]
    if kind == "sync":
        return s["plan"].run(s["u0"], c["r"], s["c1"], s["cN"], c["K"])
    if kind == "async":
        mode = abi.HEAT1D_ASYNC_EMULATED if c["mode"] == "emulated" else abi.HEAT1D_ASYNC_HARDWARE
        return s["plan"].run(s["u0"], c["r"], s["c1"], s["cN"], c["K"], c["d"], s["seed"], mode)
    if kind == "async_grads":
        gu, gr, g1, gN, uK = s["plan"].adjoint(s["u0"], s["gK"], c["r"], s["c1"], s["cN"], c["K"],
                                               c["d"], s["seed"])
        return dict(grad_u0=gu, grad_r=gr, grad_c1=g1, grad_cN=gN, uK=uK)
    if kind == "batched":
        return s["plan"].run(s["u0"], *s["dev"])
    if kind == "heatfn":
        r, c1, cN = s["par"]
        uK = HeatFn.apply(s["u0"], r, c1, cN, c["K"], c["rods"])
        loss = 0.5 * ((uK - s["target"]) ** 2).sum()
        gu, gr, g1, gN = torch.autograd.grad(loss, [s["u0"], r, c1, cN])
        return dict(uK=uK.detach(), grad_u0=gu, grad_r=gr, grad_c1=g1, grad_cN=gN)
    if kind == "ensemble":
        uK, norms = s["plan"].run(s["u0"], 0.5, 1.0, 0.0, c["K"], c["d"], s["seeds"], c["every"])
        return dict(uK=uK, norms=norms)
    gu, gr, g1, gN, uK = s["plan"].adjoint(s["u0"], s["gK"], 0.5, 1.0, 0.0, c["K"], c["d"],
                                           s["seeds"], want_uK=True)
    return dict(grad_u0=gu, grad_r=gr, grad_c1=g1, grad_cN=gN, uK=uK)


def _reach(r, K):
    """How far a point's weight in u(K) stays above about 1e-16 of the whole, in points."""
    return min(float(K), 8.3 * math.sqrt(2 * r * K))


def work(case):
    """Each input read and each output written once; and, as u(K) is a linear map of u0 whose rows
    hold 2 reach + 1 weights that matter (fewer on a shorter rod), two operations for each of them."""
    s, kind = (4 if case["dtype"] == "f32" else 8), case["kind"]
    if kind == "batched":
        n, K, r, _, _ = _ragged(case, 0)
        flops = sum(2.0 * a * min(2 * _reach(b, k) + 1, 2 * a) for a, k, b in zip(n, K, r))
        return dict(bytes=2.0 * s * float(n.sum()), flops=flops)
    N, K, r = case["N"], case["K"], case.get("r", 0.5)
    rods = case.get("rods", case.get("members", 1))
    pts = float(N) * rods
    arrays = {"sync": 2, "async": 2, "ensemble": 2, "heatfn": 4, "async_grads": 4,
              "ensemble_grads": 4}[kind]
    maps = {"heatfn": 3, "async_grads": 3, "ensemble_grads": 3}.get(kind, 1)
    nbytes = arrays * s * pts
    if kind == "ensemble":
        nbytes += 8.0 * rods * (K // case["every"] + 1)
    if kind in ("ensemble", "ensemble_grads"):
        # every point reads with a delay of its own at every step: no step can be left out
        return dict(bytes=nbytes, flops=4.0 * pts * K * (1 if kind == "ensemble" else 3))
    return dict(bytes=nbytes, flops=2.0 * pts * min(2 * _reach(r, K) + 1, 2 * N) * maps)


# ------------------------------------------------------------------------------------ 64 bits

def _rounded(x, case):
    return float(np.float32(x)) if case["dtype"] == "f32" else float(x)


def _symbol(n, r, K):
    """g^K for g = 1 - 4 r sin^2(w/2) at the n//2 + 1 frequencies of a real transform of length n."""
    h = torch.arange(n // 2 + 1, dtype=torch.float64, device=DEV) * (math.pi / n)
    a = 4 * r * torch.sin(h) ** 2
    b = (2 - 4 * r) + 4 * r * torch.cos(h) ** 2  # 2 - a without cancellation
    low = torch.exp(K * torch.log1p(-a.clamp(max=0.999999)))
    high = torch.exp(K * torch.log1p(-b.clamp(min=0.0, max=1.0 - 1e-300)))
    mid = (1 - a).abs() ** K
    g = torch.where(a < 0.5, low, torch.where(b < 0.5, high, mid))
    return torch.where((a > 1) & (K % 2 == 1), -g, g)


def _extend(v, ring, m):
    """Rods of v (rows, points), m points more on each side: around the ring, or odd about both
    ends (zero there)."""
    N = v.shape[1]
    i = torch.arange(-m, N + m, device=DEV)
    if ring:
        return v[:, i % N]
    i = i % (2 * (N - 1))
    back = i > N - 1
    x = v[:, torch.where(back, 2 * (N - 1) - i, i)]
    return torch.where(back, -x, x)


def _apply(v, r, K, ring=False, laplacian=False):
    """K steps of Eq.3 (zero ends, or a ring) of the rows of v, as one cyclic convolution; with
    `laplacian`, of the second difference of v, and K steps of that."""
    rows, N = v.shape
    m = min(K, int(13 * math.sqrt(2 * r * K)) + 40) + 2
    n = 1 << (N + 2 * m - 1).bit_length()
    x = torch.fft.rfft(_extend(v, ring, m), n=n)
    h = torch.arange(n // 2 + 1, dtype=torch.float64, device=DEV) * (math.pi / n)
    x.mul_(_symbol(n, r, K) * (-4 * torch.sin(h) ** 2 if laplacian else 1.0))
    return torch.fft.irfft(x, n=n)[:, m:m + N]


def _sync(u0, r, c1, cN, K, ring=False):
    u = u0.double()
    if ring:
        return _apply(u, r, K, True)
    N = u.shape[1]
    s = c1 + (cN - c1) * torch.arange(N, dtype=torch.float64, device=DEV) / (N - 1)
    v = u - s
    v[:, 0] = v[:, -1] = 0
    out = _apply(v, r, K) + s
    out[:, 0], out[:, -1] = c1, cN
    return out


_M64 = (1 << 64) - 1


def _i64(x):
    x &= _M64
    return x - (1 << 64) if x >> 63 else x


def _shr(z, n):
    return (z >> n) & ((1 << (64 - n)) - 1)


def _sm64(s):
    """SplitMix64's output function on int64 tensors."""
    z = s + _i64(0x9E3779B97F4A7C15)
    z = (z ^ _shr(z, 30)) * _i64(0xBF58476D1CE4E5B9)
    z = (z ^ _shr(z, 27)) * _i64(0x94D049BB133111EB)
    return z ^ _shr(z, 31)


def _delays(seeds, k0, k1, P, d):
    """Delay of (step, member, subdomain, side), for steps k0..k1-1."""
    k = torch.arange(k0, k1, device=DEV).view(-1, 1, 1, 1)
    p = torch.arange(P, device=DEV).view(1, 1, -1, 1)
    side = torch.arange(2, device=DEV).view(1, 1, 1, 2)
    x = _sm64(seeds.view(1, -1, 1, 1) ^ _sm64(((k * P + p) << 1) | side))
    return (_shr(x, 32) * (d + 1)) >> 32


class _Edges:
    """Where the reads across subdomain edges are: point `at` reads its neighbour `other` with the
    delay of entry `col` of a step's table (2 P entries)."""

    def __init__(self, N, P, ring):
        lo = torch.tensor([p * N // P for p in range(P + 1)], device=DEV)
        p = torch.arange(P, device=DEV)
        at = torch.cat([lo[:-1], lo[1:] - 1])
        other = torch.cat([lo[:-1] - 1, lo[1:]])
        col = torch.cat([2 * p, 2 * p + 1])
        if ring:
            keep = torch.full_like(at, P > 1, dtype=torch.bool)
        else:
            keep = (at > 0) & (at < N - 1) & (other >= 0) & (other < N)
        self.at, self.col, self.other = at[keep], col[keep], other[keep] % N
        self.n = int(self.at.numel())


def _async(u0, gK, r, c1, cN, K, P, d, seeds, ring, every=0):
    """The emulated run of the rows of u0 (Eq.4), with the norms every `every` steps, and with gK
    its gradients: dL/dr from the derivative of the run in r, the others from the transposed run."""
    E, N = u0.shape
    u = u0.double().clone()
    if not ring:
        u[:, 0], u[:, -1] = c1, cN
    e = _Edges(N, P, ring)
    v = torch.zeros_like(u) if gK is not None else None
    H = d + 1
    hist = torch.zeros((H, E, e.n), dtype=torch.float64, device=DEV)
    vist = torch.zeros_like(hist)
    rows = torch.arange(E, device=DEV).view(-1, 1)
    cols = torch.arange(e.n, device=DEV).view(1, -1)
    norms = [u.norm(dim=1)] if every else None
    chunk = max(1, min(K, (1 << 22) // max(1, E * 2 * P)))
    D = None
    for k in range(K):
        if k % chunk == 0:
            D = _delays(seeds, k, min(K, k + chunk), P, d).view(-1, E, 2 * P)[:, :, e.col]
        hist[k % H] = u[:, e.other]
        slot = (k - D[k % chunk]).clamp_(min=0) % H
        lap = torch.empty_like(u)
        lap[:, 1:-1] = u[:, :-2] + u[:, 2:] - 2 * u[:, 1:-1]
        if ring:
            lap[:, 0] = u[:, -1] + u[:, 1] - 2 * u[:, 0]
            lap[:, -1] = u[:, -2] + u[:, 0] - 2 * u[:, -1]
        else:
            lap[:, 0] = lap[:, -1] = 0
        # index_add_ because the two sides of one point may both be edges
        lap.index_add_(1, e.at, hist[slot, rows, cols] - hist[k % H])
        if v is not None:
            vist[k % H] = v[:, e.other]
            lv = torch.zeros_like(v)
            lv[:, 1:-1] = v[:, :-2] + v[:, 2:] - 2 * v[:, 1:-1]
            if ring:
                lv[:, 0] = v[:, -1] + v[:, 1] - 2 * v[:, 0]
                lv[:, -1] = v[:, -2] + v[:, 0] - 2 * v[:, -1]
            lv.index_add_(1, e.at, vist[slot, rows, cols] - vist[k % H])
            v.add_(lv, alpha=r).add_(lap)
            if not ring:
                v[:, 0] = v[:, -1] = 0
        u.add_(lap, alpha=r)
        if not ring:
            u[:, 0], u[:, -1] = c1, cN
        if every and (k + 1) % every == 0:
            norms.append(u.norm(dim=1))
    if gK is None:
        return (u, torch.stack(norms, 1)) if every else u
    g = gK.double()
    grad_r = (g * v).sum(1)
    lam = g.clone()
    if not ring:
        lam[:, 0] = lam[:, -1] = 0
    g1 = torch.zeros(E, dtype=torch.float64, device=DEV)
    gN = torch.zeros_like(g1)
    # what the delayed reads return to the points that were read, by the step they read
    few, where = torch.unique(e.other, return_inverse=True)
    keep = torch.zeros((H, E, int(few.numel())), dtype=torch.float64, device=DEV)
    for k in range(K - 1, -1, -1):
        if D is None or k % chunk == chunk - 1 or k == K - 1:
            k0 = k - k % chunk
            D = _delays(seeds, k0, min(K, k0 + chunk), P, d).view(-1, E, 2 * P)[:, :, e.col]
        if not ring:
            g1 += r * lam[:, 1]
            gN += r * lam[:, -2]
        new = lam * (1 - 2 * r)
        new[:, :-1] += r * lam[:, 1:]
        new[:, 1:] += r * lam[:, :-1]
        if ring:
            new[:, -1] += r * lam[:, 0]
            new[:, 0] += r * lam[:, -1]
        back = r * lam[:, e.at]
        new.index_add_(1, e.other, -back)
        slot = (k - D[k % chunk]).clamp_(min=0) % H
        keep.index_put_((slot, rows.expand_as(slot), where.view(1, -1).expand_as(slot)), back,
                        accumulate=True)
        new[:, few] += keep[k % H]
        keep[k % H] = 0
        if not ring:
            new[:, 0] = new[:, -1] = 0
        lam = new
    if not ring:
        g1, gN = g1 + g[:, 0], gN + g[:, -1]
    return dict(grad_u0=lam, grad_r=grad_r, grad_c1=g1, grad_cN=gN, uK=u)


def exact(case, seed):
    s, kind = _inputs(case, seed), case["kind"]
    r = _rounded(case.get("r", 0.5), case)
    if kind == "sync":
        c1, cN = _rounded(s["c1"], case), _rounded(s["cN"], case)
        return _sync(s["u0"].view(1, -1), r, c1, cN, case["K"], case["ring"]).view(-1)
    if kind == "batched":
        n, K, rr, c1, cN = _ragged(case, seed)
        off = np.concatenate([[0], np.cumsum(n)])
        return torch.cat([_sync(s["u0"][off[b]:off[b + 1]].view(1, -1), _rounded(rr[b], case),
                                _rounded(c1[b], case), _rounded(cN[b], case), int(K[b])).view(-1)
                          for b in range(case["rods"])])
    if kind == "heatfn":
        B, N, K = case["rods"], case["N"], case["K"]
        c1, cN = _rounded(s["c1"], case), _rounded(s["cN"], case)
        u0 = s["u0"].detach().double().view(B, N)
        uK = _sync(u0, r, c1, cN, K)
        g = uK - s["target"].double().view(B, N)
        gi = g.clone()
        gi[:, 0] = gi[:, -1] = 0
        lam = _apply(gi, r, K)
        lam[:, 0] = lam[:, -1] = 0
        line = c1 + (cN - c1) * torch.arange(N, dtype=torch.float64, device=DEV) / (N - 1)
        v = u0 - line
        v[:, 0] = v[:, -1] = 0
        # A and the second difference commute: every one of the K terms of dL/dr is the same
        grad_r = K * (gi * _apply(v, r, K - 1, laplacian=True)).sum()
        one = torch.zeros((1, N), dtype=torch.float64, device=DEV)
        w = _sync(one, r, 1.0, 0.0, K)[0]
        return dict(uK=uK.reshape(-1), grad_u0=lam.reshape(-1), grad_r=grad_r,
                    grad_c1=(g * w).sum(), grad_cN=(g * w.flip(0)).sum())
    if kind == "ensemble":
        u, norms = _async(s["u0"], None, 0.5, 1.0, 0.0, case["K"], case["P"], case["d"],
                          s["seeds"], case["ring"], case["every"])
        return dict(uK=u, norms=norms)
    if kind == "ensemble_grads":
        return _async(s["u0"], s["gK"], 0.5, 1.0, 0.0, case["K"], case["P"], case["d"],
                      s["seeds"], case["ring"])
    if case.get("mode") == "hardware":
        return None  # which values a run reads depends on timing
    if case["K"] > (5000 if kind == "async_grads" else 20000):
        return None
    seeds = torch.tensor([s["seed"]], device=DEV)
    c1, cN = _rounded(s["c1"], case), _rounded(s["cN"], case)
    if kind == "async":
        return _async(s["u0"].view(1, -1), None, r, c1, cN, case["K"], case["P"], case["d"], seeds,
                      False).view(-1)
    got = _async(s["u0"].view(1, -1), s["gK"].view(1, -1), r, c1, cN, case["K"], case["P"],
                 case["d"], seeds, False)
    return {k: x.reshape(-1) for k, x in got.items()}
