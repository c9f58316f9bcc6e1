"""The transverse passes off the ordinary sizes: the compile-time 128- and 512-point
passes over several tiles per workgroup, with and without a cut-off; the passes
before a bf16 grid; lengths that the general kernels have no plan for; arrays of
4 GiB and more."""
from functools import lru_cache

import numpy as np
import pytest
import torch

from oracle import cutoff, recon
from paper_0808_3510_amd import inputs, pat

pytestmark = pytest.mark.gpu
DEV = "cuda"
OPS = ["reconstruct", "reconstruct_adjoint", "forward", "forward_adjoint"]
TOL = {"f32": 1e-5, "f64": 1e-9}


def geo(n1, n2, nt, nz):
    return dict(n1=n1, n2=n2, nt=nt, nz=nz, dx=1.0, dt=0.9, dz=1.1, vs=1.05)


def plan_of(g, prec, **kw):
    return pat.Plan(g["n1"], g["n2"], g["nt"], g["nz"], g["dx"], g["dt"], g["dz"], g["vs"], precision=prec, device=DEV, **kw)


def data(g, op, seed):
    n = g["nt"] if op in ("reconstruct", "forward_adjoint") else g["nz"]
    return inputs.random_array((g["n1"], g["n2"], n) if g["n2"] > 1 else (g["n1"], n), seed)


def errors(y, exp):
    d = y.cpu().double().numpy() - exp
    return np.linalg.norm(d) / np.linalg.norm(exp), np.abs(d).max() / np.abs(exp).max()


@lru_cache(maxsize=1)
def expected(n1, n2, nt, nz, op):
    g = geo(n1, n2, nt, nz)
    x = data(g, op, 3000 + n1)
    return x, getattr(recon, op)(x, g)


# two to four tiles per resident workgroup on x1 and c2r (x2) over the time axis (R and A^T
# forward, R^T and A inverse), some workgroups one fewer
MANY = [(128, 98, 1050, 8), (512, 66, 520, 8), (98, 128, 1050, 8), (34, 512, 1026, 6)]


@pytest.mark.parametrize("prec", ["f32", "f64"])
@pytest.mark.parametrize("op", ["reconstruct", "reconstruct_adjoint"])
@pytest.mark.parametrize("n1,n2,nt,nz", MANY)
def test_many_tiles_per_workgroup(n1, n2, nt, nz, op, prec):
    x, exp = expected(n1, n2, nt, nz, op)
    plan = plan_of(geo(n1, n2, nt, nz), prec)
    rel, mx = errors(getattr(plan, op)(torch.from_numpy(x).to(DEV, plan.dtype)), exp)
    print(f"  {op} {prec} {n1}x{n2}x{nt} -> {nz}: {rel:.2e}, max {mx:.2e}", flush=True)
    assert rel <= TOL[prec] and mx <= TOL[prec], (rel, mx)


def weights(n1, n2, nt, eps):
    """w_cut over the data grid: it depends on the distances min(s, n - s) to the faces, up
    to 2 eps, so a small box holds every value."""
    e = int(np.ceil(2 * eps))
    table = torch.from_numpy(cutoff.apply(np.ones((4 * e,) * 3), geo(4 * e, 4 * e, 4 * e, 2), eps)[:e + 1, :e + 1, :e + 1])
    band = [torch.tensor([min(s, n - s, e) for s in range(n)]) for n in (n1, n2, nt)]
    return table.contiguous().to(DEV)[band[0].to(DEV)][:, band[1].to(DEV)][:, :, band[2].to(DEV)]


@pytest.mark.parametrize("n1,n2,nt,nz", [(128, 96, 1024, 8), (256, 70, 520, 8), (512, 64, 512, 8)])
@pytest.mark.parametrize("eps", [4.0, 2.5])
@pytest.mark.parametrize("prec", ["f32", "f64"])
def test_cutoff_over_many_tiles(n1, n2, nt, nz, eps, prec):
    """The weights, applied by x1 as it loads and by c2r as it stores, whose slices change
    with the detector column: against the same plan without a cut-off on data weighted
    outside, R(w p), w R^T(q), w A(f) and A^T(w p).  FP32 1e-6, FP64 1e-13 (one
    rounding of the weight and of each product, with a margin of 10)."""
    g = geo(n1, n2, nt, nz)
    a, b = plan_of(g, prec, cutoff=eps), plan_of(g, prec)
    w = weights(n1, n2, nt, eps)
    assert 0 < (w < 1).double().mean().item() < 0.9
    worst = 0.0
    for op in OPS:
        x = torch.from_numpy(data(g, op, 3100 + n1)).to(DEV, a.dtype)
        on_data = op in ("reconstruct", "forward_adjoint")
        got = getattr(a, op)(x).double()
        exp = getattr(b, op)((w * x).to(a.dtype)).double() if on_data else w * getattr(b, op)(x).double()
        worst = max(worst, ((got - exp).norm() / exp.norm()).item(), ((got - exp).abs().max() / exp.abs().max()).item())
    print(f"  {prec} eps={eps} {n1}x{n2}x{nt}: {worst:.2e}", flush=True)
    assert worst <= {"f32": 1e-6, "f64": 1e-13}[prec], worst


# the pipelines before a bf16 grid at radices up to 7 and up to 23 and at 512 points
BF16 = [(24, 20, 48, 24), (46, 26, 44, 22), (14, 10, 28, 14), (512, 4, 16, 8), (4, 512, 16, 8), (100, 38, 52, 34), (1000, 1, 40, 20)]


@pytest.mark.parametrize("op", OPS)
@pytest.mark.parametrize("n1,n2,nt,nz", BF16)
def test_bf16_grid_lengths(n1, n2, nt, nz, op):
    """Against the oracle: a grid value is off by up to 2^-9 of itself, 1.1e-3 in the
    mean square; R and its like sum 12 of them with one dominant, and 2.5e-3 leaves a
    margin of 2.  A wrong bin or root shows as 1e-2 and more."""
    g = geo(n1, n2, nt, nz)
    x = data(g, op, 3200 + n1)
    rel, _ = errors(getattr(plan_of(g, "bf16grid"), op)(torch.from_numpy(x).to(DEV, torch.float32)), getattr(recon, op)(x, g))
    print(f"  {op} {n1}x{n2}x{nt} -> {nz}: {rel:.2e}", flush=True)
    assert rel <= 2.5e-3, rel


# 578 = 2 17^2, 646 = 2 17 19, 722 = 2 19^2: no three radices of the general kernels' set
NO_PLAN = [(578, 2, 8, 4), (4, 646, 10, 6), (722, 1, 20, 10), (128, 578, 8, 4), (578, 24, 12, 6)]


@pytest.mark.parametrize("prec", ["f32", "f64"])
@pytest.mark.parametrize("op", OPS)
@pytest.mark.parametrize("n1,n2,nt,nz", NO_PLAN)
def test_lengths_without_a_general_plan(n1, n2, nt, nz, op, prec):
    g = geo(n1, n2, nt, nz)
    x = data(g, op, 3300 + n1)
    plan = plan_of(g, prec)
    rel, mx = errors(getattr(plan, op)(torch.from_numpy(x).to(DEV, plan.dtype)), getattr(recon, op)(x, g))
    print(f"  {op} {prec} {n1}x{n2}x{nt} -> {nz}: {rel:.2e}, max {mx:.2e}", flush=True)
    assert rel <= TOL[prec] and mx <= TOL[prec], (rel, mx)


@pytest.mark.parametrize("prec", ["f32", "f64"])
def test_batch_with_a_length_without_a_general_plan(prec):
    """A batch whose members have and lack a plan: one-tile kernels and general ones."""
    gs = [geo(578, 2, 8, 4), geo(24, 20, 48, 24), geo(4, 646, 10, 6), geo(16, 16, 32, 16)]
    plans = [plan_of(g, prec) for g in gs]
    xs = [data(g, "reconstruct", 3400 + i) for i, g in enumerate(gs)]
    outs, _ = pat.reconstruct_batched(plans, [torch.from_numpy(x).to(DEV, p.dtype) for x, p in zip(xs, plans)])
    for g, x, y in zip(gs, xs, outs):
        rel, mx = errors(y, recon.reconstruct(x, g))
        assert rel <= TOL[prec] and mx <= TOL[prec], (g, rel, mx)


@pytest.mark.parametrize("prec,nt", [("f32", 4096), ("f64", 2048)])
def test_arrays_past_4_gib(prec, nt):
    """512 x 512 detectors with spectra of 4.3e9 bytes, past the 32-bit offsets of the
    general and fixed-length kernels.  Separable inputs u(x1) v(x2) s(.): a line's
    values are u^ v^ times those of one line."""
    n1, n2, nz = 512, 512, 8
    g = geo(n1, n2, nt, nz)
    plan = plan_of(g, prec)
    rg = inputs.rng(3500)
    u, v = rg.standard_normal(n1), rg.standard_normal(n2)
    dev = lambda x: torch.from_numpy(x).to(DEV, plan.dtype)  # noqa: E731
    lines = [(0, 0), (1, 0), (0, 256), (256, 256), (256, 3), (255, -255), (17, 100), (200, -1)]
    hat = np.outer(np.fft.fft(u), np.fft.fft(v))
    l = recon.int_freqs(nz)

    def phases(a, b):
        return np.exp(-2j * np.pi * np.mod(np.outer(recon.nodes(a, b, l, g), np.arange(nt)), nt) / nt)

    s = rg.standard_normal(nt)
    f = plan.reconstruct(dev(u)[:, None, None] * (dev(v)[:, None] * dev(s)))
    F = torch.fft.fft2(f.double(), dim=(0, 1)).cpu().numpy()
    worst = 0.0
    for a, b in lines:
        def line(a, b):
            return np.fft.ifft(hat[a % n1, b % n2] * (phases(a, b) @ s) * recon.weights(a, b, l, g))
        exp = 0.5 * (line(a, b) + np.conj(line(-a, -b)))
        worst = max(worst, np.linalg.norm(F[a % n1, b % n2] - exp) / np.linalg.norm(exp))
    del f
    q = rg.standard_normal(nz)
    p = plan.reconstruct_adjoint(dev(u)[:, None, None] * (dev(v)[:, None] * dev(q)))
    ts = [0, 1, nt // 2 - 1, nt - 7, nt - 1]
    P = torch.fft.fft2(p[:, :, ts].double(), dim=(0, 1)).cpu().numpy()
    scale = 0.0
    off = 0.0
    for a, b in lines:
        def back(a, b):
            return hat[a % n1, b % n2] * ((np.fft.fft(q) * recon.weights(a, b, l, g)) @ np.conj(phases(a, b))) / nz
        exp = 0.5 * (back(a, b) + np.conj(back(-a, -b)))
        off = max(off, np.abs(P[a % n1, b % n2] - exp[ts]).max())
        scale = max(scale, np.abs(exp).max())
    print(f"  {prec} nt={nt}: R {worst:.2e}, R^T {off / scale:.2e}", flush=True)
    assert worst <= TOL[prec] and off <= TOL[prec] * scale, (worst, off / scale)
