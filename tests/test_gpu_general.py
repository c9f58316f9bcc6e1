"""The general-length kernels (transverse passes and fused line stages of
every length that is no power of two) against the oracle's direct sums.

The transverse lengths and depth lengths below make every radix from 2 to 23 a
last stage and every radix of the set a first or middle one; the time lengths
put the line kernels' own grid (the next 8 r1 rl >= 2 nt) at the smallest and
the largest point counts, just below and just above a step, and at every
middle radix.  FP32 1e-5 (the rounding of FFTs of at most 2^11 points and the
5e-8 weight fit, with a margin of 10), FP64 1e-9 (the window's truncation of
1e-11, with a margin)."""
import numpy as np
import pytest
import torch

from oracle import recon
from paper_0808_3510_amd import inputs, pat

pytestmark = pytest.mark.gpu
DEV = "cuda"
TOL = {"f32": 1e-5, "f64": 1e-9}
OPS = ["reconstruct", "reconstruct_adjoint", "forward", "forward_adjoint"]


def geo(n1, n2, nt, nz):
    return dict(n1=n1, n2=n2, nt=nt, nz=nz, dx=1.0, dt=0.9, dz=1.1, vs=1.05)


def run(op, g, prec, seed):
    n_in = g["nt"] if op in ("reconstruct", "forward_adjoint") else g["nz"]
    shape = (g["n1"], g["n2"], n_in) if g["n2"] > 1 else (g["n1"], n_in)
    x = inputs.random_array(shape, seed)
    plan = pat.Plan(g["n1"], g["n2"], g["nt"], g["nz"], g["dx"], g["dt"], g["dz"], g["vs"], precision=prec, device=DEV)
    y = getattr(plan, op)(torch.from_numpy(x).to(DEV, torch.float64 if prec == "f64" else torch.float32))
    torch.cuda.synchronize()
    got, exp = y.cpu().double().numpy(), getattr(recon, op)(x, g)
    rel = np.linalg.norm(got - exp) / np.linalg.norm(exp)
    mx = np.abs(got - exp).max() / np.abs(exp).max()
    print(f"  {op} {prec} {g}: relL2 {rel:.2e}, max {mx:.2e}", flush=True)
    assert rel <= TOL[prec] and mx <= TOL[prec], (rel, mx)


# (n1, n2, nt, nz): last radices of n1, n2 and nz over 2 .. 23, two and three
# stages, tiles with a remainder of one column pair
LENGTHS = [(2, 6, 30, 10), (14, 10, 26, 14), (22, 26, 44, 46), (46, 38, 34, 34), (34, 18, 50, 38), (12, 20, 70, 30),
           (36, 42, 66, 50), (110, 2, 60, 22), (4, 250, 36, 18), (2, 338, 18, 6), (242, 4, 20, 26), (144, 8, 36, 20),
           (6, 176, 36, 42), (4, 136, 68, 18), (152, 2, 36, 14), (2, 184, 72, 36), (1000, 2, 6, 10), (2, 1536, 10, 6),
           (54, 2, 20, 52), (2, 98, 20, 90), (182, 2, 18, 162), (2, 70, 18, 96), (130, 4, 10, 120), (312, 2, 6, 64),
           (416, 2, 6, 16), (420, 2, 6, 150), (196, 2, 6, 200), (384, 2, 6, 210), (306, 2, 6, 128), (374, 2, 6, 30),
           (672, 2, 6, 50)]


@pytest.mark.parametrize("prec", ["f32", "f64"])
@pytest.mark.parametrize("op", OPS)
@pytest.mark.parametrize("n1,n2,nt,nz", LENGTHS)
def test_transverse_and_depth_lengths(n1, n2, nt, nz, op, prec):
    run(op, geo(n1, n2, nt, nz), prec, 1200 + n1)


# (nt, nz): grids 8 r1 rl of 64 .. 1792 points, at, just below and just above a step
TIMES = [(6, 4), (32, 18), (34, 18), (40, 22), (48, 26), (60, 32), (72, 38), (100, 52), (128, 66), (150, 76),
         (208, 104), (256, 130), (300, 150), (440, 220), (500, 252), (640, 320), (770, 384), (896, 448), (900, 450)]


@pytest.mark.parametrize("op", OPS)
@pytest.mark.parametrize("n1,n2", [(6, 10), (10, 1)])
@pytest.mark.parametrize("nt,nz", TIMES)
def test_grid_lengths(nt, nz, n1, n2, op):
    run(op, geo(n1, n2, nt, nz), "f32", 1300 + nt)


@pytest.mark.parametrize("op", OPS)
@pytest.mark.parametrize("nt,nz", [(6, 2), (46, 138), (500, 126), (896, 448), (300, 300)])
def test_grid_lengths_fp64(nt, nz, op):
    """(Also nz > nt: depth lines longer than the grid's time lines.)"""
    run(op, geo(6, 6, nt, nz), "f64", 1400 + nt)


def test_nonfinite_values_stay_in_their_lines():
    """An infinite sample spoils what its transforms reach, as before, and no
    more: a batch neighbour keeps its values."""
    g = geo(10, 6, 40, 12)
    mk = lambda: pat.Plan(g["n1"], g["n2"], g["nt"], g["nz"], precision="f32", device=DEV)  # noqa: E731
    a, b = mk(), mk()
    x = torch.from_numpy(inputs.random_array((10, 6, 40), 1500)).to(DEV, torch.float32)
    y = x.clone()
    y[3, 2, 7] = float("inf")
    fa = a.reconstruct(x).clone()
    (o1, o2), _ = pat.reconstruct_batched([a, b], [x, y])
    assert torch.equal(o1, fa)
    assert not torch.isfinite(o2).all()


def test_batch_of_mixed_lengths_matches_single_calls():
    """Instances of different lengths in one launch: each equals its single
    call bit for bit (lengths that are no powers of two), whatever their
    order and number."""
    sizes = [(24, 20, 48, 24), (10, 6, 500, 36), (46, 38, 38, 34), (6, 4, 10, 6), (12, 1, 300, 90), (24, 20, 48, 24)]
    plans = [pat.Plan(a, b, t, z, precision="f32", device=DEV) for a, b, t, z in sizes]
    xs = [torch.from_numpy(inputs.random_array((a, b, t) if b > 1 else (a, t), 1600 + i)).to(DEV, torch.float32)
          for i, (a, b, t, z) in enumerate(sizes)]
    ref = [p.reconstruct(x).clone() for p, x in zip(plans, xs)]
    for order in ([0, 1, 2, 3, 4, 5], [4, 3, 0], [5, 1]):
        outs, _ = pat.reconstruct_batched([plans[i] for i in order], [xs[i] for i in order])
        for i, o in zip(order, outs):
            assert torch.equal(o, ref[i]), sizes[i]


# (n1, n2, nt, nz): transforms of 128, 256 and 512 points along each axis with
# rows x length just past the 32 columns per CU from which they run their
# compile-time kernels (over the time axis: R forward, A^T forward, R^T and A
# inverse), rows and lengths off the tile sizes
FIXED = [(128, 66, 130, 20), (256, 34, 250, 16), (512, 18, 462, 12), (66, 128, 132, 18), (30, 256, 270, 16),
         (14, 512, 600, 12), (128, 128, 66, 66), (256, 6, 1400, 6)]


@pytest.mark.parametrize("prec", ["f32", "f64"])
@pytest.mark.parametrize("op", OPS)
@pytest.mark.parametrize("n1,n2,nt,nz", FIXED)
def test_fixed_transverse_lengths(n1, n2, nt, nz, op, prec):
    run(op, geo(n1, n2, nt, nz), prec, 1700 + n1)


@pytest.mark.parametrize("lm", [8, 9, 10, 11])
@pytest.mark.parametrize("n2", [4, 8])
def test_bf16_interpolation_with_depth_fft_matches_staged(lm, n2):
    """R with the bf16 grid runs interpolation and depth FFT in one kernel for a
    single 3D plan with nz = m/4, and apart in a batch.  The grid's bits are the same up to
    values within an FP32 rounding (1e-7 with a margin of 10) of a tie, one in
    1e-6 / 2^-8 = 3e-4, that move by up to 2^-8: 7e-5 in relative L2.  A grid
    that is not rounded, or rounded elsewhere, differs by 1e-3."""
    g = geo(8, n2, 1 << (lm - 1), 1 << (lm - 2))
    plans = [pat.Plan(g["n1"], n2, g["nt"], g["nz"], g["dx"], g["dt"], g["dz"], g["vs"], precision="bf16grid",
                      device=DEV) for _ in range(2)]
    x = torch.from_numpy(inputs.random_array((8, n2, g["nt"]), 1800 + lm)).to(DEV, torch.float32)
    one = plans[0].reconstruct(x)
    (a, b), _ = pat.reconstruct_batched(plans, [x, x])
    torch.cuda.synchronize()
    assert torch.equal(a, b)
    rel = ((one - a).double().norm() / a.double().norm()).item()
    print(f"  m=2^{lm} n2={n2}: {rel:.2e}", flush=True)
    assert rel <= 7e-5, rel


# powers of two around the column counts up to which the passes of one small plan run
# the one-length kernels (4096; FP64 x2 of 64 points and less: 1024), at the tile's
# smallest sizes, and a length of two samples, which no pipeline takes
SHORT = [(128, 16, 256, 64), (128, 2, 8, 2), (256, 4, 8, 2), (64, 32, 128, 32), (64, 64, 128, 32), (32, 64, 64, 16),
         (512, 2, 16, 8), (4, 512, 8, 4), (2, 16, 1024, 8)]


@pytest.mark.parametrize("prec", ["f32", "f64"])
@pytest.mark.parametrize("op", OPS)
@pytest.mark.parametrize("n1,n2,nt,nz", SHORT)
def test_short_transverse_passes(n1, n2, nt, nz, op, prec):
    run(op, geo(n1, n2, nt, nz), prec, 1900 + n1)


# grids of 8 x 16 x 8, 10, 12 and 14 points (the middle radix with the longest powers)
# and of 8 x 8 x 14; the detectors' step is small, so that the nodes span more than
# five time windows and the type-1 stage runs the general kernel at any line count
@pytest.mark.parametrize("op", ["reconstruct", "reconstruct_adjoint"])
@pytest.mark.parametrize("nt,nz", [(840, 420), (760, 190), (552, 276), (476, 238), (396, 198)])
def test_fused_lines_are_as_exact_as_staged(nt, nz, op):
    """The fused line kernels' FP32 error against FP64 is no larger than that of the
    staged kernels, whose FFTs read every root from the table (both sums over
    10^5 samples: equal errors differ by a percent; 5 % allowed)."""
    n1, n2 = 12, 18
    n_in = nt if op == "reconstruct" else nz
    kw = dict(dx=1.0 / (1.3 * n1), dt=1.0, dz=nt / nz, vs=1.0, device=DEV)
    x = torch.from_numpy(inputs.random_array((n1, n2, n_in), 2000 + nt)).to(DEV, torch.float32)
    exp = getattr(pat.Plan(n1, n2, nt, nz, precision="f64", **kw), op)(x.double())
    plan = pat.Plan(n1, n2, nt, nz, precision="f32", **kw)
    err = []
    for fused in (True, False):
        plan.set_fused(fused)
        err.append(((getattr(plan, op)(x).double() - exp).norm() / exp.norm()).item())
    print(f"  {op} nt={nt} nz={nz}: fused {err[0]:.2e}, staged {err[1]:.2e}", flush=True)
    assert err[0] <= 1.05 * err[1], err


# powers of two without compile-time line kernels on both sides of the line counts at
# which the type-2 stage changes to the general kernel (FP32: m = 512 at 2304 lines,
# m = 32 at 24576; FP64: 5120 lines, 563200 points; 2D: 1536 lines)
TYPE2 = [(16, 256, 256, 64), (8, 512, 256, 64), (32, 512, 16, 8), (16, 512, 32, 16), (64, 64, 128, 32),
         (2048, 1, 128, 32), (4096, 1, 128, 32), (8, 4, 64, 64), (8, 1, 64, 32)]


@pytest.mark.parametrize("prec", ["f32", "f64"])
@pytest.mark.parametrize("op", ["reconstruct", "forward_adjoint"])
@pytest.mark.parametrize("n1,n2,nt,nz", TYPE2)
def test_type2_lines_of_powers_of_two(n1, n2, nt, nz, op, prec):
    run(op, geo(n1, n2, nt, nz), prec, 2200 + n1)


# grids of their own (m = 16, 32, 140, 600) and the plan's (64, 96, 1024), lines with and
# without a compile-time kernel, few lines and many
PAIRS = [(8, 8, 16, 8), (4, 2, 8, 4), (12, 20, 70, 18), (10, 1, 300, 150), (16, 1, 32, 16), (24, 20, 48, 24), (6, 4, 512, 128),
         (128, 34, 70, 36), (64, 66, 16, 8)]


@pytest.mark.parametrize("n1,n2,nt,nz", PAIRS)
def test_transposes_share_the_window_fp64(n1, n2, nt, nz):
    """Entries of R and A^T against those of R^T and A, from unit vectors: equal to
    rounding (1e-14 of the largest, with a margin of 20), where two windows differ by
    their truncation, some 1e-11.  Both operators of a pair take the same grid
    whichever kernels they run."""
    plan = pat.Plan(n1, n2, nt, nz, 1.0, 0.9, 1.1, 1.05, precision="f64", device=DEV)

    def unit(n, i):
        x = torch.zeros(n1 * n2 * n, dtype=torch.float64, device=DEV)
        x[i] = 1.0
        return x.reshape((n1, n2, n) if n2 > 1 else (n1, n))

    for fwd, adj in (("reconstruct", "reconstruct_adjoint"), ("forward_adjoint", "forward")):
        i = n1 * n2 * nt // 3
        y = getattr(plan, fwd)(unit(nt, i)).flatten()
        off = 0.0
        for j in y.abs().topk(4).indices.tolist() + [n1 * n2 * nz // 2 + 1]:
            off = max(off, abs(getattr(plan, adj)(unit(nz, j)).flatten()[i].item() - y[j].item()))
        off /= y.abs().max().item()
        print(f"  {fwd} {n1}x{n2}x{nt} -> {nz}: {off:.1e}", flush=True)
        assert off <= 2e-13, off


# type-1 lines whose nodes reach over nine time windows (a small detector step), which
# the general kernel takes at any number of lines: every length and grid above, and
# depth lines longer than the time lines
FAR = [(6, 10, nt, nz) for nt, nz in TIMES] + [(10, 1, nt, nz) for nt, nz in TIMES[::3]] + LENGTHS + \
      [(6, 6, 46, 64), (6, 6, 20, 30), (6, 6, 300, 300)]


@pytest.mark.parametrize("prec", ["f32", "f64"])
@pytest.mark.parametrize("op", ["reconstruct_adjoint", "forward"])
@pytest.mark.parametrize("n1,n2,nt,nz", FAR)
def test_type1_lines_of_far_nodes(n1, n2, nt, nz, op, prec):
    run(op, dict(geo(n1, n2, nt, nz), dx=0.05), prec, 2300 + n1 + nt)
