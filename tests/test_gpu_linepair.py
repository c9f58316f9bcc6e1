"""Type-1 line stages by mirror line pairs.  The fused ones of a 3D plan against the
oracle on sampled lines; stand-alone FP64 spreading (3D plans with at least eight
line pairs per CU) against the interpolation, line by line: with the same kernel
weights <N U, V> = <U, N^H V> on every line, up to the rounding of sums of
nz x 12 products (1e-13 of the norms' product, with a margin of 10)."""
import numpy as np
import pytest
import torch

from oracle import recon
from paper_0808_3510_amd import inputs, pat

pytestmark = pytest.mark.gpu
DEV = "cuda"


def complex_normal(shape, seed):
    gen = torch.Generator(device=DEV).manual_seed(seed)
    return torch.randn(shape, dtype=torch.complex128, device=DEV, generator=gen)


def check_adjoint(plan, seed):
    U, V = complex_normal((plan.lines, plan.m), seed), complex_normal((plan.lines, plan.nz), seed + 1)
    NU, W = plan.nufft2_lines(U), plan.nufft1_lines(V)
    torch.cuda.synchronize()
    a, b = (V.conj() * NU).sum(-1), (W.conj() * U).sum(-1)
    off = ((a - b).abs() / (V.norm(dim=-1) * NU.norm(dim=-1))).max().item()
    print(f"  {plan.n1}x{plan.n2}x{plan.nt} -> {plan.nz}: {off:.2e}", flush=True)
    assert off <= 1e-12, off


@pytest.mark.parametrize("n1,n2", [(64, 128), (512, 16)])
def test_coinciding_nodes_on_grid_points(n1, n2):
    """Nodes that coincide on a grid point each add their edge taps: with a depth
    step 2^30 times the others c nu is whole and the same for every l on the lines
    k2 = 0 and k1 = 0, and with alpha close to pi the window's edge is 1e-3 of its
    centre."""
    plan = pat.Plan(n1, n2, 32, 18, 32.0 / n1, 1.0, 2.0 ** 30, 1.0, alpha=3.2, precision="f64", device=DEV)
    check_adjoint(plan, 2100)


# more than 4.5 line pairs per CU (FP32) or 128 lines k2 (FP64): m = 512 and 1024
FUSED = [("f32", 64, 128, 256, 128), ("f32", 128, 64, 512, 256), ("f64", 8, 128, 256, 128), ("f64", 8, 128, 512, 256)]


@pytest.mark.parametrize("op", ["reconstruct_adjoint", "forward"])
@pytest.mark.parametrize("prec,n1,n2,nt,nz", FUSED)
def test_fused_pairs_match_oracle(prec, n1, n2, nt, nz, op):
    """The unshared pairs (k2 = 0 with n2/2), mirror pairs and the highest |K|; FP32
    1e-5, FP64 1e-9 (the window's truncation, with a margin)."""
    g = dict(n1=n1, n2=n2, nt=nt, nz=nz, dx=1.0, dt=0.9, dz=1.1, vs=1.05)
    x = inputs.random_array((n1, n2, nz), 2600 + n1)
    plan = pat.Plan(n1, n2, nt, nz, g["dx"], g["dt"], g["dz"], g["vs"], precision=prec, device=DEV)
    y = getattr(plan, op)(torch.from_numpy(x).to(DEV, plan.dtype))
    torch.cuda.synchronize()
    Y = np.fft.fft2(y.cpu().double().numpy(), axes=(0, 1))
    lines = [(0, 0), (0, n2 // 2), (1, 0), (n1 // 2, 0), (n1 // 2, n2 // 2), (2, 1), (2, -1), (n1 // 2 - 1, n2 // 2 - 1),
             (n1 // 2 - 1, 1 - n2 // 2), (1, n2 // 4)]
    oracle = recon.adjoint_lines if op == "reconstruct_adjoint" else recon.forward_lines
    X = oracle(x, g, lines)
    Xm = oracle(x, g, [(-a, -b) for a, b in lines])
    worst = 0.0
    for i, (a, b) in enumerate(lines):
        exp = 0.5 * (X[i] + np.conj(Xm[i]))
        worst = max(worst, np.linalg.norm(Y[a % n1, b % n2] - exp) / np.linalg.norm(exp))
    print(f"  {op} {prec} {g}: {worst:.2e}", flush=True)
    assert worst <= {"f32": 1e-5, "f64": 1e-9}[prec], worst


# 2048 line pairs and more (4096 with several batches): depth lines of one batch, of a
# batch and one node, of two turns with a ragged last one, grids that are no power of
# two, the longest grid line that fits, and other windows of 12 taps
SPREAD = [(128, 66, 32, 18, 2.0, 3.0), (128, 128, 260, 130, 2.0, 3.0), (256, 34, 540, 540, 2.0, 3.0), (256, 34, 22, 10, 2.0, 3.0),
          (128, 66, 1260, 16, 2.0, 3.0), (64, 128, 128, 128, 2.0, 3.0), (128, 66, 40, 30, 3.0, 2.0), (128, 66, 48, 2, 1.5, 4.0)]


@pytest.mark.parametrize("n1,n2,nt,nz,c,K", SPREAD)
def test_spreading_by_pairs_is_adjoint_of_interpolation(n1, n2, nt, nz, c, K):
    plan = pat.Plan(n1, n2, nt, nz, 1.0, 0.9, 1.1, 1.05, c=c, K=K, precision="f64", device=DEV)
    check_adjoint(plan, 2700 + nz)


@pytest.mark.parametrize("op", ["reconstruct_adjoint", "forward"])
@pytest.mark.parametrize("n1,n2,nt,nz", [(128, 66, 32, 18), (128, 128, 260, 130), (256, 34, 540, 540)])
def test_staged_pairs_match_fused_fp64(n1, n2, nt, nz, op):
    """The staged operators spread by pairs (A with its node l = 0 in a turn of its
    own), the fused ones do not: equal up to the windows' truncation (1e-11, with a
    margin of 100)."""
    plan = pat.Plan(n1, n2, nt, nz, 1.0, 0.9, 1.1, 1.05, precision="f64", device=DEV)
    x = torch.from_numpy(inputs.random_array((n1, n2, nz), 2800 + nz)).to(DEV)
    a = getattr(plan, op)(x).clone()
    plan.set_fused(False)
    b = getattr(plan, op)(x)
    rel = ((a - b).norm() / b.norm()).item()
    mx = ((a - b).abs().max() / b.abs().max()).item()
    print(f"  {op} {n1}x{n2}x{nt} -> {nz}: relL2 {rel:.1e}, max {mx:.1e}", flush=True)
    assert rel <= 1e-9 and mx <= 1e-9, (rel, mx)
