"""Stand-alone FP64 spreading by mirror line pairs (3D plans with at least eight
line pairs per CU) against the interpolation, line by line: with the same kernel
weights <N U, V> = <U, N^H V> on every line, up to the rounding of sums of
nz x 12 products (1e-13 of the norms' product, with a margin of 10)."""
import pytest
import torch

from paper_0808_3510_amd import pat

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
