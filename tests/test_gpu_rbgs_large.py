"""The red-black ring kernel's march length on large grids: the values of the
register-pair kernel bit for bit."""
import pytest
import torch

pytestmark = pytest.mark.gpu

helm = pytest.importorskip("paper_2405_12380_amd.helm")


@pytest.mark.parametrize("n", [(448, 400, 469), (448, 400, 468)])  # both sides of five rounds of 64-plane marches
def test_large_marches_equal_pairs(n):
    N = n[0] * n[1] * n[2]
    g = torch.Generator(device="cuda")
    g.manual_seed(3)
    rnd = lambda: torch.view_as_complex(torch.randn(N, 2, generator=g, device="cuda"))  # noqa: E731
    mask = (torch.rand(N, generator=g, device="cuda") < 0.05).to(torch.uint8)
    op = helm.Op(n, helm.C64, torch.full((N,), 36.0, dtype=torch.float64, device="cuda"),
                 torch.full((N,), 0.05, dtype=torch.float64, device="cuda"), mask)
    f, u0 = rnd(), rnd()
    out = []
    for which in (helm.RB_PAIRS, helm.RB_RING):
        op.set_rbgs_kernel(which)
        u = u0.clone()
        op.relax(helm.RBGS, 0.9, 1, f, u)
        out.append(u)
    assert torch.equal(torch.view_as_real(out[0]), torch.view_as_real(out[1]))
    op.close()
