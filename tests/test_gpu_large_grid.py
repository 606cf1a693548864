"""The trunk matrix and the coarse set-up on a grid of more than 2^28 nodes: one
launch over all nodes has more than 2^32 work-items if a block of 32 nodes takes
512 of them along one axis."""
import numpy as np
import pytest
import torch

from paper_2405_12380_amd import inputs as I
from tests.helpers import stored_layers

pytestmark = pytest.mark.gpu

helm = pytest.importorskip("paper_2405_12380_amd.helm")


def test_setup_beyond_2_28_nodes():
    n, p = (16385, 16387), 16
    N = n[0] * n[1]
    assert N > 2 ** 28
    ksq = torch.full((N,), 81.0, dtype=torch.float64, device="cuda")
    alpha = torch.full((N,), 0.05, dtype=torch.float64, device="cuda")
    mask = torch.zeros(N, dtype=torch.uint8, device="cuda")
    holes = torch.tensor([0, 77, 2 ** 27 + 5, N - 1], device="cuda")
    mask[holes] = 1
    op = helm.Op(n, helm.C64, ksq, alpha, mask)
    del ksq, alpha, mask
    g = np.random.default_rng(4)
    trunk = I.glorot_mlp([2, 32, p], g, first_gain=10.0)
    net = helm.DeepONet(helm.C64, I.glorot_mlp([32, 16, 2 * p], g), trunk, p, head="split_output", branch_grid=(4, 4))
    T = net.trunk(op).reshape(-1, p)
    rows = np.unique(np.r_[0:50, np.linspace(0, N - 1, 400).astype(int), 2 ** 28 - 40:2 ** 28 + 40, N - 50:N])
    (W0, b0), (W1, b1) = stored_layers(trunk, True)
    x = np.stack([(rows % n[0] + 1) / (n[0] + 1), (rows // n[0] + 1) / (n[1] + 1)], axis=1)
    ref = np.tanh(x @ W0 + b0) @ W1 + b1
    got = T[torch.as_tensor(rows, device="cuda")].cpu().numpy()
    # rounded once to fp32, beside fp64 errors of the sums
    assert np.all(np.abs(got - ref) <= 2.0 ** -24 * np.abs(ref) + 1e-13)
    del T
    r, A, Q = helm.coarse_info(op, net, p_used=p, want_q=True)
    assert r == p
    Q = Q.reshape(N, p)
    assert torch.all(Q[holes] == 0)
    G = torch.zeros(p, p, dtype=torch.float64, device="cuda")
    for c in torch.chunk(Q, 64):
        G += c.double().T @ c.double()
    # every entry of Q rounded once to fp32
    assert float((G - torch.eye(p, device="cuda")).abs().max()) <= 1e-6
    for j in (0, p - 1):
        y = op.apply(Q[:, j].to(torch.complex64).contiguous())
        a = torch.zeros(p, dtype=torch.complex128, device="cuda")
        for c, v in zip(torch.chunk(Q, 64), torch.chunk(y, 64)):
            a += torch.complex(c.double().T @ v.real.double(), c.double().T @ v.imag.double())
        # A Q rounded to complex64: 2^-24 of its norm, for columns of norm 1
        assert float((a - torch.as_tensor(A[:, j], device="cuda")).abs().max()) <= 2.0 ** -23 * float(y.norm())
    op.close()
