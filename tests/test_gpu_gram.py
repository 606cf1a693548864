"""GPU parity of the set-up's symmetric Gram products (csrc/gram.hip) at the
edges of their column tiles, row steps and blocks, through the coarse matrix
and its basis."""
import numpy as np
import pytest

from paper_2405_12380_amd import inputs as I
from oracle import deeponet as don_or, coarse as co_or, operator as op_or
from tests.helpers import make_op, rel_err, to_np

pytestmark = pytest.mark.gpu

helm = pytest.importorskip("paper_2405_12380_amd.helm")


@pytest.mark.parametrize("n,p", [
    ((5, 5, 5), 1), ((5, 5, 5), 16), ((6, 7, 3), 17),             # few blocks, steps that not every share has
    ((24, 23, 31), 15), ((24, 23, 31), 64), ((24, 23, 31), 65),   # 256 blocks; the two tile grids
    ((13, 11, 9), 112), ((24, 23, 31), 113), ((24, 23, 31), 128),
    ((92, 95), 33),                                               # 2D; a last block of fewer rows
])
def test_gram_columns(n, p):
    C = I.random_problem(n, 11)
    g = np.random.default_rng(p)
    dim = len(n)
    trunk = I.glorot_mlp([dim, 160, p], g, first_gain=20.0)
    op = make_op(helm, C, helm.C128)
    net = helm.DeepONet(helm.C128, I.glorot_mlp([2 * 4 ** dim, 16, 2 * p], g), trunk, p, head="split_output",
                        branch_grid=(4,) * dim)
    s = op_or.coefficient(C["ksq"], C["alpha"])
    cs = co_or.CoarseSpace(don_or.trunk_matrix(I.node_points(n), trunk), s, C["mask"], p)
    r, Ac, Q = helm.coarse_info(op, net, p_used=p, want_q=True)
    Q = to_np(Q).reshape(-1, r)
    assert r == cs.rank
    # orthonormal and spanning the oracle's space (CholeskyQR2: a few eps of n sums)
    assert np.abs(Q.T @ Q - np.eye(r)).max() <= 1e-12
    assert rel_err(cs.Q @ (cs.Q.T @ Q), Q) <= 1e-8
    AQ = np.stack([op_or.apply(Q[:, j].reshape(np.shape(s)).astype(complex), s, C["mask"]).ravel() for j in range(r)], 1)
    # the Galerkin matrix of that basis: A_c = S^T (Q1^T A Q1) S with an inexact Q1 S
    assert rel_err(Ac, Q.T @ AQ) <= 1e-10
