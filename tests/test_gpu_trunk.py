"""GPU parity of the one-launch trunk evaluation (csrc/trunk.hip) at the edges
of its blocks, widths and activations, and of its tanh."""
import numpy as np
import pytest

from paper_2405_12380_amd import inputs as I
from oracle import deeponet as don_or
from tests.helpers import make_op, rel_err, stored_layers, to_np

pytestmark = pytest.mark.gpu

helm = pytest.importorskip("paper_2405_12380_amd.helm")


def build(n, dtype, trunk, act="tanh"):
    dim = len(n)
    p = trunk[-1][0].shape[1]
    bg = (4,) * dim
    branch = I.glorot_mlp([2 * 4 ** dim, 16, 2 * p], np.random.default_rng(2))
    op = make_op(helm, I.random_problem(n, 3), dtype)
    return op, helm.DeepONet(dtype, branch, trunk, p, head="split_output", act=act, branch_grid=bg)


@pytest.mark.parametrize("n,widths,act,dtype", [
    ((3, 3, 3), [3, 32, 16], "tanh", helm.C128),              # one partial 16-row block, one column tile
    ((5, 17, 3), [3, 64, 96, 48], "relu", helm.C128),         # 255 rows; wavefronts without columns
    ((31, 33, 8), [3, 160, 32, 112], "leaky", helm.C128),     # 8184 rows: the largest 16-row grids
    ((32, 33, 8), [3, 256, 224, 128], "tanh", helm.C128),     # 8448 rows: 32-row blocks; 14 of 16 tiles
    ((101, 83), [2, 128, 256, 256, 64], "tanh", helm.C64),    # 2D, 8383 rows: a partial last block
    ((21, 20, 21), [3, 32, 128, 128], "tanh", helm.C64),
    ((7, 9, 11), [3, 32] + [64] * 6 + [128], "tanh", helm.C128),  # the most layers the launch takes
])
def test_trunk_blocks(n, widths, act, dtype):
    g = np.random.default_rng(sum(widths))
    trunk = [(W, g.standard_normal(W.shape[1]) * 0.1) for W, _ in I.glorot_mlp(widths, g, first_gain=3.0)]
    op, net = build(n, dtype, trunk, act)
    T = to_np(net.trunk(op)).reshape(-1, widths[-1])
    ref = don_or.trunk_matrix(I.node_points(n), stored_layers(trunk, dtype == helm.C64), act)
    # sums of at most 256 products per layer in another order, at most 8 layers:
    # 8 * 256 * 1.1e-16 = 2.3e-13 bounds the fp64 error; C64 rounds T once (6e-8)
    assert rel_err(T, ref) <= (2.5e-13 if dtype == helm.C128 else 1e-7)


def test_trunk_tanh():
    """tanh alone: columns of T are tanh(2^e x) (exact arguments, a selecting
    last layer), from the linear range to saturation, both signs."""
    n = (63, 31, 7)
    e = np.concatenate([np.arange(-28, 8, 2.0), [-40.0, -60.0]])
    W0 = np.zeros((3, 64))
    b0 = np.zeros(64)
    for j, k in enumerate(e):
        W0[0, j], W0[0, 32 + j] = 2.0 ** k, -2.0 ** k
    b0[31] = np.nan
    W1 = np.eye(64)
    W1[31, :] = 0.0  # 0 * NaN = NaN: column sums that include it are NaN
    op, net = build(n, helm.C128, [(W0, b0), (W1, np.zeros(64))])
    T = to_np(net.trunk(op)).reshape(-1, 64)
    assert np.isnan(T).all()
    b0[31] = 0.0
    op, net = build(n, helm.C128, [(W0, b0), (W1, np.zeros(64))])
    T = to_np(net.trunk(op)).reshape(-1, 64)
    x = I.node_points(n).astype(np.longdouble)[:, :1] @ W0[:1].astype(np.longdouble)
    ref = np.tanh(x)
    on = np.abs(ref) > 0
    err = np.abs(T[on] - ref[on]) / np.abs(ref[on])
    # e^r - 1, its scaling, the quotient: at most about three roundings of half an ulp each, doubled
    assert float(err.max()) <= 6 * 1.11e-16
    assert np.all(T[~on] == 0)
