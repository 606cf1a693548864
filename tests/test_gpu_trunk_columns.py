"""The trunk matrix entry by entry against 80-bit arithmetic: every entry to the
error that fp64 sums of its own terms have, also where the activations that a
column selects are far smaller than others of their node, or its weights far
smaller than others of their column."""
import numpy as np
import pytest

from paper_2405_12380_amd import inputs as I
from tests.helpers import make_op, stored_layers, to_np

pytestmark = pytest.mark.gpu

helm = pytest.importorskip("paper_2405_12380_amd.helm")

U = 2.0 ** -53


def check(n, dtype, trunk):
    """max over the entries of error / bound; the bound is that of fp64 layers."""
    dim, p = len(n), trunk[-1][0].shape[1]
    branch = I.glorot_mlp([2 * 4 ** dim, 16, 2 * p], np.random.default_rng(2))
    op = make_op(helm, I.random_problem(n, 3), dtype)
    net = helm.DeepONet(dtype, branch, trunk, p, head="split_output", branch_grid=(4,) * dim)
    T = to_np(net.trunk(op)).reshape(-1, p)
    rows = np.unique(np.r_[0:64, np.linspace(0, T.shape[0] - 1, 200).astype(int), T.shape[0] - 40:T.shape[0]])
    h = I.node_points(n)[rows].astype(np.longdouble)
    e = U * h  # a coordinate is one division
    layers = stored_layers(trunk, dtype == helm.C64)
    for l, (W, b) in enumerate(layers):
        # K products and sums of at most one rounding each, the bias, and the error of the inputs
        S = h.__abs__() @ np.abs(W) + np.abs(b)
        e = e @ np.abs(W) + (W.shape[0] + 1) * U * S
        h = h @ W.astype(np.longdouble) + b.astype(np.longdouble)
        if l + 1 < len(layers):
            # |tanh'| <= 1, and tanh within 4 units in the last place
            h = np.tanh(h)
            e = e + 8 * U * np.abs(h)
    if dtype == helm.C64:
        e = e + 2.0 ** -24 * np.abs(h)
    assert np.isfinite(T).all()
    return float(np.max(np.abs(T[rows] - h) / e))


N_SMALL, N_LARGE = (15, 17, 13), (17, 16, 16)  # 3315 and 4352 nodes


@pytest.mark.parametrize("n", [N_SMALL, N_LARGE])
@pytest.mark.parametrize("dtype", [helm.C128, helm.C64])
@pytest.mark.parametrize("K,count", [(64, 1), (64, 4), (256, 16), (256, 32)])
def test_columns_of_small_features(n, dtype, K, count):
    """Columns of equal weights on `count` features whose values are 1e-12 of the others'."""
    g = np.random.default_rng(K + count)
    (W0, b0), (W1, b1) = I.glorot_mlp([3, K, 32], g, first_gain=3.0)
    W0, W1 = W0.copy(), W1.copy()
    sel = g.permutation(K)[:count]
    W0[:, sel] *= 1e-12
    W1[:, [3, 30]] = 0.0
    W1[np.ix_(sel, [3, 30])] = 0.25
    assert check(n, dtype, [(W0, b0), (W1, b1)]) <= 1.0


@pytest.mark.parametrize("n", [N_SMALL, N_LARGE])
@pytest.mark.parametrize("size", [1e-2, 1e-4, 1e-6])
def test_saturated_unit_without_weights(n, size):
    """One unit near 1 with no outgoing weights, the others of the given size."""
    g = np.random.default_rng(7)
    K = 64
    (W0, b0), (W1, b1), (W2, b2) = I.glorot_mlp([3, K, K, 48], g, first_gain=1.0)
    W0, b0, W1 = W0 * size, b0.copy(), W1.copy()
    W0[:, 5], b0[5] = 0.0, 9.0
    W1[5, :] = 0.0
    assert check(n, helm.C128, [(W0, b0), (W1, b1), (W2, b2)]) <= 1.0


@pytest.mark.parametrize("n,widths,gain", [
    ((17, 241), [2, 32, 16], 3.0),
    ((17, 16, 16), [3, 64, 96, 48], 20.0),
    ((31, 33, 8), [3, 160, 32, 112], 3.0),
    ((101, 83), [2, 128, 256, 256, 64], 3.0),
    ((23, 19, 11), [3, 32] + [64] * 6 + [128], 3.0),
])
def test_every_entry(n, widths, gain):
    """Columns of scales 1e-3 .. 1, one with a bias beside small sums."""
    g = np.random.default_rng(sum(widths))
    trunk = I.glorot_mlp(widths, g, first_gain=gain)
    trunk = [(W * 10.0 ** g.integers(-3, 1, W.shape[1]) if l else W, 0.1 * g.standard_normal(W.shape[1]))
             for l, (W, _) in enumerate(trunk)]
    assert check(n, helm.C128, trunk) <= 1.0
