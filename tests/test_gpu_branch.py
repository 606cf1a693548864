"""GPU parity of the network correction's two-launch branch (csrc/deeponet.hip)
at the edges of its chunks and column blocks, both heads, against the oracle."""
import numpy as np
import pytest

from paper_2405_12380_amd import inputs as I
from oracle import deeponet as don_or
from tests.helpers import make_op, rel_err, stored, stored_layers, to_np

pytestmark = pytest.mark.gpu

helm = pytest.importorskip("paper_2405_12380_amd.helm")


@pytest.mark.parametrize("head,bg,hidden,act,dtype", [
    ("split_output", (3, 3, 3), [], "tanh", helm.C128),                  # one layer: no tail product; K = 55 < 64
    ("split_output", (4, 4, 4), [7], "relu", helm.C128),                 # K = 129; fewer inputs than a k chunk
    ("split_output", (5, 4, 3), [257, 19, 64], "tanh", helm.C64),        # a second column block of one column
    ("split_output", (4, 5, 4), [1024, 48], "leaky", helm.C128),         # the widest layer of the tail
    ("split_output", (4, 5, 4), [1030, 48], "tanh", helm.C128),          # wider: layer by layer
    ("split_output", (4, 4, 4), [1000, 1000], "tanh", helm.C128),        # 8 MB of weights: layer by layer
    ("split_input", (8, 8, 8), [31, 16, 100], "tanh", helm.C64),
    ("split_input", (9, 11, 7), [300, 300], "tanh", helm.C128),          # the op's own grid, K = 693
])
def test_branch_shapes(head, bg, hidden, act, dtype):
    n, p = (9, 11, 7), 24
    g = np.random.default_rng(len(hidden) + 17 * bg[0])
    m = int(np.prod(bg))
    so = head == "split_output"
    widths = [2 * m + 1 if so else m] + hidden + [2 * p if so else p]
    branch = [(W, g.standard_normal(W.shape[1]) * 0.1) for W, _ in I.glorot_mlp(widths, g)]
    trunk = I.glorot_mlp([3, 32, p], g, first_gain=5.0)
    P = I.random_problem(n, 12, mask_frac=0.1)
    lo = dtype == helm.C64
    op = make_op(helm, P, dtype)
    net = helm.DeepONet(dtype, branch, trunk, p, head=head, act=act, branch_grid=bg, k_input=so)
    r = stored(P["x"] * 2.5, lo)
    du = to_np(net.full(op, op.field(r), k=7.5))
    T = don_or.trunk_matrix(I.node_points(n), stored_layers(trunk, lo), act)
    ref = don_or.infer(r, P["mask"], T, stored_layers(branch, lo), head, p, bg, k=7.5, k_input=so, act=act)
    # fp64 sums of up to 1030 products per layer: 1e-12; C64 rounds the input, every layer's output and du to fp32
    assert rel_err(du, ref) <= (1e-12 if not lo else 1e-6)
    assert np.all(du[P["mask"].ravel().astype(bool)] == 0)
