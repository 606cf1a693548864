"""GPU parity of the training step's trunk backward and output kernels
(csrc/train.hip) over their batch, output and layer-width forms, against the
oracle's backpropagation with the same bf16 operand rounding (tolerances as in
test_gpu_train)."""
import numpy as np
import pytest
import torch

from paper_2405_12380_amd import inputs as I
from oracle import training as T
from tests.helpers import rel_err, to_np

pytestmark = pytest.mark.gpu

helm = pytest.importorskip("paper_2405_12380_amd.helm")


@pytest.mark.parametrize("npts,batch,trunk_w", [
    ((4, 4, 4), 64, [64, 64]),                 # one 64-point block
    ((8, 8, 8), 128, [192, 128]),
    ((16, 12, 12), 64, [256, 64, 128]),
    ((16, 20, 14), 128, [128, 256, 64]),
    ((28, 28, 28), 64, [256, 192, 128]),       # more blocks than workgroups: 343 of 64 points
    ((28, 28, 28), 128, [64, 256, 128]),
    ((4, 8, 4), 64, [64] * 7 + [64]),          # the most trunk layers
])
def test_grad_shapes(npts, batch, trunk_w):
    p = trunk_w[-1]
    g = np.random.default_rng(sum(npts) + batch + p)
    f32 = lambda L: [(W.astype(np.float32).astype(np.float64), (0.1 * g.standard_normal(b.shape)).astype(
        np.float32).astype(np.float64)) for W, b in L]
    branch = f32(I.glorot_mlp([129, 64, 2 * p], g))
    trunk = f32(I.glorot_mlp([3] + trunk_w, g, first_gain=4.0))
    X = I.node_points(npts)
    n = 2 * batch
    F = g.standard_normal((n, 129)).astype(np.float32)
    Y = (g.standard_normal((n, X.shape[0])) + 1j * g.standard_normal((n, X.shape[0]))).astype(np.complex64)
    net = helm.DeepONet(helm.C128, branch, trunk, p, head="split_output", branch_grid=(4, 4, 4), k_input=True)
    tr = helm.Trainer(net, X, batch=batch, max_steps=2)
    tr.data(torch.as_tensor(F).cuda(), torch.as_tensor(Y).cuda())
    idx = g.permutation(n)[:batch]
    loss, grads = tr.grad(idx)
    L_or, gb, gt, _ = T.loss_and_grads(F[idx].astype(np.float64), X, Y[idx].T.astype(np.complex128), branch, trunk,
                                       rnd=T.bf16)
    assert abs(loss - L_or) <= 1e-3 * L_or
    got = tr.unflatten(grads, 0, len(branch)) + tr.unflatten(grads, 1, len(trunk))
    for (dW, db), (eW, eb) in zip(got, gb + gt):
        assert rel_err(dW, eW) <= 5e-3
        assert rel_err(db, eb) <= 5e-3
    # a second pass gives the same bits
    loss2, grads2 = tr.grad(idx)
    assert loss2 == loss and np.array_equal(to_np(grads2), to_np(grads))
