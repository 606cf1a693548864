"""The batched solve's basis products at the edges of their lane groups, load
forms and workgroup counts, against the single solves."""
import numpy as np
import pytest

from paper_2405_12380_amd import inputs as I
from tests.helpers import make_op, rel_err, to_np

pytestmark = pytest.mark.gpu

helm = pytest.importorskip("paper_2405_12380_amd.helm")


@pytest.mark.parametrize("p,dtype,q32", [
    (1, helm.C128, False), (16, helm.C128, False), (17, helm.C128, False), (32, helm.C128, False),
    (33, helm.C128, False), (34, helm.C128, False), (65, helm.C128, False), (128, helm.C128, False),
    (30, helm.C128, True), (64, helm.C128, True), (3, helm.C64, False), (36, helm.C64, False), (128, helm.C64, False)])
def test_batch_columns(p, dtype, q32):
    sizes = [(7, 6, 5), (24, 23, 31), (12, 30, 11)]
    Ps = [I.random_problem(n, 40 + i, k=6.0) for i, n in enumerate(sizes)]
    g = np.random.default_rng(p)
    net = helm.DeepONet(dtype, I.glorot_mlp([2 * 4 ** 3, 16, 2 * 128], g),
                        I.glorot_mlp([3, 160, 128], g, first_gain=20.0), 128, head="split_output",
                        branch_grid=(4, 4, 4))
    ops = [make_op(helm, P, dtype) for P in Ps]
    fs = [op.field(P["f"]) for op, P in zip(ops, Ps)]
    us = [op.field() for op in ops]
    kw = dict(tol=0.0, max_iters=2, n_r=2, omega=0.5, p_used=p, q_fp32=q32)
    helm.meta_solve_batch(ops, net, fs, us, **kw)
    for op, f, u in zip(ops, fs, us):
        u1 = op.field()
        helm.meta_solve(op, net, f, u1, kind="bicgstab", **kw)
        # the same steps with sums over other partitions of the rows
        assert rel_err(to_np(u), to_np(u1)) <= (1e-10 if dtype == helm.C128 else 2e-5)
