"""GPU parity of the restriction and prolongation (csrc/coarse_dev.h) at the
edges of their lane groups, row groups and load forms, through the Krylov
preconditioner and the network synthesis."""
import numpy as np
import pytest

from paper_2405_12380_amd import inputs as I
from oracle import coarse as co_or, deeponet as don_or, meta as meta_or, operator as op_or
from tests.helpers import make_op, rel_err, stored, stored_layers, to_np

pytestmark = pytest.mark.gpu

helm = pytest.importorskip("paper_2405_12380_amd.helm")


def setup(n, dtype, p, small_trunk):
    lo = dtype == helm.C64
    C = I.config2(0, n=n)
    g = np.random.default_rng(p)
    trunk = I.glorot_mlp([3, 64, p], g, first_gain=20.0) if small_trunk else C["trunk"]
    pn = trunk[-1][0].shape[1]
    branch = I.glorot_mlp([2 * 4 ** 3 + 1, 16, 2 * pn], g)
    op = make_op(helm, C, dtype)
    net = helm.DeepONet(dtype, branch, trunk, pn, head="split_output", branch_grid=(4, 4, 4), k_input=True)
    T = don_or.trunk_matrix(I.node_points(n), stored_layers(trunk, lo))
    s = stored(op_or.coefficient(C["ksq"], C["alpha"]), lo)
    r = stored(g.standard_normal(C["f"].shape) + 1j * g.standard_normal(C["f"].shape), lo)
    r[C["mask"].astype(bool)] = 0
    return C, op, net, branch, T, s, r, lo


@pytest.mark.parametrize("n", [(13, 11, 9), (24, 23, 31)])  # fewer groups than wavefronts; several per wavefront
@pytest.mark.parametrize("p,dtype,q32", [
    (1, helm.C128, False), (2, helm.C128, False), (15, helm.C128, False), (16, helm.C128, False),
    (18, helm.C128, False), (34, helm.C128, False), (65, helm.C128, False), (66, helm.C128, False),
    (3, helm.C128, True), (32, helm.C128, True), (36, helm.C128, True), (68, helm.C128, True),
    (4, helm.C64, False), (33, helm.C64, False), (64, helm.C64, False)])
def test_precond_columns(n, p, dtype, q32):
    C, op, net, _, T, s, r, lo = setup(n, dtype, p, False)
    cs = co_or.CoarseSpace(T, s, C["mask"], p, tau=co_or.TAU_C64 if lo else co_or.TAU_C128,
                           q_round="f32" if lo or q32 else None)
    z = to_np(helm.meta_precond(op, net, op.field(r), p_used=p, n_r=2, omega=0.5, q_fp32=q32))
    ref = meta_or.krylov_preconditioner(s, C["mask"], "jacobi", 2, 0.5, cs)(r.ravel())
    # as the preconditioner tests at p = 64; an fp32 basis is rounded from a Q known to 1e-9 (last bits flip)
    assert rel_err(z, ref) <= (2e-5 if lo else 1e-7 if q32 else 1e-10)


@pytest.mark.parametrize("p,dtype", [(1, helm.C128), (17, helm.C128), (50, helm.C128), (7, helm.C64), (20, helm.C64),
                                     (100, helm.C64)])
def test_synthesis_columns(p, dtype):
    n = (13, 11, 9)
    C, op, net, branch, T, s, r, lo = setup(n, dtype, p, True)
    du = to_np(net.full(op, op.field(r), k=3.0))
    ref = don_or.infer(r, C["mask"], T, stored_layers(branch, lo), "split_output", p, (4, 4, 4), k=3.0,
                       k_input=True)
    assert rel_err(du, ref) <= (1e-12 if not lo else 1e-6)
    assert np.all(du[C["mask"].ravel().astype(bool)] == 0)
