"""Several Jacobi sweeps per launch (csrc/relax.hip): the same values, bit for
bit, as single sweeps, at the edges of the tiles and marches, and against the
oracle."""
import numpy as np
import pytest

from paper_2405_12380_amd import inputs as I
from oracle import operator as op_or
from tests.helpers import make_op, rel_err, stored, to_np

pytestmark = pytest.mark.gpu

helm = pytest.importorskip("paper_2405_12380_amd.helm")


@pytest.mark.parametrize("dtype", [helm.C128, helm.C64])
@pytest.mark.parametrize("n,sweeps", [
    ((3, 3), 7), ((32, 32), 1), ((32, 31), 1030),        # one workgroup; more sweeps than one launch takes
    ((33, 32), 2), ((32, 65), 17), ((90, 33), 16),       # a rim on one axis only; 1 .. 8 sweeps a launch
    ((131, 77), 33), ((513, 40), 3),
    ((120, 96, 70), 3), ((119, 95, 71), 4), ((61, 133, 111), 5),  # pairs; ragged tiles and marches
    ((180, 96, 47), 6), ((240, 13, 300), 7),             # an odd number of pairs; a tile of one row
    ((256, 252, 66), 2),                                 # one pair and the copy (4 Mi nodes)
])
def test_sweeps_equal_single_sweeps(n, sweeps, dtype):
    P = I.random_problem(n, sum(n), mask_frac=0.08, k=6.0)
    lo = dtype == helm.C64
    op = make_op(helm, P, dtype)
    f = op.field(P["f"])
    u0 = stored(P["x"], lo)
    a, b, c = op.field(u0), op.field(u0), op.field(u0)
    op.relax(helm.JACOBI, 0.6, sweeps, f, a)
    for _ in range(sweeps):
        op.relax(helm.JACOBI, 0.6, 1, f, b)
    assert np.array_equal(to_np(a), to_np(b))
    if a.numel() * a.element_size() <= 64 << 20:
        op.relax_noalloc(helm.JACOBI, 0.6, sweeps, f, c)
        assert np.array_equal(to_np(a), to_np(c))
    if sweeps <= 7:
        s, fr, ref = stored(op_or.coefficient(P["ksq"], P["alpha"]), lo), stored(P["f"], lo), u0
        for _ in range(sweeps):
            ref = stored(op_or.jacobi_sweep(ref, fr, s, P["mask"], 0.6), lo)
        # a sweep's update is a few roundings of values of order 1
        assert rel_err(to_np(a), ref) <= (1e-13 if not lo else 1e-6)


def test_masked_and_nonfinite_values_stay_apart():
    """A scatterer node's own value (here NaN and Inf) is absent to its
    neighbours: only that node keeps it."""
    for n in ((40, 50), (120, 96, 70)):
        P = I.random_problem(n, 5, mask_frac=0.05, k=6.0)
        m = P["mask"].astype(bool)
        u0 = P["x"].copy()
        u0[m] = np.where(np.arange(m.sum()) % 2, np.nan, np.inf)
        op = make_op(helm, P, helm.C128)
        u = op.field(u0)
        op.relax(helm.JACOBI, 0.6, 4, op.field(P["f"]), u)
        g = to_np(u)
        assert np.isfinite(g[~m.ravel()]).all()
        assert not np.isfinite(g[m.ravel()]).any()


@pytest.mark.parametrize("dtype", [helm.C128, helm.C64])
@pytest.mark.parametrize("n", [
    (64, 8, 4), (65, 9, 3), (3, 5, 3),        # marches of an even and an odd number of planes; a tile, a node more
    (131, 70, 67), (190, 66, 130),            # marches that start on planes of either parity
    (157, 142, 131),                          # one round of 15-plane marches
])
def test_rbgs_marches_equal_pairs(n, dtype):
    """The red-black ring kernel, whatever the length and first plane of its
    marches, gives the register-pair kernel's values bit for bit."""
    P = I.random_problem(n, sum(n), mask_frac=0.08, k=6.0)
    lo = dtype == helm.C64
    op = make_op(helm, P, dtype)
    f = op.field(P["f"])
    out = []
    for which in (helm.RB_PAIRS, helm.RB_RING):
        op.set_rbgs_kernel(which)
        u = op.field(stored(P["x"], lo))
        op.relax(helm.RBGS, 0.9, 3, f, u)
        out.append(to_np(u))
    assert np.array_equal(out[0], out[1])
