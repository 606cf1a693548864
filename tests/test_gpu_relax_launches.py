"""How several Jacobi sweeps of a 2D grid are split into launches (csrc/relax.hip):
whatever the split, the values of single sweeps bit for bit."""
import numpy as np
import pytest

from paper_2405_12380_amd import inputs as I
from tests.helpers import make_op, stored, to_np

pytestmark = pytest.mark.gpu

helm = pytest.importorskip("paper_2405_12380_amd.helm")


@pytest.mark.parametrize("dtype", [helm.C128, helm.C64])
@pytest.mark.parametrize("n", [(512, 256), (513, 256), (33, 5000)])  # 512 tiles of 16 x 16 (up to 8 sweeps a launch); more (up to 5)
@pytest.mark.parametrize("sweeps", [2, 3, 10, 11, 16])
def test_2d_launches(n, sweeps, dtype):
    P = I.random_problem(n, sum(n), mask_frac=0.05, k=6.0)
    op = make_op(helm, P, dtype)
    f = op.field(P["f"])
    u0 = stored(P["x"], dtype == helm.C64)
    a, b = op.field(u0), op.field(u0)
    op.relax(helm.JACOBI, 0.6, sweeps, f, a)
    for _ in range(sweeps):
        op.relax(helm.JACOBI, 0.6, 1, f, b)
    assert np.array_equal(to_np(a), to_np(b))
