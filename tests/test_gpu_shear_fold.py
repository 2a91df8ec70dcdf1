"""The shearing box's current fold takes four rows a thread: against the oracle's on y sizes that leave one to
three rows over, with shifts Delta y_s that wrap past n_y, and a shear flow that moves rows by more than a cell."""
import numpy as np
import pytest

from _cases import Case
from paper_2602_15939_amd import _lib as L

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dim,n", [(2, (16, 4)), (2, (20, 21)), (2, (64, 18)), (3, (12, 7, 5)), (3, (24, 16, 9))])
@pytest.mark.parametrize("omega0,start", [(0.01, 0), (-0.02, 31), (0.03, 50)])
def test_shear_fold_against_oracle(dim, n, omega0, start):
    c = Case(dim, n, "shear", ppc=6, seed=5, omega0=omega0, maxwell_iters=4)
    c.gpu.set_step(start)
    c.box.step = start
    try:
        c.gpu.sort()
        c.gpu.push()
        c.gpu.remap(L.REMAP_CURRENT)
        c.oracle_step()
        J = c.gpu.get_current().cpu().numpy()
        # terms of FP32 weights and a sum of at most a few tens of them per node
        assert np.abs(J - c.J).max() <= 1e-5 * np.abs(c.J).max()
    finally:
        c.close()
