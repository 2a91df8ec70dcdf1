"""The field kernels read the cells beyond a face at their periodic (x: shearing-periodic) images
themselves; guards are filled once, at the end of a step.  One field step with a current against the
oracle's FP64 step on grids where every cell is at a face, odd sizes, one cell beyond a wave, and a
shear offset with a fractional part that wraps past n_y; the guards that the fill leaves are checked
through the next step's gather (tests of whole steps)."""
import numpy as np
import pytest
import torch

import oracle
from _cases import FRAMES, Case, random_fields
from paper_2602_15939_amd.box import Box, step_many

pytestmark = pytest.mark.gpu

SIZES = [(4, 4), (5, 7), (65, 6), (4, 4, 4), (5, 6, 9), (66, 4, 5)]


@pytest.mark.parametrize("frame", ["plain", "expand", "shear", "shear_expand"])
@pytest.mark.parametrize("n", SIZES)
@pytest.mark.parametrize("batched", [False, True])
def test_field_step_against_oracle(frame, n, batched):
    dim, start, K = len(n), 17, 4
    kw = dict(adot=2e-3, axis_mask=0b011) if "expand" in frame else {}
    sh = dict(shear_s=1.5, omega0=0.02) if "shear" in frame else {}
    b = Box(dim, n, frame=FRAMES[frame], species=((-1.0, 0.0, 16),), maxwell_iters=K,
            expand_adot=kw.get("adot", 0.0), expand_axis_mask=kw.get("axis_mask", 0),
            shear_s=sh.get("shear_s", 0.0), shear_omega0=sh.get("omega0", 0.0))
    try:
        E, B = random_fields(tuple(n) + (1,) * (3 - dim), 300 + dim)
        b.set_fields(torch.from_numpy(E), torch.from_numpy(B))
        b.set_step(start)
        J = np.random.default_rng(9).uniform(-0.01, 0.01, E.shape).astype(np.float32)
        if batched:
            J[:] = 0.0  # an empty box deposits nothing
            step_many([b], batched=True)
        else:
            cur = b.mem["current"][b.info().current_array]
            for c in range(3):
                b.interior(cur[c]).copy_(torch.from_numpy(J[c]))
            torch.cuda.synchronize()
            b.maxwell()
        box = oracle.make_box(dim, n, frame=FRAMES[frame], maxwell_iters=K, step=start, **kw, **sh)
        Eo, Bo = E.astype(np.float64), B.astype(np.float64)
        oracle.maxwell(box, Eo, Bo, J.astype(np.float64))
        # FP32: about 20 rounded terms a cell and sweep, K sweeps: well below 1e-5 of the largest value
        for g, o in zip(b.get_fields(), (Eo, Bo)):
            assert np.abs(g.cpu().numpy() - o).max() <= 1e-5 * np.abs(o).max()
    finally:
        b.close()


@pytest.mark.parametrize("frame", ["plain", "shear"])
@pytest.mark.parametrize("n", SIZES)
@pytest.mark.parametrize("batched", [False, True])
def test_folded_current_against_oracle(frame, n, batched):
    """Grids whose cells are boundary layers of every axis, some of both ends of a wave: the current of
    a step after the fold of the guards along the three axes."""
    c = Case(len(n), n, frame, ppc=6, seed=8, omega0=0.02, maxwell_iters=2)
    try:
        step_many([c.gpu], batched=batched)
        c.oracle_step()
        J = c.gpu.get_current().cpu().numpy()
        assert np.abs(J - c.J).max() <= 1e-5 * np.abs(c.J).max()
    finally:
        c.close()
