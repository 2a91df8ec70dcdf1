"""The shearing-box sweeps of large 3D grids (beyond 3 x 2^20 cells: two sweeps per pass over z where the x size is a
multiple of 64, staged single sweeps where it is one of 128; smaller grids take one thread a cell or two sweeps per
launch):
* one Maxwell step with a fixed sweep count (passes, a last single sweep where it is odd) against the oracle's FP64
  step, and the same number of single sweeps (tolerance mode with an unreachable tolerance: staged, or one thread a
  cell) bit for bit: one, three and many x tiles, y and z sizes smaller than the windows, ragged y tiles, chunks of 16
  and 64 planes, a last chunk of one plane, a single chunk, either sign of the shear, Delta y_s = 0 at t^n, and a Delta
  y_s that has a fractional part and wraps;
* a tolerance-mode step equals the fixed-count step with the sweep count it reports;
* whole steps against the oracle, on a grid on which the threads of the current's transport and fold loop too."""
import numpy as np
import pytest
import torch

import oracle
from _cases import Case, compare_particles, random_fields
from paper_2602_15939_amd import _lib as L, synth
from test_gpu_ksb_pass import S, _box, _current

pytestmark = pytest.mark.gpu


# |s omega0 nx / 2| dt stays below half a cell per step (the sweeps contract)
@pytest.mark.parametrize("n,omega0,start,K", [
    ((1024, 4, 769), -0.0012, 7, 5),  # chunks of 16 planes, the last of one; sixteen x tiles, one y tile
    ((1024, 772, 4), 0.0012, 0, 4),   # one chunk of the whole z size
    ((64, 223, 221), 0.006, 11, 3),   # one x tile: both x halos are images; a last sweep of one thread a cell
    ((192, 91, 181), -0.005, 23, 4),  # an interior x tile between the two face tiles
    ((256, 254, 65), 0.004, 19, 5),   # passes in chunks of 64 and one
    ((512, 254, 65), 0.002, 40, 3),   # staged single sweeps in chunks of 64 and one
])
def test_step_against_oracle_and_single_sweeps(n, omega0, start, K):
    print(f"[large sweeps] {n} K {K}", flush=True)
    J = _current(n, 31 + K)
    a, E, B = _box(n, omega0, start, J, maxwell_iters=K)
    b, _, _ = _box(n, omega0, start, J, maxwell_iters=K, maxwell_tol=1e-30)
    try:
        a.maxwell()
        b.maxwell()
        ia, ib = a.info(), b.info()
        assert ia.maxwell_sweeps == K and ib.maxwell_sweeps == K
        assert ia.errors & ~L.DERR_ORDER == 0 and ib.errors & L.DERR_NOCONVERGE
        got = [[t.cpu().numpy() for t in x.get_fields()] for x in (a, b)]
    finally:
        a.close()
        b.close()
    for fa, fb in zip(*got):
        np.testing.assert_array_equal(fa, fb)
    box = oracle.make_box(3, n, frame=oracle.SHEAR, shear_s=S, omega0=omega0, maxwell_iters=K, step=start)
    ref = E.astype(np.float64), B.astype(np.float64)
    oracle.maxwell(box, *ref, J.astype(np.float64))
    for g, o in zip(got[0], ref):
        assert np.abs(g - o).max() <= 1e-5 * np.abs(o).max()


def test_tolerance_step_equals_fixed_count_step():
    n = (128, 255, 97)
    J = _current(n, 3)
    a, _, _ = _box(n, 0.006, 5, J, maxwell_iters=64, maxwell_tol=1e-5)
    try:
        a.maxwell()
        info = a.info()
        assert info.errors & ~L.DERR_ORDER == 0 and 1 <= info.maxwell_sweeps < 64
        b, _, _ = _box(n, 0.006, 5, J, maxwell_iters=info.maxwell_sweeps)
        try:
            b.maxwell()
            for fa, fb in zip(a.get_fields(), b.get_fields()):
                np.testing.assert_array_equal(fa.cpu().numpy(), fb.cpu().numpy())
        finally:
            b.close()
    finally:
        a.close()


def test_steps_against_oracle():
    n = (128, 128, 257)  # 4,210,688 cells, four rows a thread: 4096 threads more than the fold's launch has
    g = torch.Generator().manual_seed(2)
    parts = []
    for s in range(2):
        cell = torch.randint(0, int(np.prod(n)), (120000,), generator=g).int()
        cell[60000:] = cell[60000:] % (2 * n[0] * n[1]) + n[0] * n[1] * (n[2] - 2)  # half of them in the last planes
        parts.append(dict(cell=cell, off=torch.rand((3, len(cell)), generator=g),
                          u=synth.mj_momenta(len(cell), 0.3, g, "cpu")))
    c = Case(3, n, "shear", parts=parts, q=1e-3, seed=61, omega0=0.004, maxwell_iters=8)
    c.gpu.set_step(19)
    c.box.step = 19
    try:
        for step in range(2):
            c.gpu.step()
            c.oracle_step(nthreads=16)
            for s in range(2):
                st = compare_particles(c, s, c.gpu_species(s))
                assert st["err_u"] < 2e-6 and st["err_x"] < 2e-6, (step, s, st)
            J = c.gpu.get_current().cpu().numpy()
            for part in (slice(None), slice(n[2] - 1, None)):
                ref = c.J[:, part]
                assert np.abs(ref).max() > 0 and np.abs(J[:, part] - ref).max() <= 1e-5 * np.abs(ref).max(), step
            for f, o in zip(c.gpu.get_fields(), (c.E, c.B)):
                assert np.abs(f.cpu().numpy() - o).max() <= 1e-5 * np.abs(o).max(), step
        info = c.gpu.info()
        assert info.errors & ~L.DERR_ORDER == 0 and info.n_slow == 0 and info.maxwell_sweeps == 8
    finally:
        c.close()
