"""The staged shearing-box sweeps cut z into chunks of 4 to 64 planes by the grid's column tiles.  The
two-sweep pass equals single sweeps (tolerance mode with an unreachable tolerance) bit for bit where
the two cut differently: one whole chunk against chunks of 4, a ragged last chunk, one plane more
than a chunk, and one-thread-per-cell single sweeps (x size 64)."""
import numpy as np
import pytest

from paper_2602_15939_amd import _lib as L
from test_gpu_ksb_pass import _box, _current

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n", [(128, 1024, 6), (64, 256, 130), (128, 256, 65), (256, 12, 33)])
def test_pass_equals_single_sweeps_for_any_chunks(n):
    J = _current(n, 5)
    boxes = [_box(n, 0.003, 13, J, maxwell_iters=4, maxwell_tol=t)[0] for t in (0.0, 1e-30)]
    try:
        for b in boxes:
            b.maxwell()
            assert b.info().errors & ~(L.DERR_ORDER | L.DERR_NOCONVERGE) == 0
        for fa, fb in zip(boxes[0].get_fields(), boxes[1].get_fields()):
            np.testing.assert_array_equal(fa.cpu().numpy(), fb.cpu().numpy())
    finally:
        for b in boxes:
            b.close()


# passes and staged single sweeps begin beyond 3 x 2^20 cells: one, three and sixteen x tiles, ragged y tiles,
# y smaller than the windows, a ragged last chunk, odd counts (a last single sweep, one thread a cell unless
# the x size is a multiple of 128)
@pytest.mark.parametrize("n,K", [((64, 250, 200), 4), ((192, 91, 181), 3), ((1024, 4, 801), 5)])
def test_pass_equals_single_sweeps_beyond_its_line(n, K):
    test_pass_equals_staged_single_sweeps(n, K)


# a last chunk of one plane, ragged y tiles, one and two x tiles; odd counts end in a single sweep
@pytest.mark.parametrize("n,K", [((128, 255, 97), 4), ((256, 126, 100), 5)])
def test_pass_equals_staged_single_sweeps(n, K):
    J = _current(n, 7)
    boxes = [_box(n, 0.003, 13, J, maxwell_iters=K, maxwell_tol=t)[0] for t in (0.0, 1e-30)]
    try:
        for b in boxes:
            b.maxwell()
            assert b.info().errors & ~(L.DERR_ORDER | L.DERR_NOCONVERGE) == 0
        for fa, fb in zip(boxes[0].get_fields(), boxes[1].get_fields()):
            np.testing.assert_array_equal(fa.cpu().numpy(), fb.cpu().numpy())
    finally:
        for b in boxes:
            b.close()
