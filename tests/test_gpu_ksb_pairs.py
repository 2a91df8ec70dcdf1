"""Two sweeps per launch on small shearing-box grids: equal to single sweeps (tolerance mode with an
unreachable tolerance) bit for bit, on tiles cut short on any axis, one and several tiles, grids smaller
than a tile and its surroundings, even and odd counts, with the combined frame's operator, alone and batched."""
import numpy as np
import pytest
import torch

from _cases import random_fields
from paper_2602_15939_amd import _lib as L
from paper_2602_15939_amd.box import Batch, Box, step_many

pytestmark = pytest.mark.gpu


def _box(n, frame, K, tol, stream=None):
    dim = len(n)
    n3 = tuple(n) + (1,) * (3 - dim)
    b = Box(dim, n, frame=frame, species=((-1.0, 0.0, 16),), shear_s=1.5, shear_omega0=0.004, expand_adot=2e-3,
            expand_axis_mask=0b011, maxwell_iters=K, maxwell_tol=tol, stream=stream)
    E, B = random_fields(n3, 77)
    b.set_fields(torch.from_numpy(E), torch.from_numpy(B))
    b.set_step(23)  # a Delta y_s with a fraction, beyond n_y on the narrow grids
    torch.cuda.synchronize()
    cur = b.mem["current"][b.info().current_array]
    rng = np.random.default_rng(3)
    for c in range(3):
        b.interior(cur[c]).copy_(torch.from_numpy(rng.uniform(-0.01, 0.01, n3[::-1]).astype(np.float32)))
    torch.cuda.synchronize()
    return b


SIZES = [(32, 16), (33, 17), (64, 64), (31, 5), (4, 4), (8, 8, 4), (9, 17, 5), (20, 12, 16), (4, 4, 4), (65, 7, 9)]


@pytest.mark.parametrize("n", SIZES)
@pytest.mark.parametrize("frame,K", [(L.FRAME_SHEAR, 2), (L.FRAME_SHEAR, 5), (L.FRAME_SHEAR_EXPAND, 4)])
def test_pairs_equal_single_sweeps(n, frame, K):
    boxes = [_box(n, frame, K, tol) for tol in (0.0, 1e-30)]
    try:
        for b in boxes:
            b.maxwell()
            info = b.info()
            assert info.maxwell_sweeps == K and info.errors & ~(L.DERR_ORDER | L.DERR_NOCONVERGE) == 0
        for fa, fb in zip(boxes[0].get_fields(), boxes[1].get_fields()):
            np.testing.assert_array_equal(fa.cpu().numpy(), fb.cpu().numpy())
    finally:
        for b in boxes:
            b.close()


@pytest.mark.parametrize("graph", [False, True])
def test_batched_pairs_equal_single_sweeps(graph):
    st = torch.cuda.Stream()
    with torch.cuda.stream(st):
        mix = [(n, f, K) for n, f, K in zip([(33, 17), (64, 64), (9, 17, 8), (20, 12, 16), (32, 16)],
                                            [L.FRAME_SHEAR, L.FRAME_SHEAR, L.FRAME_SHEAR, L.FRAME_SHEAR_EXPAND, L.FRAME_SHEAR],
                                            [2, 5, 3, 4, 1])]
        batch = Batch(st, nbytes=1 << 20)
        sides = [[_box(n, f, K, tol, st) for n, f, K in mix] for tol in (0.0, 1e-30)]
        try:
            for bs in sides:
                for _ in range(4):
                    step_many(bs, batched=True, batch=batch, graph=graph)
            torch.cuda.synchronize()
            for a, b in zip(*sides):
                for fa, fb in zip(a.get_fields(), b.get_fields()):
                    np.testing.assert_array_equal(fa.cpu().numpy(), fb.cpu().numpy())
        finally:
            for bs in sides:
                for b in bs:
                    b.close()
            batch.close()
