"""The migration sort on tile grids of any shape: two tiles on an axis, sizes that are no multiple of
the tile, a last tile of two cells, and (shearing box) the x-face crossings onto such y tiles at
offsets Delta y_s over the whole period.  Permutation and offsets after every push against the
oracle's stable sort of the tile keys, bit for bit; the sorts that must be migrations are counted."""
import numpy as np
import pytest
import torch

import oracle
from _cases import Case, cell_coords
from paper_2602_15939_amd import _lib as L

pytestmark = pytest.mark.gpu

# (dim, n, frame, more, tile, whether the migration sort applies)
CASES = [
    (3, (16, 20, 9), "plain", dict(), (8, 8, 8), True),       # two tiles, ragged, two ragged
    (3, (26, 18, 25), "expand", dict(), (8, 8, 8), True),     # last tiles of two, two and one cell
    (3, (17, 33, 12), "plain", dict(tile=(4, 4, 4)), (4, 4, 4), True),
    (2, (40, 23), "leaky", dict(leaky_mode=L.LEAKY_PROBABILISTIC, t_esc=9.0, gamma_thr=1.5), (16, 16, 1), True),
    (2, (12, 90), "plain", dict(tile=(8, 8, 1)), (8, 8, 1), True),
    (3, (24, 26, 12), "shear", dict(omega0=0.05), (8, 8, 8), True),   # last y tile of two rows
    (3, (30, 31, 8), "shear", dict(omega0=-0.04), (8, 8, 8), True),   # of seven rows, x ragged too
    (2, (50, 20), "shear", dict(omega0=0.03), (16, 16, 1), True),     # two y tiles
    (2, (33, 10), "shear", dict(omega0=0.04), (16, 16, 1), True),     # one y tile, a last x tile of one cell
    (2, (41, 37), "shear", dict(omega0=0.04, tile=(8, 8, 1)), (8, 8, 1), True),
    (3, (24, 25, 8), "shear", dict(omega0=0.05), (8, 8, 8), False),   # a last y tile of one row: radix
    (3, (16, 24, 8), "shear", dict(omega0=0.05), (8, 8, 8), False),   # two x tiles: radix
]


@pytest.mark.parametrize("dim,n,frame,kw,tile,migrates", CASES, ids=["%s%s" % (c[2], "x".join(map(str, c[1]))) for c in CASES])
def test_sort_after_push_any_tile_grid(dim, n, frame, kw, tile, migrates):
    c = Case(dim, n, frame, ppc=5, seed=60 + dim, theta=0.6, maxwell_iters=2, **kw)
    nt = [-(-c.n[d] // tile[d]) for d in range(3)]
    try:
        up = [len(p["cell"]) for p in c.parts]
        for step in range(14):
            if frame == "shear":  # offsets spread over the period
                c.gpu.set_step(7 * step * step)
            want = []
            for s in range(2):
                cell = c.gpu.get_particles(s)["cell"].cpu().numpy().astype(np.int64)
                i, j, k = cell_coords(np.maximum(cell, 0), c.n)
                key = i // tile[0] + nt[0] * (j // tile[1] + nt[1] * (k // tile[2]))
                key[cell < 0] = np.prod(nt)
                want.append(np.concatenate([key, np.full(up[s] - len(key), np.prod(nt))]))
            c.gpu.sort()
            for s in range(2):
                ref, roff = oracle.stable_sort(want[s], int(np.prod(nt)))
                perm, off = c.gpu.get_sort(s)
                np.testing.assert_array_equal(off.cpu().numpy(), roff[: np.prod(nt) + 1], err_msg=f"step {step}")
                np.testing.assert_array_equal(perm.cpu().numpy(), ref[: roff[np.prod(nt)]], err_msg=f"step {step}")
            c.gpu.push(fuse=True)
        info = c.gpu.info()
        assert info.n_sort_migrations == (2 * 13 if migrates else 0) and info.n_sort_fallbacks == 0
        assert info.n_slow == 0
    finally:
        c.close()


def test_scan_on_more_tiles_than_the_scatter_scans():
    """1200 tiles (the scan kernel's ragged end) and a species without particles."""
    n, tile = (240, 320), (8, 8, 1)
    parts = [dict(cell=torch.randint(0, n[0] * n[1], (m,), generator=torch.Generator().manual_seed(3)).int(),
                  off=torch.rand(2, m), u=torch.randn(3, m)) for m in (20000, 0)]
    c = Case(2, n, "plain", parts=parts, tile=tile)
    try:
        for step in range(3):
            cell = c.gpu.get_particles(0)["cell"].cpu().numpy().astype(np.int64)
            key = (cell % n[0]) // 8 + 30 * (cell // n[0] // 8)
            c.gpu.sort()
            ref, roff = oracle.stable_sort(key, 1200)
            perm, off = c.gpu.get_sort(0)
            np.testing.assert_array_equal(off.cpu().numpy(), roff[:1201])
            np.testing.assert_array_equal(perm.cpu().numpy(), ref)
            assert int(c.gpu.get_sort(1)[1].abs().max()) == 0
            c.gpu.push()
        assert c.gpu.info().n_sort_migrations == 4
    finally:
        c.close()
