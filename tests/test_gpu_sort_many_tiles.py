"""The migration sort about the tile count where its scans change from one workgroup (here with a last round of a single
word) to several launches: permutation and offsets after a push against the oracle's stable sort, bit for bit, with a
species of few particles and an empty one."""
import numpy as np
import pytest
import torch

import oracle
from paper_2602_15939_amd import _lib as L
from paper_2602_15939_amd.box import Box

pytestmark = pytest.mark.gpu


# 256 x 256 tiles, 257 x 256, 300 x 250 ragged
@pytest.mark.parametrize("n", [(2048, 2048), (2056, 2048), (2397, 1995)])
def test_sort_on_many_tiles(n):
    print(f"[many tiles] {n}", flush=True)
    m, g = 300000, torch.Generator().manual_seed(4)
    nt = [-(-v // 8) for v in n]
    tiles = nt[0] * nt[1]
    b = Box(2, (*n, 1), frame=L.FRAME_PLAIN, species=((-1.0, -1e-3, m), (1.0, 1e-3, 16)), tile=(8, 8, 1))
    try:
        b.set_particles(0, torch.randint(0, n[0] * n[1], (m,), generator=g).int(), torch.rand((2, m), generator=g),
                        torch.randn((3, m), generator=g))
        b.set_particles(1, torch.zeros(0, dtype=torch.int32), torch.zeros((2, 0)), torch.zeros((3, 0)))
        b.sort()
        for step in range(2):
            b.push()
            cell = b.get_particles(0)["cell"].cpu().numpy().astype(np.int64)
            ref, roff = oracle.stable_sort(cell % n[0] // 8 + nt[0] * (cell // n[0] // 8), tiles)
            b.sort()
            perm, off = b.get_sort(0)
            np.testing.assert_array_equal(off.cpu().numpy(), roff[: tiles + 1])
            np.testing.assert_array_equal(perm.cpu().numpy(), ref)
            assert not b.get_sort(1)[1].cpu().numpy().any()
        info = b.info()
        assert info.n_sort_migrations == 4 and info.n_sort_fallbacks == 0 and info.errors == 0
        assert list(info.n_particles) == [m, 0]
    finally:
        b.close()
