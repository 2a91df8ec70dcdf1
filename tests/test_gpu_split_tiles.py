"""Tiles shared out to several workgroups (boxes of few, full tiles): fused and unfused pushes against
the oracle, and the migration counts that the parts add up against the oracle's stable sort, with a
full and a nearly empty species, one tile and ragged ones, and slot counts at the edges of a round."""
import numpy as np
import pytest
import torch

import oracle
from _cases import Case, cell_coords, compare_particles
from paper_2602_15939_amd import _lib as L

pytestmark = pytest.mark.gpu


def parts_of(dim, n, counts, seed):
    g = torch.Generator().manual_seed(seed)
    return [dict(cell=torch.randint(0, int(np.prod(n)), (m,), generator=g).int(), off=torch.rand((dim, m), generator=g),
                 u=0.5 * torch.randn((3, m), generator=g)) for m in counts]


# slots of the fuller species per tile: 32 and 33 rounds of 256, one more than a round, 2 of 512
@pytest.mark.parametrize("dim,n,frame,counts", [
    (2, (16, 16), "plain", (8192, 1)),
    (2, (16, 16), "expand", (8193, 300)),
    (2, (48, 20), "shear", (6 * 700, 6 * 257)),
    (3, (8, 8, 8), "plain", (40000, 513)),
    (3, (24, 11, 9), "shear", (12 * 1025, 40)),
])
@pytest.mark.parametrize("fuse", [True, False])
def test_split_tiles_against_oracle(dim, n, frame, counts, fuse):
    tile = (8, 8, 8) if dim == 3 else (16, 16, 1)
    c = Case(dim, n, frame, parts=parts_of(dim, n, counts, 11 + dim), q=1e-4, omega0=0.02, maxwell_iters=4)
    nt = [-(-c.n[d] // tile[d]) for d in range(3)]
    try:
        for step in range(3):
            c.gpu.sort()
            c.gpu.push(fuse=fuse)
            if not fuse:
                c.gpu.deposit()
            c.gpu.remap(L.REMAP_CURRENT)
            c.gpu.maxwell()
            c.oracle_step()
            for s in range(2):
                st = compare_particles(c, s, c.gpu_species(s))
                assert st["n"] == counts[s] and st["err_u"] < 4e-6 and st["err_x"] < 4e-6, (step, s, st)
            J = c.gpu.get_current().cpu().numpy()
            assert np.abs(J - c.J).max() <= 1e-5 * np.abs(c.J).max(), step
        keys = []
        for s in range(2):
            i, j, k = cell_coords(c.gpu.get_particles(s)["cell"].cpu().numpy(), c.n)
            keys.append(i // tile[0] + nt[0] * (j // tile[1] + nt[1] * (k // tile[2])))
        c.gpu.sort()
        for s in range(2):
            ref, roff = oracle.stable_sort(keys[s], int(np.prod(nt)))
            perm, off = c.gpu.get_sort(s)
            np.testing.assert_array_equal(off.cpu().numpy(), roff[: np.prod(nt) + 1])
            np.testing.assert_array_equal(perm.cpu().numpy(), ref)
        assert c.gpu.info().errors & ~L.DERR_ORDER == 0
    finally:
        c.close()
