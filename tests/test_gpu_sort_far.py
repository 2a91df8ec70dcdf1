"""Particles moved out of their tiles in the caller's memory between sort and push: the push handles them outside the
tile (PIC_DERR_ORDER, n_slow), and where one is beyond the neighbouring tiles the next sort, batched or not, is a radix
sort by one workgroup.  Permutation, offsets and live counts of that sort and of the next one, again a migration,
against the oracle's stable sort, bit for bit."""
import numpy as np
import pytest
import torch

import oracle
from _cases import Case, cell_coords
from paper_2602_15939_amd import _lib as L
from paper_2602_15939_amd.box import Batch

pytestmark = pytest.mark.gpu


def cell_array(b, s):
    """The caller's tensor with the packed cells of species s."""
    lay = b.layout
    per = 1 + b.dim + 3 + bool(lay.has_id) + 3 * bool(lay.has_dr)
    k = b.info().particle_copy[s]
    return b._tensors[6 * lay.field_sets + 3 * lay.current_arrays + (2 * s + k) * per]


def keys_of(c, s, tile, nt):
    cell = c.gpu.get_particles(s)["cell"].cpu().numpy().astype(np.int64)
    i, j, k = cell_coords(np.maximum(cell, 0), c.n)
    key = i // tile[0] + nt[0] * (j // tile[1] + nt[1] * (k // tile[2]))
    key[cell < 0] = np.prod(nt)
    return key


def check_sort(c, keys, nt):
    live = []
    for s, key in enumerate(keys):
        ref, roff = oracle.stable_sort(key, nt)
        perm, off = c.gpu.get_sort(s)
        np.testing.assert_array_equal(off.cpu().numpy(), roff[: nt + 1])
        np.testing.assert_array_equal(perm.cpu().numpy(), ref[: roff[nt]])
        live.append(int(roff[nt]))
    return live


# tile counts of one, two and (3D) one radix digits; whole, ragged and two-tile grids; dead particles
@pytest.mark.parametrize("dim,n,tile,frame,kw", [
    (2, (64, 48), (16, 16, 1), "plain", {}),
    (2, (200, 168), (8, 8, 1), "leaky", dict(leaky_mode=L.LEAKY_PROBABILISTIC, t_esc=9.0, gamma_thr=1.1)),
    (3, (40, 32, 24), (8, 8, 8), "shear", dict(omega0=0.02)),
    (3, (26, 18, 16), (8, 8, 8), "plain", {}),
])
@pytest.mark.parametrize("batched", [False, True])
def test_sort_after_particles_were_moved_far(dim, n, tile, frame, kw, batched):
    c = Case(dim, n, frame, ppc=3, seed=17, tile=tile, maxwell_iters=4, **kw)
    nt3 = [-(-c.n[d] // tile[d]) for d in range(3)]
    nt = int(np.prod(nt3))
    bits = [max(c.n[d] - 1, 1).bit_length() for d in range(2)]
    rng = np.random.default_rng(3)
    try:
        c.gpu.step()
        c.gpu.sort()
        before = c.gpu.info()
        cells = cell_array(c.gpu, 1)
        live = before.n_particles[1]
        which = rng.choice(live, min(300, live // 2), replace=False)
        to = [rng.integers(0, c.n[d], len(which)) for d in range(3)]
        packed = to[0] | to[1] << bits[0] | to[2] << (bits[0] + bits[1])
        torch.cuda.synchronize()
        at = torch.from_numpy(which).cuda()
        keep = cells[at] >= 0
        cells[at[keep]] = torch.from_numpy(packed.astype(np.int32)).cuda()[keep]
        torch.cuda.synchronize()
        c.gpu.push()
        keys = [keys_of(c, s, tile, nt3) for s in range(2)]
        if batched:
            c.gpu.remap(L.REMAP_CURRENT)
            c.gpu.maxwell()
            batch = Batch(c.gpu.stream)
            batch.step([c.gpu])
            torch.cuda.synchronize()
            batch.close()
            live = check_sort(c, keys, nt)
        else:
            c.gpu.sort()
            live = check_sort(c, keys, nt)
            c.gpu.push()
        info = c.gpu.info()
        assert info.n_slow > 0 and info.errors & L.DERR_ORDER and not info.errors & L.DERR_SORT
        assert info.n_sort_fallbacks == 1  # the other species' sort was a migration
        assert list(info.n_particles) == live
        keys = [keys_of(c, s, tile, nt3) for s in range(2)]
        c.gpu.sort()
        check_sort(c, keys, nt)
        assert c.gpu.info().n_sort_fallbacks == 1
    finally:
        c.close()
