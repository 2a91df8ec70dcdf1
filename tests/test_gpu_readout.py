"""Read-out kernels where they can go wrong: particle copies of counts around their groups of four (the
rows of the dense arrays then start at any 4-byte boundary), and the energy histogram at energies on,
one unit beside and within 1e-5 of the edges, and at the ends of FP32's range, with few and with the
most bins."""
import numpy as np
import pytest
import torch

import oracle
from paper_2602_15939_amd import _lib as L
from paper_2602_15939_amd.box import Box

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n", [1, 2, 3, 4, 5, 1023, 4097])
@pytest.mark.parametrize("dim,use3", [(2, 0), (3, 1)])
def test_particles_in_and_out(n, dim, use3):
    size = (13, 7) if dim == 2 else (13, 7, 6)
    b = Box(dim, size, frame=L.FRAME_LEAKY, leaky_l_esc=3.0, leaky_theta_inj=0.3, leaky_use_3vec=use3,
            species=((-1.0, -1e-3, n + 3),))
    try:
        g = torch.Generator().manual_seed(n)
        cell = torch.randint(0, int(np.prod(size)), (n,), generator=g).int()
        off, u, dr = torch.rand((dim, n), generator=g), torch.randn((3, n), generator=g), torch.randn((3, n), generator=g)
        ids = torch.randint(0, 2**31 - 1, (n,), generator=g)
        b.set_particles(0, cell, off, u, ids=ids, dr=dr)
        p = {k: v.cpu() for k, v in b.get_particles(0).items()}
        assert torch.equal(p["cell"], cell) and torch.equal(p["off"], off) and torch.equal(p["u"], u)
        assert torch.equal(p["id"], ids.int()) and torch.equal(p["dr"][:2], dr[:2])
        assert torch.equal(p["dr"][2], dr[2] if use3 else torch.zeros(n))
        b.set_particles(0, cell, off, u)  # ids 0 .. n - 1, no displacement
        p = {k: v.cpu() for k, v in b.get_particles(0).items()}
        assert torch.equal(p["id"], torch.arange(n).int()) and not p["dr"].any()
    finally:
        b.close()


@pytest.mark.parametrize("static", [False, True])
def test_histogram_beside_the_edges(static):
    rng = np.random.default_rng(3)
    u = rng.normal(size=(3, 400)) * 10.0 ** rng.uniform(-6, 6, 400)
    u = u.astype(np.float32)
    uu = (u.astype(np.float64) ** 2).sum(0)
    k = np.sort(uu / (1.0 + np.sqrt(1.0 + uu)))
    edges = np.unique(np.concatenate([k[::7], np.nextafter(k[1::7], 0), np.nextafter(k[2::7], 1e300), k[3::7] * (1 + 1e-6),
                                      k[4::7] * (1 - 3e-6), k[5::7] * (1 + 1e-5), [-1.0, 0.0, 1e-44, 1e39]]))
    ends = np.array([[0, 0, 0], [1e-20, 0, 0], [1e-16, 3e-16, 0], [1e15, 1e15, 1], [3e19, 0, 0], [np.inf, 0, 0], [np.nan, 1, 1]],
                    np.float32).T
    u = np.concatenate([u, ends], axis=1)
    more = np.concatenate([edges[:-1], np.geomspace(1e10, 1e38, 4097 - len(edges)), edges[-1:]])
    b = Box(2, (8, 8), species=((-1.0, -1e-3, u.shape[1]),))
    try:
        n = u.shape[1]
        b.set_particles(0, torch.zeros(n).int(), torch.rand(2, n), torch.from_numpy(u))
        for e in (edges, edges[::9], edges[:2], np.unique(more)):
            h = b.energy_histogram(0, list(e), static=static)
            assert list(h) == list(oracle.energy_histogram(u[0], u[1], u[2], e)), len(e)
    finally:
        b.close()


@pytest.mark.parametrize("n", [(5, 4), (6, 7), (7, 5), (4, 4, 5), (9, 5, 4), (66, 5, 6)])
def test_fields_in_and_out_at_any_row_length(n):
    """Rows of one to four elements beyond whole quads, from and to dense arrays whose rows start anywhere."""
    from paper_2602_15939_amd.box import Box

    n3 = tuple(n) + (1,) * (3 - len(n))
    g = torch.Generator().manual_seed(2)
    E, B = (torch.randn((3, n3[2], n3[1], n3[0]), generator=g) for _ in range(2))
    b = Box(len(n), n, frame=L.FRAME_PLAIN, species=((-1.0, 0.0, 16),))
    try:
        b.set_fields(E, B)
        e, f = b.get_fields()
        assert torch.equal(e.cpu(), E) and torch.equal(f.cpu(), B)
    finally:
        b.close()
