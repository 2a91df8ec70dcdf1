"""A particle whose momentum is not finite latches its error and stays in its cell (its offset becomes NaN), also in
cells at the faces, at the edges of tiles and in a later step; the other particles move as without it."""
import numpy as np
import pytest
import torch

from _cases import Case, random_fields
from paper_2602_15939_amd import _lib as L, synth

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dim,n,frame", [(2, (40, 33), "plain"), (2, (48, 32), "shear"), (3, (24, 16, 9), "shear"),
                                         (3, (16, 16, 24), "expand")])
def test_non_finite_momentum_stays(dim, n, frame):
    at = sorted({0, 7, 8, 15, 16 % n[0], n[0] - 1})  # x, on every edge kind; y and z at both faces
    cells = [x + n[0] * (y + n[1] * z) for x in at for y in (0, n[1] - 1) for z in ((0, n[2] - 1) if dim == 3 else (0,))]
    base = synth.pair_plasma(n, 3, 0.3, 5)
    m = len(cells)
    bad = {k: torch.zeros((*v.shape[:-1], m), dtype=v.dtype) + (0.25 if k == "off" else 0) for k, v in base[0].items()}
    bad["cell"] = torch.tensor(cells, dtype=base[0]["cell"].dtype)
    bad["u"][:, 0::3], bad["u"][:, 1::3], bad["u"][1, 2::3] = float("nan"), float("inf"), float("-inf")
    parts = [{k: torch.cat([v.cpu(), bad[k]], -1) for k, v in base[0].items()}, {k: v.cpu() for k, v in base[1].items()}]
    fields = random_fields(tuple(n) + (1,) * (3 - dim), 8)
    got = []
    for p in (parts, base):
        c = Case(dim, n, frame, parts=p, fields=fields, q=0.0, omega0=0.01)
        try:
            for _ in range(3):
                c.gpu.step()
            g = c.gpu_species(0)
            got.append({k: v[..., np.argsort(g["id"])] for k, v in g.items()})
            assert bool(c.gpu.info().errors & L.DERR_NAN) == (p is parts)
        finally:
            c.close()
    live = len(base[0]["cell"])
    np.testing.assert_array_equal(got[0]["cell"][live:], cells)
    assert np.isnan(got[0]["off"][:, live:]).all()
    for k in ("cell", "off", "u"):
        np.testing.assert_array_equal(got[0][k][..., :live], got[1][k])
