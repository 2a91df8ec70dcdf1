"""The deposit's branches: every combination of side, direction and crossed axes, fused and not, on tile
edges and inside, against the oracle, node by node."""
import itertools

import numpy as np
import pytest
import torch

from _cases import Case
from paper_2602_15939_amd import _lib as L

pytestmark = pytest.mark.gpu


# one particle about every (tile / 2)-th node, shifted by shift cells: on tile edges and inside
@pytest.mark.parametrize("dim,tile", [(3, 8), (3, 4), (2, 16), (2, 8)])
@pytest.mark.parametrize("shift", [0, 1])
@pytest.mark.parametrize("fuse", [True, False])
def test_crossings_against_oracle(dim, tile, shift, fuse):
    step = max(4, tile // 2)
    n = (4 * step,) * dim
    node, rel, u = [], [], []
    for combo in itertools.product(range(4), repeat=dim):  # per axis: side and direction
        node.append([(c * step + shift) % (4 * step) for c in combo])
        rel.append([0.1 if c & 1 else -0.1 for c in combo])
        u.append([(0.9 if c & 2 else -0.9) for c in combo] + [0.4] * (3 - dim))
    x = (np.array(node) + np.array(rel)).T % n[0]
    cell = np.floor(x).astype(np.int64)
    off = torch.from_numpy((x - cell).astype(np.float32))
    ijk = sum(cell[d] * n[0] ** d for d in range(dim))
    part = dict(cell=torch.from_numpy(ijk.astype(np.int32)), off=off, u=torch.from_numpy(np.array(u, np.float32).T.copy()))
    other = dict(cell=torch.zeros(1, dtype=torch.int32), off=torch.full((dim, 1), 0.25), u=torch.zeros((3, 1)))
    zero = np.zeros((3,) + ((n[0],) if dim == 3 else (1,)) + (n[0],) * 2, np.float32)
    q, dt = 1e-4, 0.45
    c = Case(dim, n, "plain", parts=[part, other], q=q, dt=dt, fields=(zero, zero), maxwell_iters=4,
             tile=(tile, tile, tile if dim == 3 else 1))
    # a weight or displacement is off by a few units of 2^-24 a step (four steps), a current by that times q/dt
    tol = 2e-6 * q / dt
    try:
        for k in range(4):  # the first and the last cross a node
            c.gpu.sort()
            c.gpu.push(fuse=fuse)
            if not fuse:
                c.gpu.deposit()
            c.gpu.remap(L.REMAP_CURRENT)
            c.gpu.maxwell()
            c.oracle_step()
            J = c.gpu.get_current().cpu().numpy()
            assert np.abs(c.J).max() > 0.05 * q / dt
            assert np.abs(J - c.J).max() <= tol, (k, np.abs(J - c.J).max() / tol)
    finally:
        c.close()
