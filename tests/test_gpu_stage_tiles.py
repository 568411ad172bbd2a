"""Register-round stages over tile shapes: tile I/O by digits (one step, several,
all steps of a tile in flight or D at a time) and by runs (D = 7, 8, 9 in a
256-lane workgroup), tiles of the whole register, several registers, forward
and adjoint, against the oracle."""
import numpy as np
import pytest

import qf_inputs as qi
from oracle import grad, sim
from tests.gpu_helpers import TOL, maxabs, to_dev, to_np

pytestmark = pytest.mark.gpu

SHAPES = [(2, 9, 4), (2, 11, 0), (2, 12, 10), (3, 6, 3), (3, 9, 6), (3, 9, 7), (4, 6, 2), (4, 7, 5), (5, 5, 3),
          (5, 6, 5), (6, 5, 4), (7, 5, 4), (8, 4, 3), (8, 5, 4), (9, 4, 3), (10, 4, 3), (11, 3, 2), (13, 3, 2),
          (16, 3, 2)]


@pytest.mark.parametrize("dtype", ["c64", "c128"])
@pytest.mark.parametrize("D,n,tile", SHAPES)
def test_stage_tile_shapes(D, n, tile, dtype):
    import paper_2409_17716_amd as qf
    if dtype == "c128" and D ** tile * 16 > 64 * 1024:
        tile -= 1
    adj = tile if 2 * D ** tile * (8 if dtype == "c64" else 16) <= 120 * 1024 else tile - 1
    c = qi.hea(D, n, 1, 8, pairs=[(0, 1)], types=("x", "y"), clock=False, cz_stride=2)
    psi = qi.random_state(D, n, 10, batch=2)
    p = qf.plan_for(c, dtype, tile_digits=tile, adj_tile_digits=adj)
    t = to_dev(psi.reshape(-1), dtype)
    p.forward(t, c.theta)
    want = np.stack([sim.run(c, psi[b]) for b in range(2)])
    assert maxabs(to_np(t), want.reshape(-1)) <= TOL[dtype]
    terms = qi.zsum_terms(n)
    g = p.adjoint_grad(t, qf.new_state(n, D, dtype, batch=2), c.theta, terms)
    rel = 1e-4 if dtype == "c64" else 1e-9
    for b in range(2):
        ref = grad.adjoint(c, terms, psi_final=want[b])
        assert np.all(np.abs(g[b] - ref) <= rel * np.abs(ref).max())
