"""The adjoint's per-tile M sums and their reduction over the tiles: one launch up
to 32 * (256 // D^2) tiles per register, two above (chunks of about the square root),
rows of D^2 entries for every D, a ragged last chunk, several registers."""
import numpy as np
import pytest

import qf_inputs as qi
from oracle import grad, sim
from tests.gpu_helpers import to_dev

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("D,n,tile", [(2, 12, 2), (2, 12, 1), (3, 8, 2), (3, 8, 1), (4, 6, 1), (5, 5, 1), (10, 4, 1),
                                      (11, 4, 1), (16, 3, 1), (2, 13, 1), (5, 4, 1), (10, 3, 2), (16, 3, 2)])
def test_adjoint_sums_over_many_tiles(D, n, tile):
    import paper_2409_17716_amd as qf
    c = qi.hea(D, n, 1, 5, pairs=[(0, D - 1)], clock=False)
    terms = qi.zsum_terms(n)
    psi = qi.random_state(D, n, 9, batch=2)
    p = qf.plan_for(c, "c128", adj_tile_digits=tile, low_digits=1)
    t = to_dev(psi.reshape(-1), "c128")
    p.forward(t, c.theta)
    lam = qf.new_state(n, D, "c128", batch=2)
    g = p.adjoint_grad(t, lam, c.theta, terms)
    for b in range(2):
        ref = grad.adjoint(c, terms, psi_final=sim.run(c, psi[b]))
        assert np.all(np.abs(g[b] - ref) <= 1e-9 * np.abs(ref).max())
