"""Small registers: expectations of one chunk (written by the first kernel) and of
two, and plans whose matrices go by kernel argument (up to 3840 bytes) or by a
copy, called again with other angles before the first call has run."""
import numpy as np
import pytest

import qf_inputs as qi
from oracle import measure, sim
from tests.gpu_helpers import TOL, maxabs, rounded, to_dev, to_np

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("D,n,batch", [(2, 1, 1), (3, 4, 3), (2, 12, 2), (2, 13, 2), (3, 8, 2), (3, 9, 1), (16, 3, 2),
                                       (16, 4, 1), (10, 4, 3)])
@pytest.mark.parametrize("dtype", ["c64", "c128"])
def test_expect_chunks(D, n, batch, dtype):
    import torch

    import paper_2409_17716_amd as qf
    psi = qi.random_state(D, n, 21, batch=batch).reshape(batch, -1)
    t = to_dev(psi.reshape(-1), dtype)
    ref = rounded(psi, dtype)
    for terms in (qi.z0_terms(), qi.zsum_terms(n)):
        want = [measure.expect_diag(ref[b], D, n, terms) for b in range(batch)]
        out = torch.full((2 * batch,), 7.0, dtype=torch.float64, device="cuda")
        for got in (qf.qf_expect(t, n, D, terms), qf.qf_expect_noalloc(t, n, D, terms, out)):
            g = to_np(got).reshape(batch, 2)
            assert maxabs(g[:, 0] + 1j * g[:, 1], want) <= 1e-12 * n


@pytest.mark.parametrize("dtype", ["c64", "c128"])
@pytest.mark.parametrize("layers", [1, 2, 3, 4, 9])
def test_matrix_uploads(layers, dtype):
    import paper_2409_17716_amd as qf
    c = qi.hea(3, 6, layers, 12)
    p = qf.plan_for(c, dtype)
    runs = []
    for k in range(4):
        theta = c.theta * (0.5 + 0.25 * k)
        t = qf.new_state(c.n, c.dim, dtype)
        qf.qf_state_init(t, c.n, c.dim, None)
        p.forward(t, theta)
        runs.append((t, theta))
    for t, theta in runs:
        want = sim.run(qi.Circuit(c.dim, c.n, c.ops, theta))
        assert maxabs(to_np(t), want) <= TOL[dtype]
