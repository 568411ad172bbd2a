"""Per-gate gradients whose runs have more rows of partial sums than one workgroup adds
in four turns (32 * (256 // d^2)): chunks first, with a ragged last one; runs of both
kinds in one launch, several registers."""
import numpy as np
import pytest

import qf_inputs as qi
from oracle import mixed

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dims,batch", [([16, 16, 16, 5, 3], 2),   # 15 rows of d = 16: one launch
                                        ([16, 16, 16, 16, 3], 1),  # 48 rows: chunks of 7, the last of 6
                                        ([11, 13, 12, 10, 9], 2),  # chunks of 47 and 51 rows (13, 12), one launch (others)
                                        ([2, 10, 10, 10, 10, 10], 1)])  # 391 rows of d = 2, 79 of d = 10
def test_rows_in_chunks(dims, batch):
    import paper_2409_17716_amd as qf
    n = len(dims)
    ops, p = [], 0
    for q in range(n):
        ops += [("rx", q, 0, dims[q] - 1, p), ("ry", q, 0, 1, p + 1)]
        p += 2
    ops += [("csum", 0, 1), ("ry", 1, 0, 1, p), ("rx", 1, 0, 1, p + 1)]
    theta = np.random.default_rng(3).uniform(-2, 2, size=p + 2)
    c = qi.MixedCircuit(dims, [("h", q) for q in range(n)] + ops, theta)
    terms = qi.zsum_terms(n)
    plan = qf.plan_for(c, "c64")
    psi, lam = (qf.new_state(n, dims, "c64", batch=batch) for _ in range(2))
    qf.qf_state_init(psi, n, dims, None)
    plan.forward(psi, theta)
    g = np.asarray(plan.adjoint_grad(psi, lam, theta, terms)).reshape(batch, -1)
    ref = mixed.adjoint(c, terms)
    for b in range(batch):
        assert np.all(np.abs(g[b] - ref) <= 1e-4 * np.abs(ref).max())
