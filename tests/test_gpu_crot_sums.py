"""Gradients of controlled rotations whose partial sums fill from one to thousands of
rows: every amplitude of the register carries its share of gradients of order one, so a
lost row or remainder changes them by its share (1 / 2048 and more)."""
import numpy as np
import pytest

import qf_inputs as qi
from oracle import grad, sim
from tests.gpu_helpers import TOL, maxabs, to_np

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("D,n", [(2, 3), (2, 19), (2, 20), (3, 13), (5, 9), (16, 5)])
@pytest.mark.parametrize("dtype,rel", [("c128", 1e-9), ("c64", 1e-4)])
def test_crot_gradient_sums(D, n, dtype, rel):
    import paper_2409_17716_amd as qf
    a, b, m = 0, n - 1, 1  # the rotated qudits; the others stay in the uniform superposition
    ops = [("h", q) for q in range(n) if q not in (a, b, m)]
    ops += [("ry", a, 0, 1, 0), ("ry", b, 0, 1, 1), ("ry", m, 0, 1, 2), ("rx", m, 0, 1, 3)]
    ops += [("crx", a, b, 0, 1, 4), ("cry", b, a, 0, 1, 5), ("crz", a, m, 1, 6), ("rx", m, 0, 1, 7),
            ("cry", m, b, 0, 1, 8)]
    c = qi.Circuit(D, n, ops, np.array([1.1, -0.8, 0.9, 0.5, 0.7, -1.3, 0.6, 0.4, 1.2]))
    terms = qi.zsum_terms(n)
    t = qf.new_state(n, D, dtype)
    qf.qf_state_init(t, n, D, None)
    p = qf.plan_for(c, dtype)
    p.forward(t, c.theta)
    want = sim.run(c)
    assert maxabs(to_np(t), want) <= TOL[dtype]
    g = p.adjoint_grad(t, qf.new_state(n, D, dtype), c.theta, terms)
    ref = grad.adjoint(c, terms, psi_final=want)
    crot = np.abs(ref[[4, 5, 6, 8]])
    assert crot.min() >= 0.05 * np.abs(ref).max()  # a share of 1 / 2048 is 2e-5 of the largest
    assert np.all(np.abs(g - ref) <= rel * np.abs(ref).max())
