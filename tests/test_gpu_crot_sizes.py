"""Controlled rotations at the register sizes where the forward kernel changes from
one fibre per lane to four, with remainders, and the gradients' partial sums of
several gates reduced together (one to thousands of rows each)."""
import numpy as np
import pytest

import qf_inputs as qi
from oracle import grad, sim
from tests.gpu_helpers import TOL, maxabs, to_dev, to_np

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("D,n", [(2, 3), (2, 19), (2, 20), (3, 13), (5, 9), (16, 5)])
def test_crot_forward_and_gradient(D, n):
    import paper_2409_17716_amd as qf
    ops = [("crx", 0, n - 1, 0, 1, 0), ("cry", n - 1, 0, 0, D - 1, 1), ("crz", 0, 1, 1, 2), ("ry", 1, 0, 1, 3)]
    c = qi.Circuit(D, n, ops, np.array([0.4, -1.1, 0.7, 0.3]))
    psi = qi.random_state(D, n, 31)
    p = qf.plan_for(c, "c64")
    t = to_dev(psi, "c64")
    p.forward(t, c.theta)
    want = sim.run(c, psi)
    assert maxabs(to_np(t), want) <= TOL["c64"]
    terms = qi.zsum_terms(n)
    g = p.adjoint_grad(t, qf.new_state(n, D, "c64"), c.theta, terms)
    ref = grad.adjoint(c, terms, psi_final=want)
    # every entry is a sum over the amplitudes, each with a rounding error of a few
    # 2^-24: bounded by those times the norms, |O| <= n
    assert np.all(np.abs(g - ref) <= 16 * 2.0 ** -24 * n * D)
