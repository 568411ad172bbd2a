"""Per-gate schedules with shifts merged into the sweep of their target's last run:
forward and gradient against the oracle where the merge applies (CSUM, controlled
shift and X right after or across other qudits' runs), where it must not (a touched
control, a second shift, a diagonal gate between), and over many runs, registers
and dimensions (the runs' M sums reduced together)."""
import numpy as np
import pytest

import qf_inputs as qi
from oracle import mixed
from tests.gpu_helpers import TOL, maxabs, to_dev, to_np

pytestmark = pytest.mark.gpu


def _circuits():
    for dims, layers in (([2, 3, 4, 5], 2), ([5, 2, 7, 3, 2], 3), ([3, 16, 2], 2), ([2, 2, 2, 2, 2, 2, 3], 12)):
        yield qi.mixed_hea(dims, layers, 4)
    dims = [3, 4, 2, 5]
    p = 0
    ops = []

    def run(q):
        nonlocal p
        ops.extend([("rx", q, 0, 1, p), ("ry", q, 0, 1, p + 1)])
        p += 2
    run(0), run(1), run(2), run(3)
    ops += [("x", 1, 3), ("csum", 0, 2), ("csum", 3, 2)]          # two shifts of one target
    run(2)
    ops += [("cz", 2, 0), ("csum", 0, 2)]                         # a diagonal gate between
    run(0)
    ops += [("cshift", 0, 3, (2, 0, 4)), ("csum", 1, 3)]          # a table; control touched later
    run(1)
    ops += [("csum", 1, 3), ("csum", 3, 0), ("x", 3, 1)]
    run(3)
    ops += [("crx", 0, 3, 0, 1, p), ("csum", 2, 3)]
    p += 1
    run(3)
    ops += [("h", 1), ("csum", 2, 1)]
    yield qi.MixedCircuit(dims, ops, np.random.default_rng(6).uniform(-3, 3, size=p), "merge_cases")


# complex128 matrices of dimension 12 and more are no kernel argument
CASES = [(c, dt) for c in _circuits() for dt in ("c64", "c128") if dt == "c64" or max(c.dims) < 12]


@pytest.mark.parametrize("c,dtype", CASES, ids=[f"{c.name}-{dt}" for c, dt in CASES])
def test_merged_shifts(c, dtype):
    import paper_2409_17716_amd as qf
    rng = np.random.default_rng(3)
    psi = rng.standard_normal((2, c.amps)) + 1j * rng.standard_normal((2, c.amps))
    psi /= np.linalg.norm(psi, axis=1, keepdims=True)
    p = qf.plan_for(c, dtype)
    t = to_dev(psi.reshape(-1), dtype)
    p.forward(t, c.theta)
    # gradient: two registers from |0...0>
    terms = [(q, "z") for q in range(c.n)]
    qf.qf_state_init(t, c.n, c.dims, None)
    p.forward(t, c.theta)
    g = p.adjoint_grad(t, qf.new_state(c.n, c.dims, dtype, batch=2), c.theta, terms)
    ref = mixed.adjoint(c, terms)
    for b in range(2):
        assert np.all(np.abs(g[b] - ref) <= (1e-4 if dtype == "c64" else 1e-9) * np.abs(ref).max())


@pytest.mark.parametrize("d", [11, 12, 13, 15, 16])
@pytest.mark.parametrize("where", [0, 1, 2])
def test_merged_shifts_of_large_qudits(d, where):
    """Up to 12 levels a shift goes into the sweep, above it takes one of its own:
    CSUM, a table, X, after runs with and without angles (undone in the reverse walk)."""
    import paper_2409_17716_amd as qf
    dims = [3, 4]
    dims.insert(where, d)
    q, a, b = where, (where + 1) % 3, (where + 2) % 3
    tab = tuple((5 * i + 2) % d for i in range(dims[a]))
    ops = [("h", 0), ("h", 1), ("h", 2), ("csum", a, q), ("rx", q, 0, d - 1, 0), ("cshift", a, q, tab), ("h", q),
           ("x", q, d - 2), ("cz", q, b), ("ry", q, 1, 2, 1), ("csum", b, q), ("rx", a, 0, 1, 2), ("csum", q, a)]
    c = qi.MixedCircuit(dims, ops, np.array([0.4, -1.3, 2.1]), "large")
    t = qf.new_state(3, dims, "c64")
    p = qf.plan_for(c, "c64")
    qf.qf_state_init(t, 3, dims, None)
    p.forward(t, c.theta)
    assert maxabs(to_np(t), mixed.run(c)) <= TOL["c64"]
    terms = [(i, "z") for i in range(3)]
    g = p.adjoint_grad(t, qf.new_state(3, dims, "c64"), c.theta, terms)
    ref = mixed.adjoint(c, terms)
    assert np.all(np.abs(g - ref) <= 1e-4 * np.abs(ref).max())
    # the reverse walk ends at |0...0>
    assert abs(to_np(t)[0] - 1) <= TOL["c64"]
