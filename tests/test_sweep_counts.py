"""Kernel passes that a per-gate plan reports: a shift after a run on its target costs no
sweep of its own up to 12 levels, above it one where the run has no reverse kernel that
folds it in (the forward walk; the reverse walk of a run without angles)."""
import pytest

import qf_inputs as qi


@pytest.mark.parametrize("d,folded", [(5, True), (12, True), (13, False), (16, False)])
def test_reported_sweeps(d, folded):
    import paper_2409_17716_amd as qf
    rot = [("rx", 0, 0, 1, 0), ("ry", 0, 0, 1, 1), ("csum", 1, 0)]
    fixed = [("h", 0), ("csum", 1, 0)]
    for ops, nparams, fwd, rev in ((rot, 2, 1 if folded else 2, 1), (fixed, 0, *([1, 1] if folded else [2, 2]))):
        p = qf.plan_for(qi.MixedCircuit([d, 3], ops, [0.1] * nparams), "c64")
        assert (p.num_stages, p.num_adjoint_stages) == (fwd, rev)
