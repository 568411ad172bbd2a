"""The reverse walks' buffers of collected partial sums: their sizes (host check), and
gradients of batches whose sums fill a buffer more than once or need more than its
usual size for one gate."""
import os
import shutil
import subprocess

import numpy as np
import pytest

import qf_inputs as qi

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def test_collect_size_host(tmp_path):
    """A walk that empties the buffer when it is full stays inside it, in any order of
    the gates (a running sum, capped and raised to each need in turn, forgets a larger
    need met before)."""
    hipcc = shutil.which("hipcc") or "/opt/rocm/bin/hipcc"
    if not os.path.exists(hipcc):
        pytest.skip("hipcc not available")
    exe = str(tmp_path / "collect_check")
    src = os.path.join(ROOT, "tests", "collect_check.cpp")
    r = subprocess.run([hipcc, "-O2", "-std=c++17", "-x", "hip", "--offload-arch=gfx950", src, "-o", exe],
                       capture_output=True, text=True)
    assert r.returncode == 0, r.stderr
    r = subprocess.run([exe], capture_output=True, text=True)
    assert r.returncode == 0 and "OK" in r.stdout, r.stdout


def _gradients(dims, ops, theta, batch, parts):
    """Gradients of a batch of registers in basis states, by one call and by `parts`
    calls, which have to agree bit for bit; and some against the oracle."""
    import paper_2409_17716_amd as qf
    from oracle import mixed
    n = len(dims)
    terms = qi.zsum_terms(n)
    dim = dims if len(set(dims)) > 1 else dims[0]
    p = qf.Plan(dim, n, ops, len(theta), "c64")
    digits = np.stack([np.arange(batch) // 7 ** q % dims[q] for q in range(n)], axis=1).astype(np.int32)

    def grads(lo, hi):
        psi, lam = (qf.new_state(n, dim, "c64", batch=hi - lo) for _ in range(2))
        qf.qf_state_init(psi, n, dim, digits[lo:hi])
        p.forward(psi, theta)
        return np.asarray(p.adjoint_grad(psi, lam, theta, terms)).reshape(hi - lo, -1)
    whole = grads(0, batch)
    cuts = [batch * i // parts for i in range(parts + 1)]
    assert np.array_equal(whole, np.concatenate([grads(a, b) for a, b in zip(cuts, cuts[1:])]))
    for b in (0, 1, batch // 2 + 1, batch - 1):
        c = qi.MixedCircuit(list(dims), [("x", q, int(digits[b, q])) for q in range(n)] + ops, theta)
        ref = mixed.adjoint(c, terms)
        assert np.all(np.abs(whole[b] - ref) <= 1e-4 * np.abs(ref).max())


@pytest.mark.gpu
@pytest.mark.parametrize("dims,batch,parts", [([16, 2], 33000, 3),       # one run alone above the usual size
                                              ([2, 16], 33000, 3),
                                              ([13, 2, 3], 21000, 4)])   # two runs together above it
def test_rows_of_runs_over_a_full_buffer(dims, batch, parts):
    ops, p = [], 0
    for _ in range(3 if len(dims) > 2 else 1):
        for q in range(len(dims)):
            ops += [("rx", q, 0, dims[q] - 1, p), ("ry", q, 0, 1, p + 1)]
            p += 2
        ops.append(("csum", 0, 1))
    _gradients(dims, ops, np.random.default_rng(8).uniform(-2, 2, size=p), batch, parts)


@pytest.mark.gpu
def test_controlled_rotations_over_a_full_buffer():
    ops = [("ry", 0, 0, 1, 0), ("rx", 1, 0, 1, 1)]
    for i in range(36):  # 500,000 values each: the buffer fills twice
        ops.append((("crx", "cry")[i // 2 % 2], i % 2, (i + 1) % 2, 0, 1, i + 2))
    _gradients([2, 2], ops, np.random.default_rng(9).uniform(-2, 2, size=38), 500000, 4)
