"""The work a user of this framework has it do, as timed cases.

A user builds a register of qudits, runs circuits on it through a plan (or gate
by gate), and then reads probabilities, expectation values, shots or adjoint
gradients.  Every case goes through the package's public calls; sizes are those
of the repository's workloads, tests and benchmark, or spread between them.

    listed()             the fixed cases
    draw(rng)            one more case of the same ranges
    prepare(case, seed)  what a program holds before the call
    run(state)           one pass, and its outputs
    work(case)           bytes and operations a pass cannot do without
    exact(case, seed)    the outputs in 64 bits from plain torch
"""
from __future__ import annotations

import math
import random
from types import SimpleNamespace

import numpy as np
import torch

# ---------------------------------------------------------------------------
# Circuits.  Gate descriptors as the package takes them: ("rx"|"ry", q, j, k, p),
# ("rz", q, j, p), ("clock", q, a), ("csum", c, t), ("cz", c, t), ("h", q),
# ("crx"|"cry", c, t, j, k, p), ("crz", c, t, j, p).
# ---------------------------------------------------------------------------


def _dims(case):
    return [int(d) for d in case["dims"].split(",")] if "dims" in case else [case["dim"]] * case["n"]


def _dim_arg(case):
    return _dims(case) if "dims" in case else case["dim"]


def _amps(case):
    return math.prod(_dims(case))


def _circuit(case, clocks):
    """Gate list and number of angles of a case's circuit; clocks: exponents of
    the clock gates in order (one per layer and qudit)."""
    dims = _dims(case)
    n, ops, p = len(dims), [], 0
    if case.get("start_h"):
        ops += [("h", q) for q in range(n)]
    for layer in range(case["layers"]):
        for t in case["types"]:
            for j in range(case["pairs"]):
                for q in range(n):
                    if j + 1 >= dims[q]:
                        continue
                    ops.append(("rz", q, j + 1, p) if t == "z" else ("r" + t, q, j, j + 1, p))
                    p += 1
        if case.get("clock"):
            ops += [("clock", q, int(clocks[layer * n + q])) for q in range(n)]
        if case["entangler"] == "ring":
            ops += [("csum", i, (i + 1) % n) for i in range(n)]
        elif case["entangler"] == "chain":
            ops += [("csum", i, i + 1) for i in range(n - 1)]
        elif case["entangler"] == "rotations":
            for i in range(n):
                t, kind = (i + 1) % n, ("crx", "cry", "crz")[i % 3]
                ops.append(("crz", i, t, 1, p) if kind == "crz" else (kind, i, t, 0, 1, p))
                p += 1
        if case.get("cz") and n > 2:
            ops += [("cz", i, (i + 2) % n) for i in range(n)]
    return ops, p


def _problem(case, seed):
    """Gate list, number of angles and the angles (batch x angles) of a case."""
    rng = np.random.default_rng([seed, 7])
    dims = _dims(case)
    clocks = rng.integers(0, min(dims), size=max(1, case["layers"]) * len(dims))
    ops, nparams = _circuit(case, clocks)
    theta = rng.uniform(-np.pi, np.pi, size=(case.get("batch", 1), nparams))
    return ops, nparams, theta


def _zterms(n):
    return [(q, "z") for q in range(n)]


def _torch_dtype(case):
    return torch.complex64 if case["dtype"] == "c64" else torch.complex128


def _random_state(case, seed):
    """Normalised complex Gaussian registers (the states deep random circuits end in)."""
    gen = torch.Generator(device="cuda").manual_seed(1000003 * seed + 17)
    b, N = case.get("batch", 1), _amps(case)
    x = torch.randn((b, N, 2), generator=gen, device="cuda", dtype=torch.float64)
    x /= x.reshape(b, -1).norm(dim=1).reshape(b, 1, 1)
    return torch.view_as_complex(x).to(_torch_dtype(case)).reshape(-1).contiguous()


def _unitary(m, rng, real=False):
    z = rng.standard_normal((m, m))
    if not real:
        z = z + 1j * rng.standard_normal((m, m))
    q, r = np.linalg.qr(z)
    d = np.diag(r)
    return (q * (d / np.abs(d))).astype(np.complex128)


# ---------------------------------------------------------------------------
# Cases.
# ---------------------------------------------------------------------------

def listed():
    return [
        # the smallest call there is: a four-qutrit example circuit in double precision,
        # run and measured (state, probabilities, expectation); launches and host time
        dict(name="forward_d3_n4_c128", kind="forward", dim=3, n=4, dtype="c128", layers=2, types="y", pairs=2,
             entangler="chain", start_h=True),
        # one training step of a small variational model through autograd
        dict(name="train_d3_n7_c128", kind="train", dim=3, n=7, dtype="c128", layers=3, types="xyz", pairs=2,
             entangler="ring", batch=4),
        # the benchmark's workload: a deep qutrit ansatz on 43 million amplitudes
        dict(name="forward_d3_n16_c64", kind="forward", dim=3, n=16, dtype="c64", layers=10, types="xyz", pairs=2,
             clock=True, entangler="ring"),
        # loss and gradient of a register that fits the caches (D = 5, ten million amplitudes)
        dict(name="gradient_d5_n10_c64", kind="gradient", dim=5, n=10, dtype="c64", layers=8, types="xyz", pairs=4,
             entangler="ring", cz=True),
        # the largest: loss and checkpointed gradient on 10^8 amplitudes
        dict(name="gradient_d10_n8_c64", kind="gradient", dim=10, n=8, dtype="c64", layers=12, types="y", pairs=9,
             entangler="ring", ckpt=320),
        # gradient through controlled rotations (per-gate kernels between the stages)
        dict(name="gradient_crot_d4_n9_c128", kind="gradient", dim=4, n=9, dtype="c128", layers=3, types="y", pairs=2,
             entangler="rotations"),
        # loss and gradient on a register of qudits of different dimensions
        dict(name="gradient_mixed_c64", kind="gradient", dims="2,3,4,5,2,3,4,5,2,3,4,5", dtype="c64", layers=3,
             types="xyz", pairs=1, entangler="ring"),
        # a training step of 1024 uneven circuits as one graph replay
        dict(name="ragged_1024_c64", kind="ragged", dtype="c64", layers=6, types="xyz", pairs=2, clock=True,
             entangler="ring", d3=768, d4=256),
        # circuits written gate by gate: every one-gate call over a whole register
        dict(name="gates_d3_n15_c64", kind="gates", dim=3, n=15, dtype="c64"),
        # a user's own dense blocks over adjacent qudits (K = 49, complex)
        dict(name="blocks_d7_n9_c64", kind="blocks", dim=7, n=9, dtype="c64", span=2, real=False),
        # probabilities, marginals and expectation values of several registers
        dict(name="measure_d4_n11_c64", kind="measure", dim=4, n=11, dtype="c64", batch=3),
        # a million shots of a large register, and of two of its qudits
        dict(name="shots_d3_n16_c64", kind="shots", dim=3, n=16, dtype="c64", shots=1 << 20),
    ]


def _pick_register(rng, lo, hi, dims=(2, 3, 3, 3, 4, 5, 6, 7, 8, 9, 10)):
    """A dimension and a qudit count with lo <= D^n <= hi (log-uniform)."""
    d = rng.choice(dims)
    target = math.exp(rng.uniform(math.log(lo), math.log(hi)))
    n = max(2, int(round(math.log(target) / math.log(d))))
    while n > 2 and d ** n > hi:
        n -= 1
    return d, n


def draw(rng: random.Random):
    kind = rng.choice(["forward", "forward", "gradient", "gradient", "mixed", "train", "ragged", "gates", "blocks",
                       "measure", "shots"])
    dtype = rng.choice(["c64", "c64", "c128"])
    if kind in ("forward", "gradient"):
        d, n = _pick_register(rng, 64, 4.3e7 if kind == "forward" else 1e7)
        case = dict(kind=kind, dim=d, n=n, dtype=dtype, layers=rng.randint(1, 8),
                    types=rng.choice(["y", "xyz", "xyz", "xz"]), pairs=rng.randint(1, min(4, d - 1)),
                    entangler=rng.choice(["ring", "ring", "chain", "rotations"]), clock=rng.random() < 0.4,
                    cz=rng.random() < 0.3)
        if kind == "gradient" and rng.random() < 0.3:
            case["ckpt"] = rng.randint(20, 120)
        return case
    if kind == "mixed":
        pool = [2, 3, 4, 5, 6, 7]
        dims, target = [], math.exp(rng.uniform(math.log(64), math.log(4e6)))
        while len(dims) < 2 or math.prod(dims) * 2 <= target:
            dims.append(rng.choice(pool))
        if len(set(dims)) == 1:
            dims[0] = dims[0] + 1
        return dict(kind="gradient", dims=",".join(map(str, dims)), dtype=dtype, layers=rng.randint(1, 4),
                    types=rng.choice(["y", "xyz"]), pairs=1, entangler=rng.choice(["ring", "chain"]))
    if kind == "train":
        d, n = _pick_register(rng, 27, 3e5)
        return dict(kind="train", dim=d, n=n, dtype=dtype, layers=rng.randint(1, 4), types=rng.choice(["y", "xyz"]),
                    pairs=rng.randint(1, min(3, d - 1)), entangler=rng.choice(["ring", "chain"]),
                    batch=rng.randint(1, 8))
    if kind == "ragged":
        return dict(kind="ragged", dtype="c64", layers=rng.randint(2, 6), types=rng.choice(["y", "xyz"]), pairs=2,
                    clock=rng.random() < 0.5, entangler="ring", d3=rng.randint(20, 400), d4=rng.randint(10, 150))
    if kind == "blocks":
        d, n = _pick_register(rng, 4e3, 1.2e7)
        span = rng.randint(1, max(1, min(n, int(math.log(256) / math.log(d)))))
        return dict(kind="blocks", dim=d, n=n, dtype=dtype, span=span, real=rng.random() < 0.4)
    if kind == "gates":
        d, n = _pick_register(rng, 100, 1.5e7)
        return dict(kind="gates", dim=d, n=max(3, n) if d ** 3 <= 1000 else n, dtype=dtype)
    if kind == "measure":
        d, n = _pick_register(rng, 64, 1.2e7)
        return dict(kind="measure", dim=d, n=n, dtype=dtype, batch=rng.randint(1, 4))
    d, n = _pick_register(rng, 64, 4.3e7)
    return dict(kind="shots", dim=d, n=n, dtype="c64" if d ** n > 1e7 else dtype,
                shots=int(math.exp(rng.uniform(math.log(1000), math.log(1 << 20)))))


# ---------------------------------------------------------------------------
# Inputs of the cases that are not one circuit.
# ---------------------------------------------------------------------------

def _ragged_sizes(case):
    """(D, n) of every circuit: the work list is part of the case, its angles are not."""
    rng = np.random.default_rng([case["d3"], case["d4"], 11])
    return [(3, int(n)) for n in rng.integers(6, 11, size=case["d3"])] + \
           [(4, int(n)) for n in rng.integers(5, 9, size=case["d4"])]


def _ragged_circuits(case, seed):
    rng = np.random.default_rng([seed, 13])
    out = []
    for d, n in _ragged_sizes(case):
        sub = dict(case, dim=d, n=n)
        clocks = rng.integers(0, d, size=case["layers"] * n)
        ops, nparams = _circuit(sub, clocks)
        out.append(SimpleNamespace(dim=d, n=n, ops=ops, nparams=nparams, clocks=clocks,
                                   theta=rng.uniform(-np.pi, np.pi, size=nparams)))
    return out


def _gate_list(case, seed):
    """One call of every per-gate entry point, at several places of the register."""
    rng = np.random.default_rng([seed, 5])
    D, n = case["dim"], case["n"]
    calls = [("1q", q, _unitary(D, rng)) for q in range(n)]
    for q in range(n - 1):
        calls.append(("ctrl", q, q + 1, [int(v) for v in rng.integers(0, D, size=D)]))
    for q in sorted({0, n // 2, n - 1}):
        o = (q + n // 2) % n if n > 1 else q
        o = o if o != q else (q + 1) % n
        w = np.exp(2j * np.pi * rng.random(D * D))
        calls.append(("diag", (q, o), w))
        a = float(rng.uniform(-np.pi, np.pi))
        calls.append(("rot", "rx", q, 0, D - 1, a))
        calls.append(("rot", "rz", q, 1, 0, -a))
        calls.append(("crot", "cry", o, q, 0, 1, a))
        calls.append(("crot", "crz", q, o, 1, 0, a))
        calls.append(("swap", q, o))
        if n >= 3:
            t = next(i for i in range(n) if i not in (q, o))
            calls.append(("mcx", (q, o), t))
    return calls


def _blocks(case, seed):
    rng = np.random.default_rng([seed, 3])
    K = case["dim"] ** case["span"]
    return [(q0, _unitary(K, rng, case["real"])) for q0 in range(case["n"] - case["span"] + 1)]


def _measured(case):
    """Qudit lists of the marginals: one, a far pair, and up to four in any order."""
    n = case["n"]
    return [[n // 2], [n - 1, 0], sorted({0, n // 3, n // 2, n - 1}, reverse=True)]


def _tables(case, seed):
    """A user's own diagonal observable: one complex table per qudit of a few."""
    rng = np.random.default_rng([seed, 19])
    D = case["dim"]
    qs = sorted({0, case["n"] // 2, case["n"] - 1})
    return [(q, rng.standard_normal(D) + 1j * rng.standard_normal(D)) for q in qs]


def _uniforms(case, seed):
    return np.random.default_rng([seed, 23]).random(case["shots"])


# ---------------------------------------------------------------------------
# prepare / run.
# ---------------------------------------------------------------------------

def prepare(case, seed):
    import paper_2409_17716_amd as qf
    kind = case["kind"]
    s = SimpleNamespace(kind=kind, case=case, qf=qf)
    if kind in ("forward", "gradient"):
        ops, nparams, theta = _problem(case, seed)
        s.dim, s.n = _dim_arg(case), len(_dims(case))
        s.plan = qf.Plan(s.dim, s.n, ops, nparams, case["dtype"], ckpt_every=case.get("ckpt", 0))
        s.theta = theta[0].copy()
        s.terms = _zterms(s.n)
        s.psi = qf.new_state(s.n, s.dim, case["dtype"])
        if kind == "gradient":
            s.lam = qf.new_state(s.n, s.dim, case["dtype"])
    elif kind == "train":
        from paper_2409_17716_amd.autograd import DeviceCircuit
        ops, nparams, theta = _problem(case, seed)
        s.terms = _zterms(case["n"])
        s.dc = DeviceCircuit(dim=case["dim"], n=case["n"], ops=ops, nparams=nparams, dtype=case["dtype"],
                             batch=case["batch"])
        s.theta = torch.tensor(theta, dtype=torch.float64, device="cuda", requires_grad=True)
    elif kind == "ragged":
        from paper_2409_17716_amd.batched import RaggedBatch
        s.rb = RaggedBatch(_ragged_circuits(case, seed), dtype=case["dtype"])
        s.rb.capture()
    elif kind == "gates":
        s.calls = _gate_list(case, seed)
        s.psi = qf.new_state(case["n"], case["dim"], case["dtype"])
    elif kind == "blocks":
        s.blocks = [(q0, torch.tensor(B, dtype=_torch_dtype(case), device="cuda")) for q0, B in _blocks(case, seed)]
        s.psi = qf.new_state(case["n"], case["dim"], case["dtype"])
        w = np.exp(2j * np.pi / case["dim"])
        k = np.arange(case["dim"])
        s.h = w ** np.outer(k, k) / np.sqrt(case["dim"])
    elif kind == "measure":
        s.psi = _random_state(case, seed)
        s.tables = _tables(case, seed)
    elif kind == "shots":
        s.psi = _random_state(case, seed)
        s.u = torch.from_numpy(_uniforms(case, seed)).cuda()
    else:
        raise ValueError(kind)
    return s


def run(s):
    qf, case, kind = s.qf, s.case, s.kind
    if kind == "forward":
        qf.qf_state_init(s.psi, s.n, s.dim, None)
        s.plan.forward(s.psi, s.theta)
        return [s.psi, qf.qf_probs(s.psi, s.n, s.dim), qf.qf_expect(s.psi, s.n, s.dim, s.terms)]
    if kind == "gradient":
        qf.qf_state_init(s.psi, s.n, s.dim, None)
        s.plan.forward(s.psi, s.theta)
        loss = qf.qf_expect(s.psi, s.n, s.dim, s.terms)
        return [loss, s.plan.adjoint_grad(s.psi, s.lam, s.theta, s.terms)]
    if kind == "train":
        s.theta.grad = None
        loss = s.dc.expectation(s.theta, s.terms)
        loss.sum().backward()
        return [loss.detach(), s.theta.grad]
    if kind == "ragged":
        s.rb.replay()
        return [g.loss for g in s.rb.groups] + [g.grad[:, :g.nrot] for g in s.rb.groups]
    D, n = case["dim"], case["n"]
    if kind == "gates":
        qf.qf_state_init(s.psi, n, D, None)
        for c in s.calls:
            if c[0] == "1q":
                qf.qf_apply_1q(s.psi, n, D, c[1], c[2])
            elif c[0] == "ctrl":
                qf.qf_apply_ctrl(s.psi, n, D, c[1], c[2], c[3])
            elif c[0] == "diag":
                qf.qf_apply_diag(s.psi, n, D, c[1], c[2])
            elif c[0] == "rot":
                qf.qf_apply_rot(s.psi, n, D, *c[1:])
            elif c[0] == "crot":
                qf.qf_apply_crot(s.psi, n, D, *c[1:])
            elif c[0] == "swap":
                qf.qf_apply_swap(s.psi, n, D, c[1], c[2])
            else:
                qf.qf_apply_mcx(s.psi, n, D, c[1], c[2])
        return s.psi
    if kind == "blocks":
        qf.qf_state_init(s.psi, n, D, None)
        for q in range(n):
            qf.qf_apply_1q(s.psi, n, D, q, s.h)
        for q0, B in s.blocks:
            qf.qf_apply_fused(s.psi, n, D, q0, case["span"], B)
        return s.psi
    if kind == "measure":
        out = [qf.qf_probs(s.psi, n, D)]
        out += [qf.qf_probs(s.psi, n, D, qudits=qs) for qs in _measured(case)]
        out += [qf.qf_expect(s.psi, n, D, t) for t in ([(0, "z")], _zterms(n), s.tables)]
        return out
    return [qf.qf_sample(s.psi, n, D, case["shots"], s.u),
            qf.qf_sample(s.psi, n, D, case["shots"], s.u, qudits=[0, n - 1])]


# ---------------------------------------------------------------------------
# Least work of a pass: every input read once, every output written once; the
# arithmetic of each gate as written (a rotation moves the levels it names).
# ---------------------------------------------------------------------------

def _gate_flops(op, dims):
    """Operations per amplitude of the register."""
    if op[0] in ("rx", "ry"):
        return 6.0 * 2 / dims[op[1]]
    if op[0] == "rz":
        return 6.0 * (op[2] + 1) / dims[op[1]]
    if op[0] in ("crx", "cry"):
        return 6.0 * 2 / dims[op[2]] * (dims[op[1]] - 1) / dims[op[1]]
    if op[0] == "crz":
        return 6.0 * (op[3] + 1) / dims[op[2]] * (dims[op[1]] - 1) / dims[op[1]]
    if op[0] == "h":
        return 8.0 * dims[op[1]]
    return 6.0 if op[0] in ("clock", "cz") else 0.0


def work(case):
    kind, esz = case["kind"], 8 if case["dtype"] == "c64" else 16
    if kind == "ragged":
        total = dict(bytes=0.0, flops=0.0)
        for d, n in _ragged_sizes(case):
            ops, p = _circuit(dict(case, dim=d, n=n), [1] * (case["layers"] * n))
            total["bytes"] += 8.0 * (2 * p + case["layers"] * n + 2)
            total["flops"] += 3.0 * d ** n * sum(_gate_flops(op, [d] * n) for op in ops)
        return total
    N, b, dims = _amps(case), case.get("batch", 1), _dims(case)
    if kind in ("forward", "gradient", "train"):
        ops, p = _circuit(case, [1] * max(1, case["layers"] * len(dims)))
        f = b * N * (sum(_gate_flops(op, dims) for op in ops) + 4.0)
        if kind == "forward":
            return dict(bytes=b * N * esz * 1.5 + 8.0 * p, flops=f)
        # forward, reverse walk of psi and of lambda, and one inner product per angle
        return dict(bytes=16.0 * b * p + 16.0 * b, flops=3.0 * f)
    if kind == "gates":
        ncalls = case["n"] * 2 + 18
        return dict(bytes=float(ncalls * 2 * N * esz), flops=8.0 * dims[0] * N * case["n"])
    if kind == "blocks":
        K, m = dims[0] ** case["span"], case["n"] - case["span"] + 1
        return dict(bytes=float(m * 2 * N * esz + m * K * K * esz),
                    flops=(4.0 if case["real"] else 8.0) * K * N * m)
    if kind == "measure":
        return dict(bytes=b * N * esz * 1.5, flops=b * N * 3.0)
    return dict(bytes=N * esz + 8.0 * N + 8.0 * case["shots"], flops=4.0 * N)


# ---------------------------------------------------------------------------
# The same in 64 bits with plain torch: registers as (batch, d_0, ..., d_{n-1})
# complex128 tensors, gates by their definitions.
# ---------------------------------------------------------------------------

def _view1(x, dims, q):
    return x.view(x.shape[0], math.prod(dims[:q]), dims[q], math.prod(dims[q + 1:]))


def _view2(x, dims, a, b):
    """(batch, H, d_lo, M, d_hi, L) for lo < hi, and whether a comes first."""
    lo, hi = min(a, b), max(a, b)
    return x.view(x.shape[0], math.prod(dims[:lo]), dims[lo], math.prod(dims[lo + 1:hi]), dims[hi],
                  math.prod(dims[hi + 1:])), a < b


def _col(v, ref):
    return v.reshape(-1, *([1] * (ref.dim() - 1)))


def _rotate(kind, x, axis, j, k, th):
    """exp(-i th S / 2) along axis of x in place; th: one angle per register."""
    if kind == "z":
        scale = math.sqrt(2.0 / (j * (j + 1)))
        up = _col(torch.exp(-0.5j * scale * th), x)
        dn = _col(torch.exp(0.5j * scale * j * th), x)
        x.narrow(axis, 0, j).mul_(up)
        x.narrow(axis, j, 1).mul_(dn)
        return
    a, b = x.narrow(axis, j, 1), x.narrow(axis, k, 1)
    c = _col(torch.cos(th / 2).to(torch.complex128), x)
    s = _col(torch.sin(th / 2).to(torch.complex128), x)
    old = a.clone()
    if kind == "x":
        a.mul_(c).sub_(1j * s * b)
        b.mul_(c).sub_(1j * s * old)
    else:
        a.mul_(c).sub_(s * b)
        b.mul_(c).add_(s * old)


def _generator_im(kind, lam, psi, axis, j, k):
    """Im <lam| S |psi> per register."""
    def dot(u, v):
        r = (u.conj() * v).reshape(u.shape[0], -1).sum(dim=1)
        return r
    if kind == "z":
        scale = math.sqrt(2.0 / (j * (j + 1)))
        r = dot(lam.narrow(axis, 0, j), psi.narrow(axis, 0, j)) - \
            j * dot(lam.narrow(axis, j, 1), psi.narrow(axis, j, 1))
        return scale * r.imag
    lj, lk = lam.narrow(axis, j, 1), lam.narrow(axis, k, 1)
    pj, pk = psi.narrow(axis, j, 1), psi.narrow(axis, k, 1)
    if kind == "x":
        return (dot(lj, pk) + dot(lk, pj)).imag
    return (-1j * dot(lj, pk) + 1j * dot(lk, pj)).imag


def _permute_levels(v, caxis, taxis, dt, amount):
    """x_t -> x_t + amount(x_c) in place."""
    for m in range(v.shape[caxis]):
        s = amount(m) % dt
        if s:
            w = v.select(caxis, m)
            ax = taxis - (1 if caxis < taxis else 0)
            w.copy_(torch.roll(w, s, dims=ax))


def _apply(op, x, dims, theta, inverse=False):
    """One gate in place; theta: (batch, angles) tensor."""
    sgn = -1.0 if inverse else 1.0
    kind = op[0]
    if kind in ("rx", "ry", "rz"):
        v = _view1(x, dims, op[1])
        k = op[3] if kind != "rz" else 0
        _rotate(kind[1], v, 2, op[2], k, sgn * theta[:, op[-1]])
    elif kind in ("crx", "cry", "crz"):
        v, first = _view2(x, dims, op[1], op[2])
        cax, tax = (2, 4) if first else (4, 2)
        for m in range(1, dims[op[1]]):
            w = v.select(cax, m)
            k = op[4] if kind != "crz" else 0
            _rotate(kind[2], w, tax - (1 if cax < tax else 0), op[3], k, sgn * m * theta[:, op[-1]])
    elif kind == "h":
        d = dims[op[1]]
        k = torch.arange(d, device=x.device, dtype=torch.float64)
        U = torch.exp(sgn * 2j * math.pi / d * torch.outer(k, k)) / math.sqrt(d)
        _dense(x, dims, op[1], 1, U)
    elif kind == "clock":
        d = dims[op[1]]
        a = op[2] if torch.is_tensor(op[2]) else torch.full((1,), float(op[2]), device=x.device, dtype=torch.float64)
        k = torch.arange(d, device=x.device, dtype=torch.float64)
        ph = torch.exp(sgn * 2j * math.pi / d * (a.reshape(-1, 1) * k))
        _view1(x, dims, op[1]).mul_(ph.reshape(-1, 1, d, 1))
    elif kind == "csum":
        v, first = _view2(x, dims, op[1], op[2])
        cax, tax = (2, 4) if first else (4, 2)
        _permute_levels(v, cax, tax, dims[op[2]], lambda m: int(sgn) * m)
    elif kind == "cz":
        v, first = _view2(x, dims, op[1], op[2])
        dc, dt = dims[op[1]], dims[op[2]]
        c = torch.arange(dc, device=x.device, dtype=torch.float64)
        t = torch.arange(dt, device=x.device, dtype=torch.float64)
        ph = torch.exp(sgn * 2j * math.pi / dt * torch.outer(c, t))
        ph = ph if first else ph.T
        v.mul_(ph.reshape(1, 1, ph.shape[0], 1, ph.shape[1], 1))
    else:
        raise ValueError(kind)


def _dense(x, dims, q0, span, U):
    K = math.prod(dims[q0:q0 + span])
    v = x.view(x.shape[0], math.prod(dims[:q0]), K, math.prod(dims[q0 + span:]))
    y = torch.zeros_like(v)
    if K <= 16:
        for a in range(K):
            for b in range(K):
                y[:, :, a].add_(v[:, :, b] * U[a, b])
    else:
        t = v.movedim(2, -1).reshape(-1, K)
        y = (t @ U.T.contiguous()).view(v.shape[0], v.shape[1], v.shape[3], K).movedim(-1, 2)
    v.copy_(y)


def _gradient(op, psi, lam, dims, theta):
    """d Re<O> / d angle of a rotation that psi and lam have just passed."""
    kind = op[0]
    if kind in ("rx", "ry", "rz"):
        k = op[3] if kind != "rz" else 0
        return _generator_im(kind[1], _view1(lam, dims, op[1]), _view1(psi, dims, op[1]), 2, op[2], k)
    v, first = _view2(psi, dims, op[1], op[2])
    w, _ = _view2(lam, dims, op[1], op[2])
    cax, tax = (2, 4) if first else (4, 2)
    out = 0
    for m in range(1, dims[op[1]]):
        k = op[4] if kind != "crz" else 0
        out = out + m * _generator_im(kind[2], w.select(cax, m), v.select(cax, m), tax - (1 if cax < tax else 0),
                                      op[3], k)
    return out


def _diagonal(dims, terms, dev):
    """sum of one-qudit diagonal tables over the register."""
    n = len(dims)
    out = torch.zeros(dims, dtype=torch.complex128, device=dev)
    for q, t in terms:
        if isinstance(t, str):
            k = torch.arange(dims[q], device=dev, dtype=torch.float64)
            t = torch.exp(2j * math.pi / dims[q] * k)
        else:
            t = torch.tensor(np.asarray(t), dtype=torch.complex128, device=dev)
        out += t.reshape([dims[q] if i == q else 1 for i in range(n)])
    return out.reshape(1, -1)


def _expect64(psi, dims, terms):
    e = (psi.abs().square() * _diagonal(dims, terms, psi.device)).sum(dim=1)
    return torch.view_as_real(e).reshape(-1)


def _start(case, batch, dev):
    dims = _dims(case)
    x = torch.zeros((batch, math.prod(dims)), dtype=torch.complex128, device=dev)
    x[:, 0] = 1
    return x, dims


def _run64(case, ops, theta, want_grad, dev):
    """Final state, <sum_i Z_i> and, if asked, the gradient (batch x angles)."""
    psi, dims = _start(case, theta.shape[0], dev)
    for op in ops:
        _apply(op, psi, dims, theta)
    terms = _zterms(len(dims))
    loss = _expect64(psi, dims, terms)
    if not want_grad:
        return psi, loss, None
    lam = psi * _diagonal(dims, terms, dev).real
    grad = torch.zeros(theta.shape, dtype=torch.float64, device=dev)
    for op in reversed(ops):
        if op[0][0] in "rc" and op[0] not in ("clock", "csum", "cz"):
            grad[:, op[-1]] += _gradient(op, psi, lam, dims, theta)
        _apply(op, psi, dims, theta, inverse=True)
        _apply(op, lam, dims, theta, inverse=True)
    return psi, loss, grad


def _marginal64(psi, dims, qs):
    n = len(dims)
    p = psi.abs().square().reshape([psi.shape[0]] + dims)
    rest = [q + 1 for q in range(n) if q not in qs]
    if rest:
        p = p.sum(dim=rest)
    kept = sorted(qs)
    return p.permute([0] + [kept.index(q) + 1 for q in qs]).reshape(-1)


def exact(case, seed):
    dev, kind = "cuda", case["kind"]
    if kind in ("forward", "gradient", "train"):
        ops, _, theta = _problem(case, seed)
        th = torch.tensor(theta, dtype=torch.float64, device=dev)
        psi, loss, grad = _run64(case, ops, th, kind != "forward", dev)
        if kind == "forward":
            return [psi.reshape(-1), psi.abs().square().reshape(-1), loss]
        if kind == "gradient":
            return [loss, grad.reshape(-1)]
        return [loss.reshape(-1, 2)[:, 0], grad]
    if kind == "ragged":
        circuits = _ragged_circuits(case, seed)
        groups = {}
        for c in circuits:
            groups.setdefault((c.dim, c.n), []).append(c)
        losses, grads = [], []
        for (d, n), cs in sorted(groups.items()):
            th = torch.tensor(np.stack([c.theta for c in cs]), dtype=torch.float64, device=dev)
            ck = torch.tensor(np.stack([c.clocks for c in cs]), dtype=torch.float64, device=dev)
            ops, i = [], 0
            for op in cs[0].ops:
                if op[0] == "clock":
                    op, i = ("clock", op[1], ck[:, i]), i + 1
                ops.append(op)
            _, loss, grad = _run64(dict(case, dim=d, n=n), ops, th, True, dev)
            losses.append(loss.reshape(-1, 2))
            grads.append(grad)
        return losses + grads
    if kind in ("gates", "blocks"):
        psi, dims = _start(case, 1, dev)
        if kind == "blocks":
            for q in range(case["n"]):
                _apply(("h", q), psi, dims, None)
            for q0, B in _blocks(case, seed):
                # the block as the program holds it, in the state's precision
                Bt = torch.tensor(B, dtype=_torch_dtype(case), device=dev).to(torch.complex128)
                _dense(psi, dims, q0, case["span"], Bt)
            return psi.reshape(-1)
        for c in _gate_list(case, seed):
            if c[0] == "1q":
                _dense(psi, dims, c[1], 1, torch.tensor(c[2], device=dev))
            elif c[0] == "ctrl":
                v, first = _view2(psi, dims, c[1], c[2])
                cax, tax = (2, 4) if first else (4, 2)
                _permute_levels(v, cax, tax, dims[c[2]], lambda m: c[3][m])
            elif c[0] == "diag":
                v, first = _view2(psi, dims, *c[1])
                w = torch.tensor(c[2], device=dev).reshape(dims[c[1][0]], dims[c[1][1]])
                w = w if first else w.T
                v.mul_(w.reshape(1, 1, w.shape[0], 1, w.shape[1], 1))
            elif c[0] in ("rot", "crot"):
                th = torch.tensor([[c[-1]]], dtype=torch.float64, device=dev)
                if c[0] == "rot":
                    op = (c[1], c[2], c[3], 0) if c[1] == "rz" else (c[1], c[2], c[3], c[4], 0)
                else:
                    op = (c[1], c[2], c[3], c[4], 0) if c[1] == "crz" else (c[1], c[2], c[3], c[4], c[5], 0)
                _apply(op, psi, dims, th)
            elif c[0] == "swap":
                v, _ = _view2(psi, dims, c[1], c[2])
                v.copy_(v.transpose(2, 4).clone())
            else:
                full = psi.view([1] + dims)
                (a, b), t = c[1], c[2]
                for xa in range(1, dims[a]):
                    for xb in range(1, dims[b]):
                        idx = [slice(None)] * (len(dims) + 1)
                        idx[a + 1], idx[b + 1] = slice(xa, xa + 1), slice(xb, xb + 1)
                        w = full[tuple(idx)]
                        w.copy_(torch.roll(w, (xa * xb) % dims[t], dims=t + 1))
        return psi.reshape(-1)
    dims = _dims(case)
    psi = _random_state(case, seed).to(torch.complex128).reshape(case.get("batch", 1), -1)
    if kind == "measure":
        out = [psi.abs().square().reshape(-1)]
        out += [_marginal64(psi, dims, qs) for qs in _measured(case)]
        out += [_expect64(psi, dims, t) for t in ([(0, "z")], _zterms(case["n"]), _tables(case, seed))]
        return out
    return None  # shots are whole numbers: they have to stay equal
