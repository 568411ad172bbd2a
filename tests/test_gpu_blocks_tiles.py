"""Dense blocks of 32 <= K <= 128 in complex64 on both sides of the rule for the tiles: up
to 4096 fibres in tiles of 16, above in tiles of 32 (K <= 48) or 64, every row-block count,
remainders, every position of the block; and infinite amplitudes in large registers."""
import numpy as np
import pytest

import qf_inputs as qi
from tests.gpu_helpers import to_dev, to_np

pytestmark = pytest.mark.gpu

# dims, span, q0, batch: 4096 and 4097 fibres, then more with a remainder of 64 or 32
CASES = [([5, 7], 2, 0, 4096), ([5, 7], 2, 0, 4097), ([7, 7], 2, 0, 4096), ([7, 7], 2, 0, 4097),
         ([2] * 17, 5, 3, 1), ([2] * 18, 5, 13, 1), ([6] * 7, 2, 2, 1), ([6, 7] + [3] * 8, 2, 0, 1),
         ([7] * 7, 2, 5, 1), ([3, 7, 8] + [5] * 5, 2, 1, 1), ([5, 13, 3, 11, 13, 2, 5], 2, 0, 1),
         ([3] * 12, 4, 0, 1), ([9] * 6, 2, 1, 1), ([10] * 6, 2, 4, 1), ([10] * 6, 2, 0, 1), ([11, 11, 5, 7, 11, 13], 2, 0, 1),
         ([5] * 9, 3, 2, 1), ([2] * 20, 7, 0, 1), ([2] * 20, 7, 13, 1)]


def _case(dims, span, q0, batch, rng):
    n, N = len(dims), int(np.prod(dims))
    K = int(np.prod(dims[q0:q0 + span]))
    H, L = batch * int(np.prod(dims[:q0])), int(np.prod(dims[q0 + span:]))
    x = rng.standard_normal((H, K, L), dtype=np.float32) + 1j * rng.standard_normal((H, K, L), dtype=np.float32)
    return n, K, N, x.astype(np.complex64)


def _run(dims, span, q0, U, x):
    import paper_2409_17716_amd as qf
    dim = dims[0] if len(set(dims)) == 1 else dims
    t = to_dev(x.reshape(-1), "c64")
    qf.Plan(dim, len(dims), [("u", q0, span, U.astype(np.complex128))], 0, "c64").forward(t, np.zeros(0))
    return to_np(t).reshape(x.shape)


@pytest.mark.parametrize("dims,span,q0,batch", CASES)
@pytest.mark.parametrize("real", [False, True])
def test_tiles(dims, span, q0, batch, real):
    rng = np.random.default_rng(53)
    n, K, N, x = _case(dims, span, q0, batch, rng)
    U = np.linalg.qr(rng.standard_normal((K, K)))[0] if real else qi.random_unitary(K, rng)
    U = U.astype(np.complex64)
    want = np.matmul(U.astype(np.complex128), x)
    err = np.abs(_run(dims, span, q0, U, x) - want)
    # each element: 2 K products of norm-1 rows, each partial sum rounded by 2^-24 of it
    assert np.all(err <= (2 * K + 8) * 2.0 ** -24 * 2 * np.linalg.norm(x, axis=1, keepdims=True))
    # and in the mean as few roundings as the sums have parts
    assert np.sqrt(np.mean(err ** 2) / np.mean(np.abs(want) ** 2)) <= (1 + (K + 31) // 32 / 2) * 2.0 ** -24


@pytest.mark.parametrize("dims,span,q0", [([6] * 7, 2, 2), ([7] * 7, 2, 5), ([10] * 6, 2, 0), ([2] * 20, 7, 13)])
def test_infinite_amplitudes_in_large_registers(dims, span, q0):
    rng = np.random.default_rng(59)
    n, K, N, x = _case(dims, span, q0, 1, rng)
    U = qi.random_unitary(K, rng).astype(np.complex64)
    H, L = x.shape[0], x.shape[2]
    flat = [0, H * L // 2 + 1, H * L - 1]  # fibres of the first, a middle and the last tile
    for i, f in enumerate(flat):
        x[f // L, (5 * i) % K, f % L] = complex(np.inf, 0.5)
    got = _run(dims, span, q0, U, x)
    clean = np.ones(H * L, dtype=bool)
    clean[flat] = False
    g = np.moveaxis(got, 1, 2).reshape(H * L, K)
    with np.errstate(invalid="ignore"):
        want = np.moveaxis(np.matmul(U.astype(np.complex128), x), 1, 2).reshape(H * L, K)
    norm = np.linalg.norm(np.moveaxis(x, 1, 2).reshape(H * L, K)[clean], axis=1, keepdims=True)
    assert np.all(np.abs(g - want)[clean] <= (2 * K + 8) * 2.0 ** -24 * 2 * norm)
    assert not np.isfinite(g[flat]).any()
