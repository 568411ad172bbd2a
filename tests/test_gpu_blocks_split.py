"""Dense blocks of 32 <= K <= 128 on the bf16 matrix cores (operands as three bf16
parts): sizes at the edges of the row and k blocks, tiles with a remainder of
fibres, every position of the block, real and complex blocks, several registers.

Tolerance: every real component of a result is a sum of 2 K products in FP32.
With rows of norm 1 (unitary blocks) the products' magnitudes sum to at most
sqrt(2) |x| for the fibre x, each partial sum rounds by 2^-24 of it, and the
dropped partial products and the operands' rounding stay below 8 * 2^-24."""
import numpy as np
import pytest

import qf_inputs as qi
from tests.gpu_helpers import to_dev, to_np

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dims,span", [([2] * 7, 5), ([6] * 3, 2), ([7] * 4, 2), ([8, 6, 3, 2], 2), ([3] * 6, 4),
                                       ([5, 13, 2, 3], 2), ([4] * 5, 3), ([10] * 4, 2), ([5] * 5, 3), ([7, 16, 3], 2),
                                       ([2] * 9, 7), ([11, 11, 2], 2)])
@pytest.mark.parametrize("real", [False, True])
def test_block_parts(dims, span, real):
    import paper_2409_17716_amd as qf
    n, batch = len(dims), 2
    N = int(np.prod(dims))
    rng = np.random.default_rng(17)
    psi = rng.standard_normal((batch, N)) + 1j * rng.standard_normal((batch, N))
    psi = (psi / np.linalg.norm(psi)).astype(np.complex64)
    uniform = len(set(dims)) == 1
    for q0 in range(n - span + 1):
        K = int(np.prod(dims[q0:q0 + span]))
        if not 32 <= K <= 128:
            continue
        U = np.linalg.qr(rng.standard_normal((K, K)))[0] if real else qi.random_unitary(K, rng)
        U = U.astype(np.complex64)
        p = qf.Plan(dims[0] if uniform else dims, n, [("u", q0, span, U.astype(np.complex128))], 0, "c64")
        t = to_dev(psi.reshape(-1), "c64")
        p.forward(t, np.zeros(0))
        H, L = int(np.prod(dims[:q0])), int(np.prod(dims[q0 + span:]))
        x = psi.astype(np.complex128).reshape(batch * H, K, L)
        want = np.matmul(U.astype(np.complex128), x)
        err = np.abs(to_np(t).reshape(want.shape) - want)
        bound = (2 * K + 8) * 2.0 ** -24 * 2 * np.linalg.norm(x, axis=1, keepdims=True)
        assert np.all(err <= bound), (q0, K, float((err / bound).max()))


@pytest.mark.parametrize("dims,span,q0", [([6] * 3, 2, 0), ([6] * 4, 2, 2), ([7] * 4, 2, 1), ([10] * 4, 2, 0), ([2] * 9, 7, 1)])
@pytest.mark.parametrize("real", [False, True])
def test_infinities_nan_and_largest_values(dims, span, q0, real):
    """Infinite, NaN and near-overflow amplitudes (above the largest bf16 value) give what
    FP32 products of the parts give; every other fibre, of the same tile too, is as before."""
    import paper_2409_17716_amd as qf
    n = len(dims)
    K, H, L = int(np.prod(dims[q0:q0 + span])), int(np.prod(dims[:q0])), int(np.prod(dims[q0 + span:]))
    rng = np.random.default_rng(23)
    U = np.linalg.qr(rng.standard_normal((K, K)))[0] if real else qi.random_unitary(K, rng)
    U = U.astype(np.complex64).astype(np.complex128)
    x = (rng.standard_normal((H, K, L)) + 1j * rng.standard_normal((H, K, L))).astype(np.complex64)
    odd = [complex(np.inf, 1), complex(1, -np.inf), complex(np.nan, 1), complex(3.395e38, 0)]
    for i, v in enumerate(odd):
        f = (i * 5) % (H * L)
        x[f // L, :, f % L] = 0.25 if i < 3 else 0.0
        x[f // L, (7 * i) % K, f % L] = v
    t = to_dev(x.reshape(-1), "c64")
    qf.Plan(dims[0], n, [("u", q0, span, U)], 0, "c64").forward(t, np.zeros(0))
    got = to_np(t).reshape(H, K, L)
    xr, xi = x.real.astype(np.float64), x.imag.astype(np.float64)
    with np.errstate(invalid="ignore"):
        wr = np.matmul(U.real, xr) - (0.0 if real else np.matmul(U.imag, xi))
        wi = np.matmul(U.real, xi) + (0.0 if real else np.matmul(U.imag, xr))
        norm = np.sqrt((xr ** 2 + xi ** 2).sum(axis=1, keepdims=True))
        for g, w in ((got.real, wr), (got.imag, wi)):
            assert np.array_equal(np.isnan(g), np.isnan(w))
            inf = np.isinf(w)
            assert np.array_equal(np.isinf(g), inf) and np.array_equal(g[inf], w[inf])
            ok = np.isfinite(w)
            bound = np.where(np.isfinite(norm), norm, 1.0) * (2 * K + 8) * 2.0 ** -24 * 2 + 0 * w
            # a component that an odd entry does not reach sums the fibre's other entries
            assert np.all(np.abs(g - w)[ok] <= np.maximum(bound, 2.0 ** -20 * K)[ok])
