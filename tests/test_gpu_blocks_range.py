"""Dense blocks of 32 <= K <= 128 in complex64 (bf16 matrix cores on three-part
operands): blocks with entries that have no such parts, amplitudes and entries near the
smallest numbers, and the precision of the products."""
import numpy as np
import pytest

import qf_inputs as qi
from tests.gpu_helpers import to_dev, to_np

pytestmark = pytest.mark.gpu

SHAPES = [([2] * 8, 5, 1), ([6] * 4, 2, 0), ([7] * 4, 2, 2), ([10] * 4, 2, 1), ([2] * 9, 7, 0)]


def _split(dims, span, q0):
    return int(np.prod(dims[:q0])), int(np.prod(dims[q0:q0 + span])), int(np.prod(dims[q0 + span:]))


def _parts(U, x, real):
    """Real and imaginary parts of U x, the real products summed by themselves."""
    xr, xi = x.real.astype(np.float64), x.imag.astype(np.float64)
    wr = np.matmul(U.real, xr) - (0.0 if real else np.matmul(U.imag, xi))
    wi = np.matmul(U.real, xi) + (0.0 if real else np.matmul(U.imag, xr))
    return wr, wi


def _apply(dims, span, q0, U, x):
    import paper_2409_17716_amd as qf
    t = to_dev(x.reshape(-1), "c64")
    qf.qf_apply_fused(t, len(dims), dims[0], q0, span, to_dev(U.reshape(-1), "c64"))
    return to_np(t).reshape(x.shape)


@pytest.mark.parametrize("dims,span,q0", SHAPES)
def test_block_entries_without_parts(dims, span, q0):
    """Infinite, NaN, and largest entries (above the largest bf16 value, and below it at a
    size whose sums could leave FP32 where the result does not): what FP32 products give."""
    H, K, L = _split(dims, span, q0)
    rng = np.random.default_rng(41)
    x = (rng.standard_normal((H, K, L)) + 1j * rng.standard_normal((H, K, L))).astype(np.complex64) * 0.01
    for v in (complex(np.inf, 0.5), complex(0.5, -np.inf), complex(np.nan, 1), 3.395e38, complex(0, -3.395e38), 2e38,
              1e30):
        U = qi.random_unitary(K, rng).astype(np.complex64)
        U[K // 3] = 0.25
        U[K // 3, K - 1] = v
        got = _apply(dims, span, q0, U, x)
        with np.errstate(invalid="ignore"):
            want = _parts(U.astype(np.complex128), x, False)
            for g, w in zip((got.real, got.imag), want):
                assert np.array_equal(np.isnan(g), np.isnan(w)), v
                inf = np.isinf(w)
                assert np.array_equal(np.isinf(g), inf) and np.array_equal(g[inf], w[inf]), v
                ok = np.isfinite(w)
                # a sum of 2 K products, each partial sum rounded by 2^-24 of at most the
                # row's largest magnitudes times the fibre's
                size = np.where(np.isfinite(U), np.abs(U).astype(np.float64), 0).max(axis=1)[None, :, None] * \
                    np.abs(x).astype(np.float64).sum(axis=1, keepdims=True) * np.ones(w.shape)
                assert np.all((np.abs(g - w) <= 4 * K * 2.0 ** -24 * size)[ok]), v


@pytest.mark.parametrize("dims,span,q0", SHAPES)
@pytest.mark.parametrize("ex,eb", [(-100, 0), (-117, 0), (-122, 0), (-60, -60), (0, -117), (20, 20), (47, 0),
                                   (50, 0), (57, 0), (0, 20), (0, 26)])
def test_scales(dims, span, q0, ex, eb):
    """Amplitudes about 2^ex and a block of 2^eb times a unitary: results keep FP32's
    relative precision as long as they are normal numbers themselves (each of the fibre's
    amplitudes and the block's entries is taken whole, a result rounds once more)."""
    H, K, L = _split(dims, span, q0)
    rng = np.random.default_rng(43)
    x = ((rng.standard_normal((H, K, L)) + 1j * rng.standard_normal((H, K, L))) * 2.0 ** ex).astype(np.complex64)
    U = (qi.random_unitary(K, rng) * 2.0 ** eb).astype(np.complex64)
    got = _apply(dims, span, q0, U, x)
    wr, wi = _parts(U.astype(np.complex128), x, False)
    err = np.sqrt(np.mean((got.real - wr) ** 2 + (got.imag - wi) ** 2) / np.mean(wr ** 2 + wi ** 2))
    # K / 4 to 2 K additions in FP32, each rounding by at most 2^-24 of a partial sum,
    # independently: sqrt(2 K / 3) 2^-24
    assert err <= np.sqrt(2 * K / 3) * 2.0 ** -24, (err, ex, eb)


@pytest.mark.parametrize("dims,span,q0", SHAPES)
@pytest.mark.parametrize("decades", [8, 30, 60])
def test_rows_of_different_sizes(dims, span, q0, decades):
    """Rows of a block over many powers of two, smallest and largest side by side: every
    row keeps FP32's relative precision (test_scales' bound)."""
    H, K, L = _split(dims, span, q0)
    rng = np.random.default_rng(45)
    x = (rng.standard_normal((H, K, L)) + 1j * rng.standard_normal((H, K, L))).astype(np.complex64)
    U = (qi.random_unitary(K, rng) * 10.0 ** rng.uniform(-decades / 2, decades / 2, size=(K, 1))).astype(np.complex64)
    got = _apply(dims, span, q0, U, x)
    wr, wi = _parts(U.astype(np.complex128), x, False)
    err = np.sqrt(((got.real - wr) ** 2 + (got.imag - wi) ** 2).mean(axis=(0, 2)) / (wr ** 2 + wi ** 2).mean(axis=(0, 2)))
    assert np.all(err <= np.sqrt(2 * K / 3) * 2.0 ** -24), (err.max(), K)


def _fp32(U, x):
    """U x for one entry per row, each part by FP32 products and one FP32 addition."""
    K = U.shape[0]
    col = np.abs(U).argmax(axis=1)
    u = U[np.arange(K), col][None, :, None]
    v = x[:, col, :]
    re = (u.real * v.real) - (u.imag * v.imag)
    im = (u.real * v.imag) + (u.imag * v.real)
    assert re.dtype == np.float32
    return re, im


@pytest.mark.parametrize("dims,span,q0", [([2] * 14, 5, 4), ([6] * 6, 2, 1), ([7] * 5, 2, 2), ([10] * 4, 2, 1),
                                          ([2] * 14, 7, 0)])
@pytest.mark.parametrize("real", [False, True])
def test_precision_of_the_products(dims, span, q0, real):
    import paper_2409_17716_amd as qf
    H, K, L = _split(dims, span, q0)
    rng = np.random.default_rng(47)
    x = (rng.standard_normal((H, K, L)) + 1j * rng.standard_normal((H, K, L))).astype(np.complex64)

    def run(U):
        t = to_dev(x.reshape(-1), "c64")
        qf.Plan(dims[0], len(dims), [("u", q0, span, U.astype(np.complex128))], 0, "c64").forward(t, np.zeros(0))
        return to_np(t).reshape(x.shape)

    def rms(g, U):
        w = np.matmul(U.astype(np.complex128), x.astype(np.complex128))
        return np.sqrt(np.mean(np.abs(g - w) ** 2) / np.mean(np.abs(w) ** 2))
    # a dense block: the sum of the leading parts' products rounds once for 32 rows (2^-24
    # of a partial sum at most), the two additions that join the sums round by 2^-25; with
    # the low parts' products left out the error is 1e-6 and more
    U = np.linalg.qr(rng.standard_normal((K, K)))[0].astype(np.complex64) if real else \
        qi.random_unitary(K, rng).astype(np.complex64)
    assert rms(run(U), U) <= (1 + (K + 31) // 32 / 2) * 2.0 ** -24
    # a permutation moves the amplitudes: hi + mid + lo is the amplitude itself
    perm = rng.permutation(K)
    P = np.eye(K)[perm].astype(np.complex64)
    assert np.array_equal(run(P), x[:, perm, :].astype(np.complex128))
    # one entry per row: no further off than FP32 products and their sum (the two errors
    # are means over at least 10^4 results, known to about 1%)
    d = rng.standard_normal(K) if real else np.exp(2j * np.pi * rng.random(K))
    D = (np.eye(K)[perm] * d).astype(np.complex64)
    re, im = _fp32(D, x)
    assert rms(run(D), D) <= 1.02 * rms(re.astype(np.float64) + 1j * im, D)
