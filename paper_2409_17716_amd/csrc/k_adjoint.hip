// Adjoint-method kernels.  For a one-qudit step U on axis q, one pass over the
// fibres of psi and lam (both taken just after U in the forward order):
//   * accumulates the D x D matrix M = sum_fibres psi_f lam_f^dagger in FP64
//     (every rotation folded into U gets its derivative from M on the host),
//   * un-applies U on both states: psi_f <- W psi_f, lam_f <- W lam_f with
//     W = U^dagger (passed in by the host).
// The reduction is deterministic: fixed per-workgroup tree, then a fixed-order
// sum over workgroups.
#include <algorithm>
#include <type_traits>

#include "qf_internal.h"

namespace qf {
namespace {

constexpr int kFB = 128;  // fibres (= lanes) per workgroup

template <typename T, int D>
struct MatArgA {
    cplx<T> m[D * D];
};

// Un-applies one fused run (W: its inverse) on psi and lam along one axis and sums
// M = sum_f psi_f lam_f^dagger before it in FP64; a row of D * D reals per
// workgroup holds M's anti-Hermitian part (a * D + c: its real part for a < c, its
// imaginary part for a >= c).  A shift merged into the run (it came after the run)
// is undone first, in the addresses of the loads.  Workgroups walk their
// register's blocks of kFB fibres with their part of M in registers; the rows of
// many runs are reduced in one launch (a launch per run took 36 x 8.6 us of the
// 2.1 ms of a 1.7 M-amplitude mixed register's gradient).
template <typename T, int D>
__global__ __launch_bounds__(kFB) void k_adj_axis(cplx<T>* __restrict__ psi, cplx<T>* __restrict__ lam,
                                                  uint32_t nfib_reg, uint32_t blocks_per_reg, uint32_t wgs_per_reg,
                                                  uint32_t N, uint32_t L, FastDiv divL, MatArgA<T, D> W,
                                                  ShiftArg sh, double* __restrict__ partial) {
    __shared__ cplx<T> sp[D][kFB];
    __shared__ cplx<T> sl[D][kFB];
    constexpr int E = D * D;
    constexpr int P = E <= kFB ? kFB / E : 1;     // parts per entry
    constexpr int NE = E <= kFB ? 1 : (E + kFB - 1) / kFB;  // entries per lane
    __shared__ double red[2][P * E];
    const uint32_t b = blockIdx.x / wgs_per_reg;
    const int e0 = E <= kFB ? threadIdx.x % E : threadIdx.x;
    const int part = E <= kFB ? threadIdx.x / E : 0;
    double ar[NE], ai[NE];
#pragma unroll
    for (int j = 0; j < NE; ++j) ar[j] = ai[j] = 0.0;
    for (uint32_t blk = blockIdx.x - b * wgs_per_reg; blk < blocks_per_reg; blk += wgs_per_reg) {
        const uint32_t f = blk * kFB + threadIdx.x;
        if (f < nfib_reg) {
            const uint32_t h = divL.div(f);
            const uint32_t l = f - h * L;
            const uint32_t base = b * N + h * (uint32_t(D) * L) + l;
            const uint32_t s = sh.template amount<D>(base);
            cplx<T> vp[D], vl[D];
#pragma unroll
            for (int d = 0; d < D; ++d) {
                const uint32_t o = base + wrap_add<D>(uint32_t(d), s) * L;
                vp[d] = psi[o];
                vl[d] = lam[o];
            }
#pragma unroll
            for (int d = 0; d < D; ++d) {
                sp[d][threadIdx.x] = vp[d];
                sl[d][threadIdx.x] = vl[d];
            }
            cplx<T> wp[D], wl[D];
#pragma unroll
            for (int a = 0; a < D; ++a) {
                wp[a] = cmake<T>(0, 0);
                wl[a] = cmake<T>(0, 0);
#pragma unroll
                for (int c = 0; c < D; ++c) {
                    cmac(wp[a], W.m[a * D + c], vp[c]);
                    cmac(wl[a], W.m[a * D + c], vl[c]);
                }
            }
#pragma unroll
            for (int d = 0; d < D; ++d) {
                psi[base + uint32_t(d) * L] = wp[d];
                lam[base + uint32_t(d) * L] = wl[d];
            }
        } else {
#pragma unroll
            for (int d = 0; d < D; ++d) {
                sp[d][threadIdx.x] = cmake<T>(0, 0);
                sl[d][threadIdx.x] = cmake<T>(0, 0);
            }
        }
        __syncthreads();
        // M[a][c] = sum_i psi_i[a] conj(lam_i[c]); entry e = a * D + c
#pragma unroll
        for (int j = 0; j < NE; ++j) {
            const int e = e0 + j * kFB;
            if (part >= P || e >= E) continue;
            const int a = e / D, c = e % D;
#pragma unroll 4
            for (int i = part; i < kFB; i += P) {
                const cplx<T> x = sp[a][i];
                const cplx<T> y = sl[c][i];
                ar[j] += double(x.re) * double(y.re) + double(x.im) * double(y.im);
                ai[j] += double(x.im) * double(y.re) - double(x.re) * double(y.im);
            }
        }
        __syncthreads();
    }
#pragma unroll
    for (int j = 0; j < NE; ++j) {
        const int e = e0 + j * kFB;
        if (part >= P || e >= E) continue;
        red[0][part * E + e] = ar[j];
        red[1][part * E + e] = ai[j];
    }
    __syncthreads();
    for (int e = threadIdx.x; e < E; e += kFB) {
        const int a = e / D, c = e % D;
        const int k = a < c ? 0 : 1;
        double x = 0.0, y = 0.0;
        for (int p = 0; p < P; ++p) {
            x += red[k][p * E + e];
            y += red[k][p * E + c * D + a];
        }
        partial[size_t(blockIdx.x) * E + e] = a < c ? 0.5 * (x - y) : 0.5 * (x + y);
    }
}

// The rows of up to kAdjRows runs, summed in a fixed order (lane = entry of one of
// 256 / E rows at a time, eight rows in flight) by one workgroup per run and register
// and written as the complex anti-Hermitian matrix.  Runs of more rows than a workgroup
// reads in four turns (AdjRows::chunk) are first summed by chunks (CHUNKS: blockIdx.y),
// each chunk's sum replacing its first row, which no other workgroup reads.
constexpr int kAdjRows = 64;

struct AdjRowsArg {
    AdjRows run[kAdjRows];
};

template <bool CHUNKS>
__global__ __launch_bounds__(256) void k_adj_reduce(double* __restrict__ partial, AdjRowsArg a, uint32_t batch,
                                                    uint32_t nslots, uint32_t slot_elems, double* __restrict__ out) {
    __shared__ double red[256];
    __shared__ double sum[256];
    const uint32_t r = blockIdx.x / batch, b = blockIdx.x - r * batch;
    const uint32_t D = a.run[r].D, rows = a.run[r].rows, chunk = a.run[r].chunk, E = D * D;
    const uint32_t first = CHUNKS ? blockIdx.y * chunk : 0u;
    if (CHUNKS && (chunk == rows || first >= rows)) return;
    const uint32_t last = CHUNKS ? min(rows, first + chunk) : rows;
    const uint32_t step = CHUNKS || chunk == rows ? 1u : chunk;
    double* p = partial + a.run[r].off + size_t(b) * rows * E;
    const uint32_t G = 256 / E, gr = threadIdx.x / E, e = threadIdx.x - gr * E;
    constexpr uint32_t kU = 8;
    double acc = 0.0;
    if (gr < G) {
        uint32_t i = first + gr * step;
        for (; i + (kU - 1) * G * step < last; i += kU * G * step) {
            double x[kU];
#pragma unroll
            for (uint32_t u = 0; u < kU; ++u) x[u] = p[size_t(i + u * G * step) * E + e];
#pragma unroll
            for (uint32_t u = 0; u < kU; ++u) acc += x[u];
        }
        for (; i < last; i += G * step) acc += p[size_t(i) * E + e];
    }
    red[threadIdx.x] = acc;
    __syncthreads();
    if (threadIdx.x < E) {
        double t = 0.0;
        for (uint32_t q = 0; q < G; ++q) t += red[q * E + threadIdx.x];
        if (CHUNKS)
            p[size_t(first) * E + threadIdx.x] = t;
        else
            sum[threadIdx.x] = t;
    }
    if (CHUNKS) return;
    __syncthreads();
    if (threadIdx.x < E) {
        const uint32_t x = threadIdx.x / D, y = threadIdx.x - x * D;
        double* o = out + ((size_t(b) * nslots + a.run[r].slot) * slot_elems + threadIdx.x) * 2;
        o[0] = x == y ? 0.0 : x < y ? sum[x * D + y] : -sum[y * D + x];
        o[1] = x < y ? sum[y * D + x] : sum[x * D + y];
    }
}

// Workgroups of a register: at most 2048 rows per run for the reduction (D = 5 on
// 1.7 M amplitudes: 18.6 us; 640 workgroups 21.4, one per block of fibres 18.7).
uint32_t adj_axis_wgs(uint32_t bpr) { return std::min(bpr, 2048u); }

template <class F>
qf_status with_dim_a(uint32_t D, F&& f) {
    switch (D) {
        case 2: return f(std::integral_constant<int, 2>{});
        case 3: return f(std::integral_constant<int, 3>{});
        case 4: return f(std::integral_constant<int, 4>{});
        case 5: return f(std::integral_constant<int, 5>{});
        case 6: return f(std::integral_constant<int, 6>{});
        case 7: return f(std::integral_constant<int, 7>{});
        case 8: return f(std::integral_constant<int, 8>{});
        case 9: return f(std::integral_constant<int, 9>{});
        case 10: return f(std::integral_constant<int, 10>{});
        case 11: return f(std::integral_constant<int, 11>{});
        case 12: return f(std::integral_constant<int, 12>{});
        case 13: return f(std::integral_constant<int, 13>{});
        case 14: return f(std::integral_constant<int, 14>{});
        case 15: return f(std::integral_constant<int, 15>{});
        case 16: return f(std::integral_constant<int, 16>{});
        default: return set_error(QF_EUNSUPPORTED, "dim %u outside 2..16", D);
    }
}

}  // namespace

AdjRows adj_axis_rows(const StateView& s, int q) {
    AdjRows r{};
    r.D = s.dims[q];
    r.rows = adj_axis_wgs((s.N / r.D + kFB - 1) / kFB);
    // more than four turns of a workgroup: chunks of the square root
    r.chunk = r.rows;
    if (r.rows > 32 * (256 / (r.D * r.D)))
        for (r.chunk = 1; r.chunk * r.chunk < r.rows;) ++r.chunk;
    return r;
}

qf_status launch_adj_axis(const StateView& s, void* lam, int q, const double* W, double* partial, hipStream_t st,
                          const ShiftArg* shift) {
    const uint32_t nfib_reg = s.N / s.dims[q];
    const uint32_t bpr = (nfib_reg + kFB - 1) / kFB;
    const uint32_t L = s.strides[q];
    auto body = [&](auto tag, auto dtag) -> qf_status {
        using T = decltype(tag);
        constexpr int D = decltype(dtag)::value;
        if constexpr (sizeof(MatArgA<T, D>) > 2048) {
            return set_error(QF_ERANGE, "dim %d too large for a complex128 adjoint matrix argument", D);
        } else {
            MatArgA<T, D> w;
            for (int i = 0; i < D * D; ++i) w.m[i] = cmake<T>(T(W[2 * i]), T(W[2 * i + 1]));
            const uint32_t wgs = adj_axis_wgs(bpr);
            hipLaunchKernelGGL((k_adj_axis<T, D>), dim3(wgs * s.batch), dim3(kFB), 0, st,
                               reinterpret_cast<cplx<T>*>(s.amps), reinterpret_cast<cplx<T>*>(lam), nfib_reg,
                               bpr, wgs, s.N, L, FastDiv(L), w, shift ? *shift : ShiftArg{}, partial);
            return check_launch("adjoint axis");
        }
    };
    return with_dim_a(s.dims[q], [&](auto dtag) -> qf_status {
        if (s.dtype == QF_C64) return body(float{}, dtag);
        return body(double{}, dtag);
    });
}

qf_status launch_adj_reduce(double* partial, const std::vector<AdjRows>& runs, uint32_t batch, double* mout,
                            uint32_t nslots, uint32_t slot_elems, hipStream_t st) {
    for (size_t i = 0; i < runs.size(); i += kAdjRows) {
        const size_t n = std::min(runs.size() - i, size_t(kAdjRows));
        AdjRowsArg a{};
        uint32_t chunks = 1;
        for (size_t j = 0; j < n; ++j) {
            a.run[j] = runs[i + j];
            chunks = std::max(chunks, (a.run[j].rows + a.run[j].chunk - 1) / a.run[j].chunk);
        }
        if (chunks > 1) {
            hipLaunchKernelGGL(k_adj_reduce<true>, dim3(uint32_t(n) * batch, chunks), dim3(256), 0, st, partial, a,
                               batch, nslots, slot_elems, mout);
            QF_CHECK(check_launch("adjoint reduce (chunks)"));
        }
        hipLaunchKernelGGL(k_adj_reduce<false>, dim3(uint32_t(n) * batch), dim3(256), 0, st, partial, a, batch,
                           nslots, slot_elems, mout);
        QF_CHECK(check_launch("adjoint reduce"));
    }
    return QF_OK;
}

}  // namespace qf
