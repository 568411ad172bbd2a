// The differentiable controlled rotation sum_m |m><m|_c (x) R^{jk}_alpha(m theta)_t
// (arXiv:2409.17716, Appendix, subsection "Controlled Rotation Gate"), and
// without a control the plain two-level rotation as a slab sweep (the memory
// form of the paper's sparse rotation, subsection "Generalized rotation gate").
//
// The register is viewed as [H][D][L] for the target t (D = d_t, L = S_t, the
// product of the dimensions after t); a fibre is the D amplitudes
// psi[h, :, l], and its control digit m (0 <= m < d_c) is read from its index.  The x- and y-type rotations mix only target levels j and k, so a
// lane reads and writes just those two amplitudes of its fibre (2/D of the
// state); the z type scales levels 0..j.  Fibres at control level 0 are left
// alone.  Consecutive lanes take consecutive l, so for L >= 64 every access of
// a wavefront is one contiguous run.  The forward kernel gives each lane
// kFPL fibres, kCB apart, and issues all their loads before the first store:
// with one fibre a wavefront keeps only 1 KB of loads in flight when the two
// levels are contiguous slabs, too little to cover the HBM latency.  A register
// whose fibres make fewer than two workgroups a CU that way takes one per lane.
//
// Per control level m the kernels read a two-entry table: x, y types
// (cos(m theta / 2), sin(m theta / 2)) in one complex entry (the inverse
// negates the sine); z type the phase of levels below j and the phase of level
// j.  The adjoint kernel takes the inverse table, adds
//   m * Im <lam_f| S |psi_f>   (the slab generator is m S)
// over its fibres in FP64 (fixed tree per workgroup, then a fixed-order sum per
// register) and un-applies the gate on psi and lam.
#include <algorithm>
#include <type_traits>

#include "qf_internal.h"

namespace qf {
namespace {

constexpr int kCB = 256;
constexpr int kFPL = 4;  // fibres per lane in the forward kernel (large registers)

struct CrGeom {
    int32_t has_ctrl;    // 0: plain rotation, every fibre uses table entry 1
    uint32_t L;          // stride of the target qudit
    FastDiv divL;
    FastDiv cstride;     // stride of the control qudit
    FastDiv divDc;       // dimension of the control qudit
    uint32_t ntab;       // table entries: 2 per control level
    uint32_t nfib;       // fibres per register, N / d_t
    uint32_t N;          // amplitudes per register
    uint32_t bpr;        // workgroups per register (one fibre per lane: the adjoint)
    uint32_t bprf;       // workgroups per register of the forward kernel with kFPL fibres per lane
    int32_t kind;        // 0 = x, 1 = y, 2 = z
    int32_t j, k;        // levels (z: j)
    double alpha;        // z: sqrt(2 / (j (j + 1)))
};

template <typename T>
struct CrTab {
    cplx<T> t[2 * kMaxDim];
};

template <typename T>
__device__ __forceinline__ void load_tab(const CrTab<T>& harg, const cplx<T>* __restrict__ dtab, size_t tab_stride,
                                         uint32_t b, uint32_t ntab, cplx<T>* tab) {
    if (threadIdx.x < ntab) tab[threadIdx.x] = dtab ? dtab[size_t(b) * tab_stride + threadIdx.x] : harg.t[threadIdx.x];
    __syncthreads();
}

__device__ __forceinline__ uint32_t ctrl_level(const CrGeom& g, uint32_t local) {
    if (!g.has_ctrl) return 1u;
    const uint32_t qv = g.cstride.div(local);
    return qv - g.divDc.div(qv) * g.divDc.d;
}

// The x- or y-type rotation of levels (j, k) with cs = (cos, sin) of half the
// angle, on the pair (a, b) = (psi_j, psi_k).  The fused operations are written out
// (which product of a sum is rounded first), so that every kernel variant of a
// direction gives the same bits.
template <typename T, bool ADJ>
__device__ __forceinline__ void rot_pair(int kind, cplx<T> cs, cplx<T>& a, cplx<T>& b) {
    const T c = cs.re, s = cs.im;
    const cplx<T> x = a, y = b;
    if (kind == 0) {  // [[c, -i s], [-i s, c]]
        a = cmake<T>(fma(s, y.im, c * x.re), fma(c, x.im, -(s * y.re)));
        b = cmake<T>(ADJ ? fma(c, y.re, s * x.im) : fma(s, x.im, c * y.re), fma(c, y.im, -(s * x.re)));
    } else {          // [[c, -s], [s, c]]
        a = cmake<T>(fma(-s, y.re, c * x.re), fma(c, x.im, -(s * y.im)));
        b = ADJ ? cmake<T>(fma(c, y.re, s * x.re), fma(c, y.im, s * x.im))
                : cmake<T>(fma(s, x.re, c * y.re), fma(s, x.im, c * y.im));
    }
}

// The z-type rotation of control level m on the fibre at base.
template <typename T>
__device__ __forceinline__ void rotate_z(cplx<T>* __restrict__ psi, const CrGeom& g, uint32_t base,
                                         const cplx<T>* tab, uint32_t m) {
    const cplx<T> p1 = tab[2 * m], p2 = tab[2 * m + 1];
    for (int d = 0; d < g.j; ++d) psi[base + uint32_t(d) * g.L] = cmul(psi[base + uint32_t(d) * g.L], p1);
    psi[base + uint32_t(g.j) * g.L] = cmul(psi[base + uint32_t(g.j) * g.L], p2);
}

template <typename T, int D, int FPL>
__global__ __launch_bounds__(kCB) void k_crot(cplx<T>* __restrict__ psi, CrGeom g, CrTab<T> harg,
                                              const cplx<T>* __restrict__ dtab, size_t tab_stride) {
    __shared__ cplx<T> tab[2 * kMaxDim];
    const uint32_t wgs = FPL == 1 ? g.bpr : g.bprf;
    const uint32_t b = blockIdx.x / wgs;
    load_tab<T>(harg, dtab, tab_stride, b, g.ntab, tab);
    const uint32_t f0 = (blockIdx.x - b * wgs) * (kCB * FPL) + threadIdx.x;
    cplx<T>* const p = psi + size_t(b) * g.N;
    uint32_t loc[FPL], lev[FPL];  // fibre base and control level (0: left alone)
#pragma unroll
    for (int i = 0; i < FPL; ++i) {
        const uint32_t f = f0 + uint32_t(i) * kCB;
        loc[i] = 0;
        lev[i] = 0;
        if (f < g.nfib) {
            const uint32_t h = g.divL.div(f);
            loc[i] = h * (uint32_t(D) * g.L) + (f - h * g.L);
            lev[i] = ctrl_level(g, loc[i]);
        }
    }
    if (g.kind == 2) {
#pragma unroll
        for (int i = 0; i < FPL; ++i)
            if (lev[i] != 0) rotate_z<T>(p, g, loc[i], tab, lev[i]);
        return;
    }
    const uint32_t oj = uint32_t(g.j) * g.L, ok = uint32_t(g.k) * g.L;
    cplx<T> va[FPL], vb[FPL];
#pragma unroll
    for (int i = 0; i < FPL; ++i) {
        va[i] = cmake<T>(0, 0);
        vb[i] = cmake<T>(0, 0);
        if (lev[i] != 0) {
            va[i] = p[loc[i] + oj];
            vb[i] = p[loc[i] + ok];
        }
    }
#pragma unroll
    for (int i = 0; i < FPL; ++i) {
        if (lev[i] == 0) continue;
        rot_pair<T, false>(g.kind, tab[2 * lev[i]], va[i], vb[i]);
        p[loc[i] + oj] = va[i];
        p[loc[i] + ok] = vb[i];
    }
}

// Deterministic workgroup sum: an xor butterfly inside each wavefront, then the
// wavefront totals in order.
__device__ inline double cr_block_sum(double v, double* sh) {
#pragma unroll
    for (int m = 32; m > 0; m >>= 1) v += __shfl_xor(v, m, 64);
    if ((threadIdx.x & 63u) == 0) sh[threadIdx.x >> 6] = v;
    __syncthreads();
    double r = sh[0];
#pragma unroll
    for (int w = 1; w < kCB / 64; ++w) r += sh[w];
    return r;
}

// psi and lam are read once: the gradient term and the rotation take the loaded
// amplitudes (with the rotation loading them again, its latency came on top of the
// gradient's: 5.4 us against 4.4 on 4^9 in complex128).
template <typename T, int D>
__global__ __launch_bounds__(kCB) void k_crot_adj(cplx<T>* __restrict__ psi, cplx<T>* __restrict__ lam, CrGeom g,
                                                  CrTab<T> harg, const cplx<T>* __restrict__ dtab, size_t tab_stride,
                                                  double* __restrict__ partial) {
    __shared__ cplx<T> tab[2 * kMaxDim];
    __shared__ double sh[kCB / 64];
    const uint32_t b = blockIdx.x / g.bpr;
    load_tab<T>(harg, dtab, tab_stride, b, g.ntab, tab);
    const uint32_t f = (blockIdx.x - b * g.bpr) * kCB + threadIdx.x;
    double acc = 0.0;
    if (f < g.nfib) {
        const uint32_t h = g.divL.div(f);
        const uint32_t local = h * (uint32_t(D) * g.L) + (f - h * g.L);
        const uint32_t m = ctrl_level(g, local);
        if (m != 0) {
            cplx<T>* p = psi + size_t(b) * g.N;
            cplx<T>* l = lam + size_t(b) * g.N;
            double im = 0.0;  // Im <lam_f| S |psi_f>
            if (g.kind == 2) {
                const cplx<T> p1 = tab[2 * m], p2 = tab[2 * m + 1];
                for (int d = 0; d <= g.j; ++d) {
                    const uint32_t i = local + uint32_t(d) * g.L;
                    const cplx<T> x = p[i], y = l[i];
                    const double w = d < g.j ? g.alpha : -g.alpha * g.j;
                    im += w * (double(y.re) * double(x.im) - double(y.im) * double(x.re));
                    const cplx<T> ph = d < g.j ? p1 : p2;
                    p[i] = cmul(x, ph);
                    l[i] = cmul(y, ph);
                }
            } else {
                const uint32_t ia = local + uint32_t(g.j) * g.L, ib = local + uint32_t(g.k) * g.L;
                cplx<T> pj = p[ia], pk = p[ib], lj = l[ia], lk = l[ib];
                // conj(lj) pk and conj(lk) pj
                const double r1 = double(lj.re) * pk.re + double(lj.im) * pk.im;
                const double i1 = double(lj.re) * pk.im - double(lj.im) * pk.re;
                const double r2 = double(lk.re) * pj.re + double(lk.im) * pj.im;
                const double i2 = double(lk.re) * pj.im - double(lk.im) * pj.re;
                im = g.kind == 0 ? i1 + i2 : r2 - r1;  // x: Im(z1 + z2); y: Im(-i z1 + i z2)
                rot_pair<T, true>(g.kind, tab[2 * m], pj, pk);
                rot_pair<T, true>(g.kind, tab[2 * m], lj, lk);
                p[ia] = pj;
                p[ib] = pk;
                l[ia] = lj;
                l[ib] = lk;
            }
            acc = double(m) * im;
        }
    }
    const double s = cr_block_sum(acc, sh);
    if (threadIdx.x == 0) partial[blockIdx.x] = s;
}

// out[b * ostride + a.gate[r].out] = sum of the partials of gate r and register b
// (fixed order), for up to kCrotRows gates in one launch.
constexpr int kCrotRows = 128;

struct CrotRowsArg {
    CrotRows gate[kCrotRows];
};

__global__ __launch_bounds__(kCB) void k_crot_reduce(const double* __restrict__ partial, CrotRowsArg a,
                                                     uint32_t batch, double* __restrict__ out, uint32_t ostride) {
    __shared__ double sh[kCB / 64];
    const uint32_t r = blockIdx.x / batch, b = blockIdx.x - r * batch;
    const uint32_t bpr = a.gate[r].rows;
    const double* p = partial + a.gate[r].off + size_t(b) * bpr;
    constexpr int kAcc = 8;  // independent loads in flight per lane
    double acc[kAcc];
#pragma unroll
    for (int j = 0; j < kAcc; ++j) acc[j] = 0.0;
    for (uint32_t i = threadIdx.x; i < bpr; i += kAcc * kCB)
#pragma unroll
        for (int j = 0; j < kAcc; ++j)
            if (i + j * kCB < bpr) acc[j] += p[i + j * kCB];
#pragma unroll
    for (int w = kAcc / 2; w > 0; w >>= 1)
#pragma unroll
        for (int j = 0; j < w; ++j) acc[j] += acc[j + w];
    const double s = cr_block_sum(acc[0], sh);
    if (threadIdx.x == 0) out[size_t(b) * ostride + a.gate[r].out] = s;
}

template <class F>
qf_status with_dim_c(uint32_t D, F&& f) {
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

CrGeom make_geom(const StateView& s, const CrotArgs& a) {
    CrGeom g{};
    g.has_ctrl = a.ctrl >= 0 ? 1 : 0;
    g.L = s.strides[a.tgt];
    g.divL.init(g.L);
    g.cstride.init(a.ctrl >= 0 ? s.strides[a.ctrl] : 1u);
    g.divDc.init(a.ctrl >= 0 ? s.dims[a.ctrl] : 2u);
    g.ntab = 2 * g.divDc.d;
    g.nfib = s.N / s.dims[a.tgt];
    g.N = s.N;
    g.bpr = (g.nfib + kCB - 1) / kCB;
    g.bprf = (g.nfib + kCB * kFPL - 1) / (kCB * kFPL);
    g.kind = a.kind;
    g.j = a.j;
    g.k = a.k;
    g.alpha = a.kind == 2 ? std::sqrt(2.0 / (double(a.j) * (a.j + 1))) : 0.0;
    return g;
}

template <typename T>
CrTab<T> host_tab(const double* htab, uint32_t ntab) {
    CrTab<T> t{};
    if (htab)
        for (uint32_t i = 0; i < ntab; ++i) t.t[i] = cmake<T>(T(htab[2 * i]), T(htab[2 * i + 1]));
    return t;
}

}  // namespace

uint32_t crot_rows(const StateView& s, int tgt) { return (s.N / s.dims[tgt] + kCB - 1) / kCB; }

qf_status launch_crot(const StateView& s, const CrotArgs& a, const void* dtab, size_t tab_stride, const double* htab,
                      hipStream_t st) {
    const CrGeom g = make_geom(s, a);
    // by workgroups at four fibres per lane: 64 3.2 us so, 2.5 with one per lane; 256 3.9, 3.4;
    // 512 4.9, 4.6; 1024 7.6, 7.1; 2048 10.5, 11.0 (complex64 qubits)
    const bool one = uint64_t(g.bprf) * s.batch < 512;
    return with_dim_c(s.dims[a.tgt], [&](auto dtag) -> qf_status {
        constexpr int D = decltype(dtag)::value;
        auto go = [&](auto tag) {
            using T = decltype(tag);
            auto* amps = reinterpret_cast<cplx<T>*>(s.amps);
            auto* tab = reinterpret_cast<const cplx<T>*>(dtab);
            if (one)
                hipLaunchKernelGGL((k_crot<T, D, 1>), dim3(g.bpr * s.batch), dim3(kCB), 0, st, amps, g,
                                   host_tab<T>(htab, g.ntab), tab, tab_stride);
            else
                hipLaunchKernelGGL((k_crot<T, D, kFPL>), dim3(g.bprf * s.batch), dim3(kCB), 0, st, amps, g,
                                   host_tab<T>(htab, g.ntab), tab, tab_stride);
        };
        if (s.dtype == QF_C64)
            go(float{});
        else
            go(double{});
        return check_launch("controlled rotation");
    });
}

qf_status launch_crot_adj(const StateView& s, void* lam, const CrotArgs& a, const void* dtab, size_t tab_stride,
                          const double* htab, double* partial, hipStream_t st) {
    const CrGeom g = make_geom(s, a);
    return with_dim_c(s.dims[a.tgt], [&](auto dtag) -> qf_status {
        constexpr int D = decltype(dtag)::value;
        if (s.dtype == QF_C64)
            hipLaunchKernelGGL((k_crot_adj<float, D>), dim3(g.bpr * s.batch), dim3(kCB), 0, st,
                               reinterpret_cast<cplx<float>*>(s.amps), reinterpret_cast<cplx<float>*>(lam), g,
                               host_tab<float>(htab, g.ntab), reinterpret_cast<const cplx<float>*>(dtab), tab_stride,
                               partial);
        else
            hipLaunchKernelGGL((k_crot_adj<double, D>), dim3(g.bpr * s.batch), dim3(kCB), 0, st,
                               reinterpret_cast<cplx<double>*>(s.amps), reinterpret_cast<cplx<double>*>(lam), g,
                               host_tab<double>(htab, g.ntab), reinterpret_cast<const cplx<double>*>(dtab), tab_stride,
                               partial);
        return check_launch("controlled rotation adjoint");
    });
}

qf_status launch_crot_reduce(const double* partial, const std::vector<CrotRows>& gates, uint32_t batch, double* out,
                             uint32_t ostride, hipStream_t st) {
    for (size_t i = 0; i < gates.size(); i += kCrotRows) {
        const size_t n = std::min(gates.size() - i, size_t(kCrotRows));
        CrotRowsArg a{};
        for (size_t j = 0; j < n; ++j) a.gate[j] = gates[i + j];
        hipLaunchKernelGGL(k_crot_reduce, dim3(uint32_t(n) * batch), dim3(kCB), 0, st, partial, a, batch, out, ostride);
        QF_CHECK(check_launch("controlled rotation gradient sums"));
    }
    return QF_OK;
}

}  // namespace qf
