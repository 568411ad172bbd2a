// Dense K x K block (K = D^k) on k adjacent qudits: psi[h, :, l] <- B psi[h, :, l]
// with the register viewed as [H][K][L].  This is a batched complex GEMM
// C[K x F] = B[K x K] X[K x F] over the F = H * L fibres.
//
// A workgroup owns a tile of NT fibres: it stages X[:, tile] in LDS (reads
// complete before any write, so the update is in place), then writes
// B X[:, tile] straight back to HBM.
#include <algorithm>

#include "qf_internal.h"

namespace qf {
namespace {

constexpr int kBlock = 256;

struct FusedGeom {
    uint32_t K;       // block size D^k
    uint32_t L;       // stride of the block's last qudit
    uint32_t nfib;    // H * L
    uint32_t NT;      // fibres per tile
    FastDiv divL;
    FastDiv divK;
    FastDiv divNT;
};

__device__ inline uint32_t fibre_base(const FusedGeom& g, uint32_t f) {
    const uint32_t h = g.divL.div(f);
    const uint32_t l = f - h * g.L;
    return h * g.K * g.L + l;
}

// Stage X[:, tile] into LDS as xs[b * NT + i].
template <typename T>
__device__ inline void load_tile(const cplx<T>* __restrict__ psi, const FusedGeom& g, uint32_t f0,
                                 uint32_t nt, cplx<T>* xs) {
    const uint32_t cnt = g.K * nt;
    if (g.L == 1) {
        // the tile is nt whole fibres of K contiguous amplitudes
        const uint32_t base = f0 * g.K;
        for (uint32_t e = threadIdx.x; e < cnt; e += kBlock) {
            const uint32_t i = g.divK.div(e);
            const uint32_t b = e - i * g.K;
            xs[b * g.NT + i] = psi[base + e];
        }
    } else {
        // consecutive lanes take consecutive fibres (consecutive l when L >= NT)
        const uint32_t cnt_full = g.K * g.NT;
        for (uint32_t e = threadIdx.x; e < cnt_full; e += kBlock) {
            const uint32_t b = g.divNT.div(e);
            const uint32_t i = e - b * g.NT;
            if (i < nt) xs[b * g.NT + i] = psi[fibre_base(g, f0 + i) + b * g.L];
        }
    }
}

// VALU path: lane (i, r) accumulates rows a = r, r + RG, ... for fibre i.
template <typename T>
__global__ __launch_bounds__(kBlock) void k_fused_valu(cplx<T>* __restrict__ psi,
                                                       const cplx<T>* __restrict__ B, FusedGeom g) {
    extern __shared__ unsigned char smem[];
    cplx<T>* xs = reinterpret_cast<cplx<T>*>(smem);
    const uint32_t f0 = blockIdx.x * g.NT;
    const uint32_t nt = min(g.NT, g.nfib - f0);
    load_tile(psi, g, f0, nt, xs);
    __syncthreads();
    const uint32_t i = threadIdx.x % g.NT;
    const uint32_t rg = kBlock / g.NT;
    const uint32_t r0 = threadIdx.x / g.NT;
    if (i >= nt) return;
    const uint32_t base = fibre_base(g, f0 + i);
    constexpr int RA = 4;
    for (uint32_t a0 = r0; a0 < g.K; a0 += rg * RA) {
        cplx<T> acc[RA];
#pragma unroll
        for (int r = 0; r < RA; ++r) acc[r] = cmake<T>(0, 0);
        for (uint32_t b = 0; b < g.K; ++b) {
            const cplx<T> x = xs[b * g.NT + i];
#pragma unroll
            for (int r = 0; r < RA; ++r) {
                const uint32_t a = a0 + r * rg;
                if (a < g.K) cmac(acc[r], B[a * g.K + b], x);
            }
        }
#pragma unroll
        for (int r = 0; r < RA; ++r) {
            const uint32_t a = a0 + r * rg;
            if (a < g.K) psi[base + a * g.L] = acc[r];
        }
    }
}

// ---------------------------------------------------------------------------
// FP32 matrix-core path (complex64, 128 < K <= 256).  Y = B X with
//   Y_re = B_re X_re - B_im X_im,  Y_im = B_re X_im + B_im X_re
// on v_mfma_f32_16x16x4f32 (A: 16 x 4, B: 4 x 16, C: 16 x 16).  Lane l of a
// wavefront supplies A[l % 16][l / 16] and B[l / 16][l % 16] and holds
// C[4 (l / 16) + r][l % 16] in accumulator register r.
//
// A workgroup owns NTM = 64 fibres.  X is staged in LDS as separate real and
// imaginary planes of Kp = ceil16(K) rows (rows >= K are zero), each row padded
// to 68 floats so that the four rows a wavefront reads per step fall in
// different banks.  B fragments are read from global memory (the K x K block
// stays in L2).  Wave w computes row blocks w, w + 4, ... against all four
// 16-fibre column blocks.  A real B (every imaginary part zero) skips the two
// products with B_im.
// ---------------------------------------------------------------------------

constexpr int NTM = 64;
constexpr int RS = NTM + 4;  // LDS row stride (floats)

typedef float f32x4 __attribute__((ext_vector_type(4)));

__global__ __launch_bounds__(kBlock) void k_fused_mfma(cplx<float>* __restrict__ psi,
                                                       const cplx<float>* __restrict__ B, FusedGeom g,
                                                       uint32_t Kp, int real) {
    extern __shared__ unsigned char smem[];
    float* xr = reinterpret_cast<float*>(smem);
    float* xi = xr + size_t(Kp) * RS;
    const uint32_t f0 = blockIdx.x * NTM;
    const uint32_t nt = min(uint32_t(NTM), g.nfib - f0);
    // stage X (zero rows >= K and columns >= nt)
    for (uint32_t e = threadIdx.x; e < Kp * NTM; e += kBlock) {
        const uint32_t b = e / NTM;
        const uint32_t i = e - b * NTM;
        cplx<float> v = cmake<float>(0.f, 0.f);
        if (b < g.K && i < nt) v = psi[fibre_base(g, f0 + i) + b * g.L];
        xr[b * RS + i] = v.re;
        xi[b * RS + i] = v.im;
    }
    __syncthreads();
    const int lane = threadIdx.x & 63;
    const int wave = threadIdx.x >> 6;
    const int lr = lane & 15;  // A row / B column / C column inside a block
    const int lk = lane >> 4;  // A column / B row inside a k step; C row group
    const uint32_t nrb = Kp / 16;
    for (uint32_t rb = wave; rb < nrb; rb += kBlock / 64) {
        f32x4 cr[4], ci[4];
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            cr[j] = f32x4{0.f, 0.f, 0.f, 0.f};
            ci[j] = f32x4{0.f, 0.f, 0.f, 0.f};
        }
        const uint32_t arow = rb * 16 + lr;
        for (uint32_t k0 = 0; k0 < Kp; k0 += 4) {
            const uint32_t acol = k0 + lk;
            cplx<float> a = cmake<float>(0.f, 0.f);
            if (arow < g.K && acol < g.K) a = B[arow * g.K + acol];
            const float* xrr = xr + (k0 + lk) * RS + lr;
            const float* xir = xi + (k0 + lk) * RS + lr;
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                const float br = xrr[j * 16];
                const float bi = xir[j * 16];
                cr[j] = __builtin_amdgcn_mfma_f32_16x16x4f32(a.re, br, cr[j], 0, 0, 0);
                ci[j] = __builtin_amdgcn_mfma_f32_16x16x4f32(a.re, bi, ci[j], 0, 0, 0);
                if (!real) {
                    cr[j] = __builtin_amdgcn_mfma_f32_16x16x4f32(-a.im, bi, cr[j], 0, 0, 0);
                    ci[j] = __builtin_amdgcn_mfma_f32_16x16x4f32(a.im, br, ci[j], 0, 0, 0);
                }
            }
        }
        // write back rows rb*16 + 4*lk + r of the four column blocks
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            const uint32_t col = uint32_t(j * 16 + lr);
            if (col >= nt) continue;
            const uint32_t base = fibre_base(g, f0 + col);
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                const uint32_t row = rb * 16 + uint32_t(4 * lk + r);
                if (row < g.K) psi[base + row * g.L] = cmake<float>(cr[j][r], ci[j][r]);
            }
        }
    }
}

// ---------------------------------------------------------------------------
// Blocks of 32 <= K <= 128 in complex64 on the bf16 matrix cores, in FP32
// precision.  Every FP32 operand is the exact sum of three bf16 values (each the
// rest of the last one rounded to nearest), and a product keeps the six partial
// products above 2^-26 of it (hi hi, hi mid, mid hi, hi lo, lo hi, mid mid),
// exact in the matrix core and added in FP32: 24 v_mfma_f32_16x16x32_bf16 (16
// cycles each) per 32 complex rows in place of 32 v_mfma_f32_16x16x4f32 (32
// cycles).  The products hi hi have an accumulator of their own: the others, 2^-8 of
// them, are summed without the rounding of the large sum, which is one addition for
// 32 rows.  Where a row's largest entry is at least 2/5 of its sum, so that a result
// can be one product with the one rounding of an FP32 product, two more are kept
// (mid lo, lo mid).  Relative error against 64 bits (rms; FP32 matrix cores, then
// these), Haar blocks on Gaussian states: K = 32 1.5e-7, 4.8e-8; K = 49 1.8e-7,
// 5.6e-8; K = 128 2.9e-7, 8.1e-8; K = 100 real 1.8e-7, 6.0e-8; diagonal phases 3.1e-8,
// 2.6e-8; real diagonals 2.5e-8, 2.5e-8; permutations exact.
//
// The amplitudes are multiplied by 2^23 and a row of the block by the power of two that
// brings its sum to 2^47 to 2^48, the results by their inverse, so that the parts of the
// smallest numbers are normal bf16 values (the matrix core takes subnormal ones for
// zero: unscaled, amplitudes of 1e-36 kept 8 bits, of 1e-39 none).  Amplitudes of 2^55
// and more, whose sums could overflow, and infinities: from a tile that holds one on (all
// tiles, where a row's sum is infinite or NaN), a workgroup writes nothing in the loop
// and takes FP32 products of the amplitudes themselves after it (plain_tile).  A NaN's
// parts are NaN, and so are its products, as in FP32.
//
// HBM-bound up to K = 49; time of a pass against the FP32 cores: K = 36 on 6^8 26 -> 20
// us, K = 49 on 7^9 317 -> 181 us (3.6 TB/s), K = 100 on 10^7 158 -> 88 us (real 125 ->
// 62), K = 128 on 2^24 280 -> 114 us.  Small registers: K = 100 on 10^5
// 18.4 -> 12 us, K = 49 on 7^5 12.7 -> 11, K = 128 on 2^15 22 -> 15.5.
//
// A persistent workgroup of NRB wavefronts owns one row block of 16 per wavefront,
// its block's operands in registers.  A tile of NF fibres lies in LDS as
// six planes (three parts of the real and imaginary values), a fibre's Kp values
// contiguous (plus 16 bytes against bank conflicts), so that an operand is one
// 16-byte read.  The next tile's amplitudes are loaded while the current one is
// multiplied, then split and stored.
// ---------------------------------------------------------------------------

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
typedef float f32x2 __attribute__((ext_vector_type(2)));
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));

// The three bf16 parts of eight floats.
__device__ __forceinline__ void split8(const float (&x)[8], u32x4 (&part)[3]) {
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        f32x2 r = {x[2 * i], x[2 * i + 1]};
#pragma unroll
        for (int p = 0; p < 3; ++p) {
            const bf16x2 h = __builtin_convertvector(r, bf16x2);  // to nearest even
            const uint32_t u = __builtin_bit_cast(uint32_t, h);
            part[p][i] = u;
            r.x -= __builtin_bit_cast(float, u << 16);
            r.y -= __builtin_bit_cast(float, u & 0xffff0000u);
        }
    }
}

// Scale of the amplitudes, and the limit of their scaled parts: with rows of sums below
// 2^48 each sum of products stays below 2^126, a difference below 2^127.
constexpr float kSplitScale = 0x1p23f, kSplitBack = 0x1p-23f;
constexpr float kSplitX = 0x1p78f;

// Fibres per tile: 64 (512-byte runs of HBM), 32 for K <= 48, where more and
// smaller workgroups do better (K = 32 on 2^24 amplitudes 54 against 70 us; K = 100
// on 10^7 108 against 85 us); 16 where the register's fibres then make at most one
// workgroup a CU (launch_split).
template <int NRB>
constexpr int split_fibres() {
    return NRB <= 3 ? 32 : 64;
}

// One tile by FP32 products from HBM: rows row0 .. row0 + 3 of the fibres col, col +
// 16, ...  Every lane of the workgroup calls it.
template <int NF, bool REAL>
__device__ __forceinline__ void plain_tile(cplx<float>* __restrict__ psi, const cplx<float>* __restrict__ B,
                                           const FusedGeom& g, uint32_t tile, int row0, int col) {
#pragma unroll 1
    for (int j = 0; j < NF / 16; ++j) {
        const uint32_t f = tile * NF + uint32_t(16 * j + col);
        const uint32_t base = f < g.nfib ? fibre_base(g, f) : 0u;
        f32x4 rr = {0.f, 0.f, 0.f, 0.f}, ii = rr, ri = rr;
#pragma unroll 1
        for (uint32_t b = 0; b < g.K; ++b) {
            const cplx<float> x = f < g.nfib ? psi[base + b * g.L] : cmake<float>(0.f, 0.f);
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                const uint32_t row = min(uint32_t(row0 + r), g.K - 1);
                const cplx<float> u = B[row * g.K + b];
                rr[r] = fmaf(u.re, x.re, rr[r]);
                ri[r] = fmaf(u.re, x.im, ri[r]);
                if constexpr (!REAL) {
                    ii[r] = fmaf(u.im, x.im, ii[r]);
                    ri[r] = fmaf(u.im, x.re, ri[r]);
                }
            }
        }
        __syncthreads();  // these fibres are read
        if (f < g.nfib) {
#pragma unroll
            for (int r = 0; r < 4; ++r)
                if (uint32_t(row0 + r) < g.K)
                    psi[base + uint32_t(row0 + r) * g.L] = cmake<float>(REAL ? rr[r] : rr[r] - ii[r], ri[r]);
        }
    }
}

// Wavefronts per SIMD the registers are held to: K <= 64 takes 3 (complex; 36 on 6^8
// 25 us with 2 of them, 22 with 3), other sizes what the compiler finds.
template <int NRB>
constexpr unsigned split_waves() {
    return NRB == 3 || NRB == 4 ? 3 : 1;
}

template <int NRB, int NF, bool REAL>
__global__ __launch_bounds__(64 * NRB) __attribute__((amdgpu_waves_per_eu(split_waves<NRB>()))) void k_fused_split(
    cplx<float>* __restrict__ psi, const cplx<float>* __restrict__ B, FusedGeom g) {
    constexpr int KB = (NRB + 1) / 2;        // k blocks of 32
    constexpr int Kp = 32 * KB;
    constexpr int CS = Kp * 2 + 16;          // bytes between fibres of a plane
    constexpr int PL = NF * CS;              // bytes of a plane
    constexpr int NT = 64 * NRB;
    constexpr int NU = NF * (Kp / 8);        // staging units: 8 rows of one fibre
    constexpr int UPL = (NU + NT - 1) / NT;  // per lane
    extern __shared__ __align__(16) unsigned char smem[];
    // the first tile that needs FP32 products; in the padding of a fibre, since a word
    // more of LDS made a pass of K = 49 twice as long (182 -> 363 us)
    uint32_t& plain = *reinterpret_cast<uint32_t*>(smem + Kp * 2);
    const int lane = threadIdx.x & 63;
    const int wave = threadIdx.x >> 6;
    const int lr = lane & 15;  // A row / B column / C column
    const int lk = lane >> 4;  // eight k of a k block; C row group
    if (threadIdx.x == 0) plain = ~0u;
    // the block's rows 16 wave + lr: parts of the real and imaginary entries
    u32x4 br[KB][3], bi[REAL ? 1 : KB][3];
    // scales of result rows 4 i .. 4 i + 3, in the fibres' padding from plane 1 on
    auto back_of = [&](int i) { return reinterpret_cast<f32x4*>(smem + (1 + i / NF) * PL + i % NF * CS + Kp * 2); };
    bool dominated, over;
    {
        const uint32_t row = uint32_t(16 * wave + lr);
        // unconditional loads stay together (K = 121 on 11^6 32 us with them under their
        // conditions, 25 us so): the last k block's past the row read its last entry
        cplx<float> u[KB][8];
#pragma unroll
        for (int kb = 0; kb < KB; ++kb)
#pragma unroll
            for (int i = 0; i < 8; ++i) {
                const uint32_t col = uint32_t(32 * kb + 8 * lk + i);
                u[kb][i] = B[min(row, g.K - 1) * g.K + (kb + 1 < KB ? col : min(col, g.K - 1))];
            }
        float largest = 0.f, sum = 0.f;  // |re| + |im| of the row's entries
#pragma unroll
        for (int kb = 0; kb < KB; ++kb)
#pragma unroll
            for (int i = 0; i < 8; ++i) {
                const bool in = kb + 1 < KB || uint32_t(32 * kb + 8 * lk + i) < g.K;
                const float m = fabsf(u[kb][i].re) + fabsf(u[kb][i].im);
                largest = fmaxf(largest, m);
                sum += in ? m : 0.f;
            }
#pragma unroll
        for (int m = 16; m < 64; m <<= 1) {
            largest = fmaxf(largest, __shfl_xor(largest, m, 64));
            sum += __shfl_xor(sum, m, 64);
        }
        over = !(sum < __builtin_inff());  // or NaN
        dominated = __any(row < g.K && largest > 0.f && sum <= 2.5f * largest);
        // the row's sum becomes 2^47 to 2^48 (2^126 is the largest scale)
        const int e = min(48 - __builtin_amdgcn_frexp_expf(sum), 126);
        const float scale = row < g.K ? ldexpf(1.f, e) : 0.f;
        if (lk == 0) reinterpret_cast<float*>(back_of(4 * wave + (lr >> 2)))[lr & 3] = ldexpf(kSplitBack, -e);
#pragma unroll
        for (int kb = 0; kb < KB; ++kb) {
            float xr[8], xi[8];
#pragma unroll
            for (int i = 0; i < 8; ++i) {
                const bool in = kb + 1 < KB || uint32_t(32 * kb + 8 * lk + i) < g.K;
                const float sc = in ? scale : 0.f;
                xr[i] = u[kb][i].re * sc;
                xi[i] = u[kb][i].im * sc;
            }
            split8(xr, br[kb]);
            if constexpr (!REAL) split8(xi, bi[kb]);
        }
    }
    const uint32_t ntiles = (g.nfib + NF - 1) / NF;
    cplx<float> x[UPL][8];
    // unit u: fibre u % NF, rows 8 (u / NF) .. + 7 (consecutive lanes: consecutive
    // fibres); where fibres are contiguous (L = 1), rows first
    auto unit = [&](int t, uint32_t& f, uint32_t& k8) {
        const uint32_t u = threadIdx.x + uint32_t(t) * NT;
        f = g.L == 1 ? u / (Kp / 8) : u % NF;
        k8 = g.L == 1 ? u % (Kp / 8) : u / NF;
        return u < uint32_t(NU);
    };
    auto fetch = [&](uint32_t tile) {
#pragma unroll
        for (int t = 0; t < UPL; ++t) {
            uint32_t f, k8;
            const bool ok = unit(t, f, k8) && tile * NF + f < g.nfib;
            const uint32_t fb = ok ? fibre_base(g, tile * NF + f) : 0u;
#pragma unroll
            for (int i = 0; i < 8; ++i) {
                const uint32_t b = 8 * k8 + i;
                x[t][i] = cmake<float>(0.f, 0.f);
                if (ok && b < g.K) x[t][i] = psi[fb + b * g.L];
            }
        }
    };
    uint32_t tile = blockIdx.x;
    if (tile < ntiles) fetch(tile);
    for (; tile < ntiles; tile += gridDim.x) {
        __syncthreads();  // the previous tile's operands are read
        float top = 0.f;  // largest part of this lane's amplitudes
#pragma unroll
        for (int t = 0; t < UPL; ++t) {
            uint32_t f, k8;
            if (!unit(t, f, k8)) continue;
            float v[8];
            u32x4 part[3];
            unsigned char* p = smem + f * CS + k8 * 16;
#pragma unroll
            for (int i = 0; i < 8; ++i) v[i] = x[t][i].re * kSplitScale;
            split8(v, part);
#pragma unroll
            for (int q = 0; q < 3; ++q) *reinterpret_cast<u32x4*>(p + q * PL) = part[q];
#pragma unroll
            for (int i = 0; i < 8; ++i) {
                top = fmaxf(top, fabsf(v[i]));
                v[i] = x[t][i].im * kSplitScale;
                top = fmaxf(top, fabsf(v[i]));
            }
            split8(v, part);
#pragma unroll
            for (int q = 0; q < 3; ++q) *reinterpret_cast<u32x4*>(p + (3 + q) * PL) = part[q];
        }
        if (over || top >= kSplitX) atomicMin(&plain, tile);
        __syncthreads();
        const uint32_t stop = plain;
        if (tile + gridDim.x < ntiles) fetch(tile + gridDim.x);
        auto mm = [](u32x4 a, u32x4 b, f32x4 c) {
            return __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, a), __builtin_bit_cast(bf16x8, b),
                                                           c, 0, 0, 0);
        };
#pragma unroll 1
        for (int j = 0; j < NF / 16; ++j) {
            // B_re X_re, B_im X_im, B_re X_im + B_im X_re: [0] the products of the
            // leading parts, [1] the others
            f32x4 rr[2] = {}, ii[2] = {}, ri[2] = {};
            const unsigned char* p = smem + (16 * j + lr) * CS + lk * 16;
            auto part = [&](int q, int kb) { return *reinterpret_cast<const u32x4*>(p + q * PL + kb * 64); };
            auto product = [&](int s, u32x4 ar, u32x4 ai, u32x4 xr, u32x4 xi) {
                rr[s] = mm(ar, xr, rr[s]);
                ri[s] = mm(ar, xi, ri[s]);
                if constexpr (!REAL) {
                    ii[s] = mm(ai, xi, ii[s]);
                    ri[s] = mm(ai, xr, ri[s]);
                }
            };
            if (dominated) {  // mid lo, lo mid
#pragma unroll
                for (int kb = 0; kb < KB; ++kb) {
                    product(1, br[kb][1], bi[REAL ? 0 : kb][1], part(2, kb), part(5, kb));
                    product(1, br[kb][2], bi[REAL ? 0 : kb][2], part(1, kb), part(4, kb));
                }
            }
#pragma unroll
            for (int kb = 0; kb < KB; ++kb) {
                u32x4 xr[3], xi[3];
#pragma unroll
                for (int q = 0; q < 3; ++q) {
                    xr[q] = part(q, kb);
                    xi[q] = part(3 + q, kb);
                }
                // smallest partial products first
                constexpr int pa[6] = {1, 2, 0, 1, 0, 0}, pb[6] = {1, 0, 2, 0, 1, 0};
#pragma unroll
                for (int q = 0; q < 6; ++q)
                    product(q < 5, br[kb][pa[q]], bi[REAL ? 0 : kb][pa[q]], xr[pb[q]], xi[pb[q]]);
            }
            rr[0] = REAL ? rr[0] + rr[1] : (rr[0] - ii[0]) + (rr[1] - ii[1]);
            ri[0] = ri[0] + ri[1];
            const uint32_t f = tile * NF + uint32_t(16 * j + lr);
            if (f < g.nfib && tile < stop) {
                const uint32_t base = fibre_base(g, f);
                const f32x4 back = *back_of(4 * wave + lk);
#pragma unroll
                for (int r = 0; r < 4; ++r) {
                    const uint32_t row = uint32_t(16 * wave + 4 * lk + r);
                    if (row < g.K) psi[base + row * g.L] = cmake<float>(rr[0][r] * back[r], ri[0][r] * back[r]);
                }
            }
        }
    }
    __syncthreads();  // plain is final also where this workgroup had no tile
    for (tile = plain; tile < ntiles; tile += gridDim.x) plain_tile<NF, REAL>(psi, B, g, tile, 16 * wave + 4 * lk, lr);
}

// The grid fills the LDS of 256 CUs once.
template <int NRB, int NF>
qf_status launch_split(const StateView& s, const FusedGeom& g, const void* B, bool real, hipStream_t st) {
    constexpr int Kp = 32 * ((NRB + 1) / 2);
    constexpr size_t lds = size_t(6) * NF * (Kp * 2 + 16);
    constexpr uint32_t cap = 256 * std::max<uint32_t>(1, uint32_t(160 * 1024 / lds));
    const uint32_t ntiles = (g.nfib + NF - 1) / NF;
    const uint32_t grid = std::min(ntiles, cap);
    auto* amps = reinterpret_cast<cplx<float>*>(s.amps);
    auto* mat = reinterpret_cast<const cplx<float>*>(B);
    if (real)
        hipLaunchKernelGGL((k_fused_split<NRB, NF, true>), dim3(grid), dim3(64 * NRB), lds, st, amps, mat, g);
    else
        hipLaunchKernelGGL((k_fused_split<NRB, NF, false>), dim3(grid), dim3(64 * NRB), lds, st, amps, mat, g);
    return check_launch("qf_apply_fused (bf16 matrix cores)");
}

// Up to 4096 fibres (a workgroup a CU) the pass waits for one tile's chain of loads, split
// and products, which is shorter for 16 fibres than for 64 on a few CUs (K = 100 on
// 10^5 19.4 -> 12 us, K = 128 on 2^15 21.7 -> 15.5, K = 36 on 6^7 12 -> 11).
template <int NRB>
qf_status launch_split(const StateView& s, const FusedGeom& g, const void* B, bool real, hipStream_t st) {
    return g.nfib <= 16 * 256 ? launch_split<NRB, 16>(s, g, B, real, st)
                              : launch_split<NRB, split_fibres<NRB>()>(s, g, B, real, st);
}

}  // namespace

qf_status launch_fused(const StateView& s, int k, int q0, const void* B, hipStream_t st, bool real) {
    const uint32_t K = span(s, q0, k);
    FusedGeom g{};
    g.K = K;
    g.L = s.strides[q0 + k - 1];
    g.nfib = s.total / K;
    const size_t esz = s.dtype == QF_C64 ? 8 : 16;
    uint32_t nt = 64;
    while (nt > 1 && size_t(K) * nt * esz > 64 * 1024) nt >>= 1;
    g.NT = nt;
    g.divL.init(g.L);
    g.divK.init(K);
    g.divNT.init(nt);
    if (s.dtype == QF_C64 && K >= 32 && K <= 128) {
        switch ((K + 15) / 16) {
            case 2: return launch_split<2>(s, g, B, real, st);
            case 3: return launch_split<3>(s, g, B, real, st);
            case 4: return launch_split<4>(s, g, B, real, st);
            case 5: return launch_split<5>(s, g, B, real, st);
            case 6: return launch_split<6>(s, g, B, real, st);
            case 7: return launch_split<7>(s, g, B, real, st);
            case 8: return launch_split<8>(s, g, B, real, st);
        }
    }
    if (s.dtype == QF_C64 && K > 128 && K <= 256) {
        const uint32_t Kp = (K + 15) / 16 * 16;
        const size_t lds = size_t(2) * Kp * RS * sizeof(float);
        const uint32_t grid = (g.nfib + NTM - 1) / NTM;
        hipLaunchKernelGGL(k_fused_mfma, dim3(grid), dim3(kBlock), lds, st, reinterpret_cast<cplx<float>*>(s.amps),
                           reinterpret_cast<const cplx<float>*>(B), g, Kp, real ? 1 : 0);
        return check_launch("qf_apply_fused (matrix cores)");
    }
    const uint32_t grid = (g.nfib + nt - 1) / nt;
    const size_t lds = size_t(K) * nt * esz;
    if (s.dtype == QF_C64) {
        hipLaunchKernelGGL(k_fused_valu<float>, dim3(grid), dim3(kBlock), lds, st,
                           reinterpret_cast<cplx<float>*>(s.amps), reinterpret_cast<const cplx<float>*>(B), g);
    } else {
        hipLaunchKernelGGL(k_fused_valu<double>, dim3(grid), dim3(kBlock), lds, st,
                           reinterpret_cast<cplx<double>*>(s.amps), reinterpret_cast<const cplx<double>*>(B), g);
    }
    return check_launch("qf_apply_fused");
}

}  // namespace qf
