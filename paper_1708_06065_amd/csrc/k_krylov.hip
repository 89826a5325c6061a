// Kernels of the flexible GMRES outer iteration (the Krylov solver the paper
// wraps its V-cycles in, Sec. 4).  Vectors hold R right-hand sides
// interleaved (element (i, q) at i R + q, R a power of two up to 32), as in
// the cycle; a basis is kc such vectors ldv elements apart.  Every kernel is
// a stream over HBM; the dot products reduce in a fixed order (per thread,
// then a fixed tree per block, then over the blocks in order), so their
// results do not depend on timing.
#include <hip/hip_runtime.h>

#include <algorithm>

#include "k_common.hpp"
#include "lair_internal.hpp"

namespace lair {

constexpr int KRY_BS = 256;
constexpr int KRY_KC = 8;        // basis vectors per dot-product pass
constexpr int KRY_GS_MAX = 24;   // basis vectors a thread holds in k_gs

// partial[(blk * kstride + kbase + k) * R + q] = the block's part of
// sum_i V_{kbase+k}[i R + q] w[i R + q], k < kc <= KRY_KC.  The grid stride
// is a multiple of R, so each thread keeps one right-hand side.
__global__ void __launch_bounds__(KRY_BS)
k_mdot(int64_t m, int R, const double *V, int64_t ldv, int kbase, int kc, int kstride,
       const double *w, double *partial) {
    __shared__ double sh[KRY_BS];
    double acc[KRY_KC];
#pragma unroll
    for (int k = 0; k < KRY_KC; ++k) acc[k] = 0.0;
    const double *Vb = V + (int64_t)kbase * ldv;
    const int64_t stride = (int64_t)gridDim.x * KRY_BS;
    for (int64_t e = (int64_t)blockIdx.x * KRY_BS + threadIdx.x; e < m; e += stride) {
        const double wv = w[e];
#pragma unroll
        for (int k = 0; k < KRY_KC; ++k)
            if (k < kc) acc[k] += Vb[(int64_t)k * ldv + e] * wv;
    }
    const int t = threadIdx.x;
    for (int k = 0; k < kc; ++k) {
        sh[t] = acc[k];
        __syncthreads();
        for (int o = KRY_BS / 2; o >= R; o >>= 1) {
            if (t < o) sh[t] += sh[t + o];
            __syncthreads();
        }
        if (t < R) partial[((int64_t)blockIdx.x * kstride + kbase + k) * R + t] = sh[t];
        __syncthreads();
    }
}

// out[k R + q] = sum over the blocks of their parts, one block per output
// (thread sums over every 256th part, then a fixed tree).  One thread per
// output, adding up to 1,024 parts in a chain, took 12 us; this takes 3.
__global__ void __launch_bounds__(KRY_BS)
k_mdot_final(int nblk, int stride, const double *partial, double *out) {
    __shared__ double sh[KRY_BS];
    const int t = threadIdx.x;
    double a = 0.0;
    for (int b = t; b < nblk; b += KRY_BS) a += partial[(int64_t)b * stride + blockIdx.x];
    sh[t] = a;
    __syncthreads();
    for (int o = KRY_BS / 2; o > 0; o >>= 1) {
        if (t < o) sh[t] += sh[t + o];
        __syncthreads();
    }
    if (t == 0) out[blockIdx.x] = sh[0];
}

// Gram-Schmidt in one pass over the basis: w -= sum_k coef[k] V_k as in k_maxpy
// (SUB), and at once the dot products of the new w with V_0 .. V_{kc-1} (DOT;
// the next pass's coefficients) or with itself (the norm).  Bound by the
// basis: each of its vectors is read once from memory where a subtraction and
// the products after it read it twice.  The block's sums go through shuffles
// (a tree in LDS for each vector took 7.6 us at 22,500 rows).
template <bool SUB, bool DOT>
__global__ void __launch_bounds__(KRY_BS)
k_gs(int64_t m, int R, const double *V, int64_t ldv, int kc, const double *coef, double *w,
     double *partial) {
    __shared__ double sh[KRY_BS / WAVE][KRY_GS_MAX * 32];
    double acc[DOT ? KRY_GS_MAX : 1];
#pragma unroll
    for (int k = 0; k < (DOT ? KRY_GS_MAX : 1); ++k) acc[k] = 0.0;
    const int64_t stride = (int64_t)gridDim.x * KRY_BS;
    for (int64_t e = (int64_t)blockIdx.x * KRY_BS + threadIdx.x; e < m; e += stride) {
        const int q = (int)(e & (R - 1));
        double v[KRY_GS_MAX], a = 0.0;
#pragma unroll
        for (int k = 0; k < KRY_GS_MAX; ++k)
            if (k < kc) v[k] = V[(int64_t)k * ldv + e];
        if (SUB) {
#pragma unroll
            for (int k = 0; k < KRY_GS_MAX; ++k)
                if (k < kc) a += coef[k * R + q] * v[k];
        }
        const double x = SUB ? w[e] - a : w[e];
        if (SUB) w[e] = x;
        if (DOT) {
#pragma unroll
            for (int k = 0; k < KRY_GS_MAX; ++k)
                if (k < kc) acc[k] += v[k] * x;
        } else {
            acc[0] += x * x;
        }
    }
    // lanes with the same right-hand side, then the block's waves in order
    const int lane = threadIdx.x & (WAVE - 1), wv = threadIdx.x / WAVE;
    const int nk = DOT ? kc : 1;
#pragma unroll
    for (int k = 0; k < (DOT ? KRY_GS_MAX : 1); ++k)
        if (k < nk) {
            double a = acc[k];
            for (int o = WAVE / 2; o >= R; o >>= 1) a += __shfl_xor(a, o);
            if (lane < R) sh[wv][k * R + lane] = a;
        }
    __syncthreads();
    for (int i = threadIdx.x; i < nk * R; i += KRY_BS) {
        double a = 0.0;
        for (int g = 0; g < KRY_BS / WAVE; ++g) a += sh[g][i];
        partial[(int64_t)blockIdx.x * nk * R + i] = a;
    }
}

// w[i R + q] -= sum_k coef[k R + q] V_k[i R + q], k ascending.
__global__ void __launch_bounds__(KRY_BS)
k_maxpy(int64_t m, int R, const double *V, int64_t ldv, int kc, const double *coef,
        double *w) {
    const int64_t e = (int64_t)blockIdx.x * KRY_BS + threadIdx.x;
    if (e >= m) return;
    const int q = (int)(e & (R - 1));
    double a = 0.0;
    for (int k = 0; k < kc; ++k) a += coef[k * R + q] * V[(int64_t)k * ldv + e];
    w[e] -= a;
}

// out[i R + q] = w[i R + q] * s[q], the factors a kernel argument
struct KryScale {
    double v[32];
};

__global__ void __launch_bounds__(KRY_BS)
k_scale_rhs(int64_t m, int R, const double *w, const KryScale s, double *out) {
    __shared__ double sc[32];
    if (threadIdx.x < 32) sc[threadIdx.x] = s.v[threadIdx.x];
    __syncthreads();
    const int64_t e = (int64_t)blockIdx.x * KRY_BS + threadIdx.x;
    if (e >= m) return;
    out[e] = w[e] * sc[e & (R - 1)];
}

static bool pow2_rhs(int R) { return R >= 1 && R <= 32 && (R & (R - 1)) == 0; }

int32_t kry_dot_blocks(int64_t m) {
    const int64_t b = (m + KRY_BS - 1) / KRY_BS;
    return (int32_t)std::max<int64_t>(1, std::min<int64_t>(b, 1024));
}

void op_mdot(int64_t n, int32_t R, const double *V, int64_t ldv, int32_t kc, const double *w,
             double *partial, double *out, hipStream_t s) {
    if (!pow2_rhs(R)) fail(LAIR_EINVAL, "right-hand sides must be a power of two up to 32");
    if (kc < 1) return;
    const int64_t m = n * R;
    const int32_t nblk = kry_dot_blocks(m);
    if (kc <= KRY_GS_MAX)
        LAIR_LAUNCH((k_gs<false, true>), dim3(nblk), dim3(KRY_BS), 0, s, m, R, V, ldv, kc,
                    (const double *)nullptr, const_cast<double *>(w), partial);
    else for (int kb = 0; kb < kc; kb += KRY_KC) {
        const int c = std::min(KRY_KC, kc - kb);
        LAIR_LAUNCH(k_mdot, dim3(nblk), dim3(KRY_BS), 0, s, m, R, V, ldv, kb, c, kc, w,
                    partial);
    }
    LAIR_LAUNCH_CHECK();
    LAIR_LAUNCH(k_mdot_final, dim3(kc * R), dim3(KRY_BS), 0, s, nblk, kc * R, partial, out);
    LAIR_LAUNCH_CHECK();
}

void op_gram_schmidt(int64_t n, int32_t R, const double *V, int64_t ldv, int32_t kc,
                     const double *coef, double *w, bool dots, double *partial, double *out,
                     hipStream_t s) {
    if (!pow2_rhs(R)) fail(LAIR_EINVAL, "right-hand sides must be a power of two up to 32");
    if (kc < 1 || n == 0) return;
    const int64_t m = n * R;
    // a thread holds its entry of every basis vector; longer bases take the
    // separate kernels
    if (kc > KRY_GS_MAX) {
        op_maxpy(n, R, V, ldv, kc, coef, w, s);
        if (dots) op_mdot(n, R, V, ldv, kc, w, partial, out, s);
        else op_mdot(n, R, w, ldv, 1, w, partial, out, s);
        return;
    }
    const int32_t nblk = kry_dot_blocks(m), no = (dots ? kc : 1) * R;
    if (dots)
        LAIR_LAUNCH((k_gs<true, true>), dim3(nblk), dim3(KRY_BS), 0, s, m, R, V, ldv, kc, coef, w,
                    partial);
    else
        LAIR_LAUNCH((k_gs<true, false>), dim3(nblk), dim3(KRY_BS), 0, s, m, R, V, ldv, kc, coef, w,
                    partial);
    LAIR_LAUNCH_CHECK();
    LAIR_LAUNCH(k_mdot_final, dim3(no), dim3(KRY_BS), 0, s, nblk, no, partial, out);
    LAIR_LAUNCH_CHECK();
}

void op_maxpy(int64_t n, int32_t R, const double *V, int64_t ldv, int32_t kc,
              const double *coef, double *w, hipStream_t s) {
    if (!pow2_rhs(R)) fail(LAIR_EINVAL, "right-hand sides must be a power of two up to 32");
    if (kc < 1 || n == 0) return;
    const int64_t m = n * R;
    LAIR_LAUNCH(k_maxpy, dim3(blocks_for(m, KRY_BS)), dim3(KRY_BS), 0, s, m, R, V, ldv, kc,
                coef, w);
    LAIR_LAUNCH_CHECK();
}

void op_scale_rhs(int64_t n, int32_t R, const double *w, const double *sc, double *out,
                  hipStream_t s) {
    if (!pow2_rhs(R)) fail(LAIR_EINVAL, "right-hand sides must be a power of two up to 32");
    if (n == 0) return;
    const int64_t m = n * R;
    KryScale k{};
    for (int32_t q = 0; q < R; ++q) k.v[q] = sc[q];
    LAIR_LAUNCH(k_scale_rhs, dim3(blocks_for(m, KRY_BS)), dim3(KRY_BS), 0, s, m, R, w, k, out);
    LAIR_LAUNCH_CHECK();
}

}  // namespace lair
