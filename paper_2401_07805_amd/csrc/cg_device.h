// Device-side pieces of the CG vector kernels, shared by the uniform-mesh
// solvers (blas.hip) and the refined-mesh solver (amr.hip).
#pragma once
#include "blas.h"

namespace vpp {

constexpr int BT = 256;

// 16-byte packet of T (two doubles or four floats): one dwordx4 access.
template <typename T>
struct alignas(16) Pack {
    static constexpr int W = 16 / (int)sizeof(T);
    T v[W];
};

// Wave sums of two doubles (butterfly); every lane receives the totals.
__device__ __forceinline__ void wave_sum2(double& a, double& b)
{
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) {
        a += __shfl_xor(a, o);
        b += __shfl_xor(b, o);
    }
}

// Workgroup sums of two doubles in a fixed order (wave_sum2, then the waves in
// index order); every thread receives the totals.
template <int NT>
__device__ __forceinline__ void block_sum2(double& a, double& b)
{
    static_assert(NT % 64 == 0, "whole waves only");
    wave_sum2(a, b);
    __shared__ double pa[NT / 64], pb[NT / 64];
    __syncthreads();
    if ((threadIdx.x & 63) == 0) {
        pa[threadIdx.x / 64] = a;
        pb[threadIdx.x / 64] = b;
    }
    __syncthreads();
    double sa = 0.0, sb = 0.0;
#pragma unroll
    for (int i = 0; i < NT / 64; ++i) {
        sa += pa[i];
        sb += pb[i];
    }
    a = sa;
    b = sb;
}

// Totals of the ng partials of both quantities (every thread receives them); the
// second quantity's start at `second`.
__device__ __forceinline__ void sum_partials(const double* red, int ng, double& a, double& b,
                                             int second = kMaxRedBlocks)
{
    a = 0.0;
    b = 0.0;
    for (int i = threadIdx.x; i < ng; i += BT) {
        a += red[i];
        b += red[second + i];
    }
    block_sum2<BT>(a, b);
}

__device__ __forceinline__ void write_partials(double* red, double a, double b, int bid, int second = kMaxRedBlocks)
{
    if (threadIdx.x == 0) {
        red[bid] = a;
        red[second + bid] = b;
    }
}
__device__ __forceinline__ void write_partials(double* red, double a, double b)
{
    write_partials(red, a, b, blockIdx.x);
}

// alpha = rz / p.Ap, with p.Ap summed from the ndot partials by every workgroup
// in the same order (extra: a further term of it); false when the system has stopped or breaks down here.
template <typename T>
__device__ __forceinline__ bool update_alpha(int bid, CgState* st, int par, const double* dot_part, int ndot, T& alpha,
                                             double extra = 0.0)
{
    // the state read at once (before the barrier of the reduction, so the loads
    // overlap it instead of following it)
    const int halt = st->halt[par];
    const double rz_par = st->rz[par];
    if (halt) return false;
    double pAp = 0.0, unused = 0.0;
    for (int i = threadIdx.x; i < ndot; i += BT) pAp += dot_part[i];
    block_sum2<BT>(pAp, unused);
    pAp += extra;
    if (bid == 0 && threadIdx.x == 0) st->pAp = pAp;
    if (!(pAp > 0.0) || !isfinite(pAp)) {
        if (bid == 0 && threadIdx.x == 0) st->breakdown = 1;
        return false;
    }
    alpha = T(rz_par / pAp);
    return true;
}

// Packets a thread handles per batch in the search-direction update.  A
// thread takes packets c, c + S, c + 2S, ... (S = threads of the system's
// grid) in that order, as a plain grid-stride loop would, but loads a whole
// batch before it uses any of it, and the first batch before the reduction
// that gives beta: each batch then costs one memory latency instead of one
// per packet.
constexpr int kBatch = 4;

// Body of the search-direction update for workgroup bid of nblk (one system;
// ng partials of the update to sum).
template <typename T>
__device__ __forceinline__ void pupdate_body(int bid, int nblk, CgState* st, int par, const double* red, int ng,
                                             T* __restrict__ x, const T* __restrict__ r, T* __restrict__ p,
                                             const T* __restrict__ invd, int64_t n, int second = kMaxRedBlocks)
{
    // every state field this kernel reads, at once (before the reduction's
    // barrier); thread 0 of workgroup 0 is the only writer, of other fields
    const int halt = st->halt[par], brk = st->breakdown;
    const double rz_par = st->rz[par], pAp_par = st->pAp, tol2 = st->tol2;
    const int iters0 = st->iters, max_iter = st->max_iter, hcap = st->hist_cap;
    double* const coef = st->coef;
    if (halt || brk) {
        if (bid == 0 && threadIdx.x == 0) st->halt[1 - par] = 1;
        return;
    }
    using P = Pack<T>;
    constexpr int W = P::W, U = kBatch;
    const int64_t np = n / W;
    const int64_t S = (int64_t)nblk * BT;
    const int64_t c0 = (int64_t)bid * BT + threadIdx.x;
    P rv[U], dv[U], pv[U], xv[U];
    auto load = [&](int64_t cb) {
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const int64_t c = cb + u * S;
            if (c < np) {
                rv[u] = reinterpret_cast<const P*>(r)[c];
                dv[u] = reinterpret_cast<const P*>(invd)[c];
                pv[u] = reinterpret_cast<const P*>(p)[c];
                xv[u] = reinterpret_cast<const P*>(x)[c];
            }
        }
    };
    load(c0);
    double rr, rzn;
    sum_partials(red, ng, rr, rzn, second);
    const double beta_d = rzn / rz_par;
    if (bid == 0 && threadIdx.x == 0) {
        const int it = iters0 + 1;
        st->iters = it;
        st->rr_last = rr;
        st->rr[par] = rr;
        st->rznew[par] = rzn;
        st->rz[1 - par] = rzn;
        if (!isfinite(rr) || !isfinite(rzn)) {
            st->breakdown = 1;
            st->halt[1 - par] = 1;
        } else if (rr < tol2 || it >= max_iter) {
            st->halt[1 - par] = 1;
        }
        if (coef && it < hcap) {
            coef[3 * it] = rz_par / pAp_par;
            coef[3 * it + 1] = beta_d;
            coef[3 * it + 2] = rzn;
        }
    }
    // the same alpha as the update's (same operands, same rounding)
    const T alpha = T(rz_par / pAp_par);
    const T beta = T(beta_d);
    for (int64_t cb = c0; cb < np; cb += U * S) {
        if (cb != c0) load(cb);
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const int64_t c = cb + u * S;
            if (c >= np) break;
#pragma unroll
            for (int j = 0; j < W; ++j) {
                xv[u].v[j] = fma(alpha, pv[u].v[j], xv[u].v[j]);
                pv[u].v[j] = fma(beta, pv[u].v[j], rv[u].v[j] * dv[u].v[j]);
            }
            reinterpret_cast<P*>(x)[c] = xv[u];
            reinterpret_cast<P*>(p)[c] = pv[u];
        }
    }
    if (bid == 0)
        for (int64_t i = np * W + threadIdx.x; i < n; i += BT) {
            x[i] = fma(alpha, p[i], x[i]);
            p[i] = fma(beta, p[i], r[i] * invd[i]);
        }
}

}  // namespace vpp
