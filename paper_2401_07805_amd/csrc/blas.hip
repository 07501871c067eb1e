// Vector kernels of the Jacobi-preconditioned CG (Krylov solvers of Sec.
// "Numerical framework", stopping rule of Table tab:solver_settings).
//
// All CG scalars live on the device in FP64 (CgState) so that a chunk of
// iterations can be recorded once in a hipGraph and replayed without host
// round trips.  One iteration is three kernels:
//   apply:    the tile kernel of q = A p with per-workgroup partials of p.q
//             (apply kernels; the shared-node assembly is left to update)
//   update:   pAp from those partials; alpha = rz/pAp; q on shared nodes from
//             the apply's partials; r -= alpha q;
//             per-workgroup partial sums of r.r and r.(D^-1 r)
//   pupdate:  every workgroup sums the partials in the same fixed order,
//             beta = rz_new/rz; x += alpha p and p = D^-1 r + beta p in one
//             pass over p; workgroup 0 records the iteration and the stop
//             decision.
// The solution update sits in pupdate because that kernel reads p anyway:
// the iteration then moves 80 instead of 88 bytes per FP64 unknown.
// Reductions use no atomics: a producer writes one partial per workgroup and
// the consumer sums them in a fixed order, so every run gives the same bits.
//
// Stop flags are double-buffered by iteration parity: the kernels of the
// iteration of parity `par` test halt[par], and pupdate(par) writes only
// halt[1-par] (propagating a stop it sees), so no kernel reads a flag that the
// same kernel writes.  Once a stop is set every later kernel returns at once.
#include "blas.h"

#include <algorithm>

#include "cg_device.h"
#include "shared_nodes.h"

namespace vpp {

// Number of workgroups of the streaming kernels (about 4 packets per thread).
template <typename T>
static int grid_for(int64_t n)
{
    const int64_t packets = (n + Pack<T>::W - 1) / Pack<T>::W;
    const int64_t want = (packets + 4 * BT - 1) / (4 * BT);
    return (int)(want < 1 ? 1 : (want > kMaxRedBlocks ? kMaxRedBlocks : want));
}

// Whether the update reads a shared-node map (4 bytes a node) or looks its
// nodes up by index arithmetic, which hides behind the memory traffic once the
// vectors are large: update in us, map / lookup, same tiles: FP64 56^3 Q2 12.1 /
// 12.4, 64^3 Q2 17.6 / 17.8, 43^3 Q3 19.8 / 18.8, 72^3 Q2 22.9 / 21.9, 96^3 Q2 55.0 /
// 47.6, 96^3 Q3 261 / 233; FP32 64^3 Q3 37.1 / 39.8, 112^3 Q2 47.5 / 51.0, 80^3 Q3
// 74.2 / 71.1, 96^3 Q3 148 / 123.
bool shared_map_pays(int64_t n, size_t value_bytes)
{
    return n <= (value_bytes == 8 ? int64_t(1) << 21 : int64_t(12000000));
}

// Workgroups of the update: one packet per thread up to three workgroups per
// CU (48^3 Q2 9.2 us, 64^3 16.8, 80^3 27.6; with four 9.7, 16.9, 29.0), four for the
// FP32 update without a map (80^3 Q3 71 us against 76; FP64 72^3 Q2 22.2 against 21.9).
template <typename T>
static int grid_update(int64_t n)
{
    const int64_t per = (int64_t)BT * Pack<T>::W;
    const int64_t cap = sizeof(T) == 4 && !shared_map_pays(n, sizeof(T)) ? kMaxRedBlocks : 768;
    return (int)std::min<int64_t>(cap, std::max<int64_t>(1, (n + per - 1) / per));
}

// Workgroups of the search-direction update, whose threads take their packets
// in batches of kBatch: two per CU while a batch covers the vector (48^3 Q2 8.3
// us, with four 8.7), then four (64^3 15.9 us, with two 17.2); above 2 10^7
// unknowns as many as give every thread whole batches (96^3 Q3 245 us, FP32 93, against
// 266 and 97 with four; 88^3 Q2 43.3 against 41.4, 128^3 Q2 FP32 68 against 64).
template <typename T>
static int grid_pupdate(int64_t n)
{
    const int64_t per = (int64_t)BT * Pack<T>::W;
    const int64_t all = std::max<int64_t>(1, (n + per - 1) / per);   // workgroups at one packet per thread
    if (all <= 512 * kBatch) return (int)std::min<int64_t>(all, 512);
    if (n <= 20000000) return 1024;
    const int64_t its = ((all + 1023) / 1024 + kBatch - 1) / kBatch * kBatch;
    return (int)((all + its - 1) / its);
}

// r = b - q (q may be null: zero initial guess), p = D^-1 r; partials of r.r
// and r.D^-1 r.
template <typename T>
__global__ void __launch_bounds__(BT) cg_init_kernel(double* red, const T* __restrict__ b, const T* __restrict__ q,
                                                     T* __restrict__ r, T* __restrict__ p,
                                                     const T* __restrict__ invd, int64_t n)
{
    double rr = 0.0, rz = 0.0;
    for (int64_t i = (int64_t)blockIdx.x * BT + threadIdx.x; i < n; i += (int64_t)gridDim.x * BT) {
        const T ri = q ? b[i] - q[i] : b[i];
        const T zi = ri * invd[i];
        r[i] = ri;
        p[i] = zi;
        rr += (double)ri * (double)ri;
        rz += (double)ri * (double)zi;
    }
    block_sum2<BT>(rr, rz);
    write_partials(red, rr, rz);
}

// One workgroup: rr_last = r.r, rz[0] = r.D^-1 r.
__global__ void __launch_bounds__(BT) cg_init_finish_kernel(CgState* st, const double* red, int ng)
{
    double rr, rz;
    sum_partials(red, ng, rr, rz);
    if (threadIdx.x == 0) {
        st->rr_last = rr;
        st->rz[0] = rz;
    }
}

// update fused with the assembly of the apply's shared-node partials: q holds
// A p on the nodes only one tile touches (and on Dirichlet rows); for a shared
// node the value is the sum of its partials in rank order, as the assembly
// kernel forms it.  p.Ap is summed from the apply's per-workgroup partials in
// the same fixed order by every workgroup.
template <typename T>
struct SharedParts {
    const unsigned* map;   // per node: 0, or where its partials are (shared_map_entry); null: looked up by e
    const T* part;
    int64_t stride;
    const double* dot_part;
    int ndot;
    SharedEnum e;
    int bcmask;
};

// Entry of the shared-node map: f << 2 | log2 of the number of partials (1, 2, 3;
// f < 2^29, since 8 rank arrays are indexed with 32 bits), 0 for a node that
// one tile holds alone or that is a Dirichlet node.
__host__ __device__ inline unsigned shared_map_entry(int f, int cnt)
{
    return (unsigned)f << 2 | (cnt == 2 ? 1u : (cnt == 4 ? 2u : 3u));
}

__global__ void __launch_bounds__(BT) shared_map_kernel(SharedEnum e, int bcmask, unsigned* __restrict__ map, int64_t n)
{
    for (int64_t g = (int64_t)blockIdx.x * BT + threadIdx.x; g < n; g += (int64_t)gridDim.x * BT) {
        int f, cnt;
        map[g] = shared_lookup(e, bcmask, (int)g, f, cnt) ? shared_map_entry(f, cnt) : 0u;
    }
}

// q on W nodes with map entries mp: on shared ones the sum of the partials, in
// rank order as the assembly kernel forms it.  Ranks 0 and 1 are loaded for
// every node (a node that is not shared reads entry 0), so only the nodes of
// two or three planes branch.
template <typename T, int W>
__device__ __forceinline__ void assemble_packet(const SharedParts<T>& sp, const unsigned (&mp)[W], T (&qv)[W])
{
    T s[W];
    unsigned top = 0;
#pragma unroll
    for (int t = 0; t < W; ++t) {
        const unsigned f = mp[t] >> 2;
        s[t] = sp.part[f] + sp.part[sp.stride + f];
        top = max(top, mp[t] & 3u);
    }
    if (top > 1) {
#pragma unroll
        for (int t = 0; t < W; ++t) {
            if ((mp[t] & 3u) < 2) continue;
            const T* const p = sp.part + (mp[t] >> 2);
            const T p2 = p[2 * sp.stride], p3 = p[3 * sp.stride];
            s[t] = (s[t] + p2) + p3;
            if ((mp[t] & 3u) == 3) {
                const T p4 = p[4 * sp.stride], p5 = p[5 * sp.stride], p6 = p[6 * sp.stride], p7 = p[7 * sp.stride];
                s[t] = (((s[t] + p4) + p5) + p6) + p7;
            }
        }
    }
#pragma unroll
    for (int t = 0; t < W; ++t)
        if (mp[t]) qv[t] = s[t];
}

// The map entries of the W nodes from g0 on, by index arithmetic (reciprocal
// divisions, the row's part once unless the packet wraps a row).
template <int W>
__device__ __forceinline__ void lookup_packet(const SharedEnum& e, int bcmask, int g0, unsigned (&mp)[W])
{
    int f[W], cnt[W];
    bool sh[W];
    const int rw = qdiv(g0, e.nn[0], e.inv_nn[0]), i0 = g0 - rw * e.nn[0];
    if (i0 + W <= e.nn[0]) {
        const int l = qdiv(rw, e.nn[1], e.inv_nn[1]);
        const SharedRow w = shared_row(e, bcmask, rw - l * e.nn[1], l);
#pragma unroll
        for (int t = 0; t < W; ++t) sh[t] = shared_in_row(e, bcmask, w, i0 + t, f[t], cnt[t]);
    } else {
#pragma unroll
        for (int t = 0; t < W; ++t) sh[t] = shared_lookup(e, bcmask, g0 + t, f[t], cnt[t]);
    }
#pragma unroll
    for (int t = 0; t < W; ++t) mp[t] = sh[t] ? shared_map_entry(f[t], cnt[t]) : 0u;
}

// assemble_packet for entries that were just computed: every partial of the
// packet loaded under its condition before any is added (the same sums).  With
// entries from the map the conditions would wait for them.  (96^3 Q2 49.3 -> 47.6
// us, 64^3 Q3 56.7 -> 55.0.)
template <typename T, int W>
__device__ __forceinline__ void assemble_computed(const SharedParts<T>& sp, const unsigned (&mp)[W], T (&qv)[W])
{
    T pv[W][8];
#pragma unroll
    for (int t = 0; t < W; ++t) {
        const int cnt = mp[t] ? 1 << (mp[t] & 3u) : 0;
        const unsigned f = mp[t] >> 2;
#pragma unroll
        for (int k = 0; k < 8; ++k) pv[t][k] = k < cnt ? sp.part[k * sp.stride + f] : T(0);
    }
#pragma unroll
    for (int t = 0; t < W; ++t)
        if (mp[t]) {
            T v = pv[t][0] + pv[t][1];
#pragma unroll
            for (int k = 2; k < 8; ++k)
                if (k < 1 << (mp[t] & 3u)) v += pv[t][k];
            qv[t] = v;
        }
}

// Body of the update for workgroup bid of one system; the workgroup returns at
// once when the system has stopped.  Share v of the nsum shares takes packets
// v BT + tid + j nsum BT and gives one partial of each sum; a workgroup has one
// share (nblk = nsum) or, with SHARES, shares bid, bid + nblk, ...: the partials
// and the sums over them are those of one share per workgroup.
template <typename T, bool SHARES, bool MAP>
__device__ __forceinline__ void assemble_update_body(int bid, int nblk, int nsum, CgState* st, int par, double* red,
                                                     const SharedParts<T>& sp, T* __restrict__ r,
                                                     const T* __restrict__ q, const T* __restrict__ invd, int64_t n)
{
    __shared__ double share_a[SHARES ? kMaxShares : 1][BT / 64], share_b[SHARES ? kMaxShares : 1][BT / 64];
    float* hist = nullptr;
    int hit = 0, hcap = 0;
    int64_t hstride = 0;
    if constexpr (sizeof(T) == 4) {
        // residual record of an FP32 phase (iterations counted by the previous
        // direction update, which has completed)
        hist = st->hist;
        hit = st->iters + 1;
        hcap = st->hist_cap;
        hstride = st->hist_stride;
    }
    using P = Pack<T>;
    constexpr int W = P::W;
    struct alignas(4 * W) Map {
        unsigned v[W];
    };
    const int64_t np = n / W;
    // a packet's map entries are loaded one packet ahead (the first before the
    // reduction), so that its partials' addresses do not wait for them
    const int64_t S = (int64_t)nsum * BT;
    int64_t c = (int64_t)bid * BT + threadIdx.x;
    Map mp{};
    if (MAP && c < np) mp = reinterpret_cast<const Map*>(sp.map)[c];
    T alpha;
    if (!update_alpha(bid, st, par, sp.dot_part, sp.ndot, alpha)) return;
    T* hrec = nullptr;
    if constexpr (sizeof(T) == 4)
        if (hist && hit < hcap) hrec = hist + (size_t)hit * (size_t)hstride;
    int share = 0;
    for (int v = bid; v < nsum; v += nblk, ++share) {
        double rr = 0.0, rz = 0.0;
        c = (int64_t)v * BT + threadIdx.x;
        const int64_t after = SHARES && v + nblk < nsum ? c + (int64_t)nblk * BT : np;   // the next share's first packet
        for (; c < np; c += S) {
            P rv = reinterpret_cast<const P*>(r)[c];
            const P dv = reinterpret_cast<const P*>(invd)[c];
            P qv = reinterpret_cast<const P*>(q)[c];
            Map now = mp;
            const int64_t next = c + S < np ? c + S : after;
            if (MAP && next < np) mp = reinterpret_cast<const Map*>(sp.map)[next];
            if constexpr (MAP) {
                assemble_packet<T, W>(sp, now.v, qv.v);
            } else {
                lookup_packet<W>(sp.e, sp.bcmask, (int)(c * W), now.v);
                assemble_computed<T, W>(sp, now.v, qv.v);
            }
#pragma unroll
            for (int t = 0; t < W; ++t) {
                const T ri = fma(-alpha, qv.v[t], rv.v[t]);
                rv.v[t] = ri;
                rr += (double)ri * (double)ri;
                rz += (double)ri * (double)(ri * dv.v[t]);
            }
            reinterpret_cast<P*>(r)[c] = rv;
            if (hrec) reinterpret_cast<P*>(hrec)[c] = rv;
        }
        if (v == 0)
            for (int64_t i = np * W + threadIdx.x; i < n; i += BT) {
                unsigned mi[1];
                if constexpr (MAP) mi[0] = sp.map[i];
                else lookup_packet<1>(sp.e, sp.bcmask, (int)i, mi);
                T qi[1] = {q[i]};
                assemble_packet<T, 1>(sp, mi, qi);
                const T ri = fma(-alpha, qi[0], r[i]);
                r[i] = ri;
                if (hrec) hrec[i] = ri;
                rr += (double)ri * (double)ri;
                rz += (double)ri * (double)(ri * invd[i]);
            }
        if constexpr (!SHARES) {
            block_sum2<BT>(rr, rz);
            write_partials(red, rr, rz, bid);
            return;
        }
        wave_sum2(rr, rz);
        if (threadIdx.x % 64 == 0) {
            share_a[share][threadIdx.x / 64] = rr;
            share_b[share][threadIdx.x / 64] = rz;
        }
    }
    // the waves of every share in index order, as block_sum2 adds them
    __syncthreads();
    if ((int)threadIdx.x < share) {
        double a = 0.0, b = 0.0;
#pragma unroll
        for (int i = 0; i < BT / 64; ++i) {
            a += share_a[threadIdx.x][i];
            b += share_b[threadIdx.x][i];
        }
        red[bid + threadIdx.x * nblk] = a;
        red[kMaxRedBlocks + bid + threadIdx.x * nblk] = b;
    }
}

template <typename T, bool MAP>
__global__ void __launch_bounds__(BT) cg_assemble_update_kernel(CgState* st, int par, double* red, SharedParts<T> sp,
                                                                T* __restrict__ r, const T* __restrict__ q,
                                                                const T* __restrict__ invd, int64_t n)
{
    assemble_update_body<T, false, MAP>(blockIdx.x, gridDim.x, gridDim.x, st, par, red, sp, r, q, invd, n);
}

template <typename T>
__global__ void __launch_bounds__(BT) cg_pupdate_kernel(CgState* st, int par, const double* red, int ng,
                                                        T* __restrict__ x, const T* __restrict__ r,
                                                        T* __restrict__ p, const T* __restrict__ invd, int64_t n)
{
    pupdate_body<T>(blockIdx.x, gridDim.x, st, par, red, ng, x, r, p, invd, n);
}

// ---------------------------------------------------------------------------
// Batched PCG: the update and the search-direction update of every system of a
// batch in one launch each.  System i owns workgroups [blk_begin, blk_begin +
// nblk) of the grid; owner[] gives the system of each.

template <typename T>
__global__ void __launch_bounds__(BT) cg_batch_update_kernel(const CgSystem<T>* sys, const int* owner, int par)
{
    const CgSystem<T>& y = sys[owner[blockIdx.x]];
    const SharedParts<T> sp{y.map, y.part, y.stride, y.dot_part, y.ndot, {}, 0};
    assemble_update_body<T, true, true>((int)blockIdx.x - y.blk_begin, y.nblk, y.nsum, y.st, par, y.red, sp, y.r, y.q, y.invd,
                                  y.n);
}

template <typename T>
__global__ void __launch_bounds__(BT) cg_batch_pupdate_kernel(const CgSystem<T>* sys, const int* owner, int par)
{
    const CgSystem<T>& y = sys[owner[blockIdx.x]];
    pupdate_body<T>((int)blockIdx.x - y.blk_begin, y.nblk, y.st, par, y.red, y.nsum, y.x, y.r, y.p, y.invd, y.n);
}

// r = b - q in FP64 and partials of r.r (outer residual of the mixed solver and
// the true residual at the end of every solve).
__global__ void __launch_bounds__(BT) residual_kernel(const double* __restrict__ b, const double* __restrict__ q,
                                                      double* __restrict__ r, int64_t n, double* red)
{
    double s = 0.0, unused = 0.0;
    for (int64_t i = (int64_t)blockIdx.x * BT + threadIdx.x; i < n; i += (int64_t)gridDim.x * BT) {
        const double v = b[i] - q[i];
        if (r) r[i] = v;
        s += v * v;
    }
    block_sum2<BT>(s, unused);
    write_partials(red, s, 0.0);
}

__global__ void __launch_bounds__(BT) sum_finish_kernel(const double* red, int ng, double* out)
{
    double a, b;
    sum_partials(red, ng, a, b);
    if (threadIdx.x == 0) *out = a;
}

__global__ void __launch_bounds__(BT) cg_replace32_kernel(const double* __restrict__ r64, double scale,
                                                          double pscale, float* __restrict__ r32,
                                                          float* __restrict__ p32, float* __restrict__ x32,
                                                          const float* __restrict__ invd, int64_t n, double* red)
{
    double rr = 0.0, rz = 0.0;
    const float ps = (float)pscale;
    for (int64_t i = (int64_t)blockIdx.x * BT + threadIdx.x; i < n; i += (int64_t)gridDim.x * BT) {
        const float ri = (float)(scale * r64[i]);
        const float zi = ri * invd[i];
        r32[i] = ri;
        x32[i] = 0.0f;
        p32[i] = pscale == 0.0 ? zi : ps * p32[i];
        rr += (double)ri * (double)ri;
        rz += (double)ri * (double)zi;
    }
    block_sum2<BT>(rr, rz);
    write_partials(red, rr, rz);
}

// One workgroup: restart the inner state at parity 0 after a replacement.
__global__ void __launch_bounds__(BT) cg_resume_kernel(CgState* st, const double* red, int ng)
{
    double rr, rz;
    sum_partials(red, ng, rr, rz);
    if (threadIdx.x == 0) {
        st->rz[0] = rz;
        st->rr_last = rr;
        st->halt[0] = 0;
        st->halt[1] = 0;
        st->breakdown = 0;
    }
}

__global__ void __launch_bounds__(BT) convert_kernel(const double* __restrict__ a, float* __restrict__ b, int64_t n)
{
    for (int64_t i = (int64_t)blockIdx.x * BT + threadIdx.x; i < n; i += (int64_t)gridDim.x * BT) b[i] = (float)a[i];
}

// x += scale * d32, in FP64.
__global__ void __launch_bounds__(BT) promote_add_kernel(double* __restrict__ x, const float* __restrict__ d,
                                                         double scale, int64_t n)
{
    for (int64_t i = (int64_t)blockIdx.x * BT + threadIdx.x; i < n; i += (int64_t)gridDim.x * BT)
        x[i] = fma(scale, (double)d[i], x[i]);
}

template <typename T>
hipError_t launch_cg_init(CgState* st, double* red, const T* b, const T* q, T* r, T* p, const T* invd, int64_t n,
                          hipStream_t s)
{
    const int g = grid_for<T>(n);
    hipLaunchKernelGGL(cg_init_kernel<T>, dim3(g), dim3(BT), 0, s, red, b, q, r, p, invd, n);
    hipLaunchKernelGGL(cg_init_finish_kernel, dim3(1), dim3(BT), 0, s, st, red, g);
    return hipGetLastError();
}

hipError_t launch_shared_map(const SharedEnum& e, int bcmask, unsigned* map, hipStream_t s)
{
    const int64_t n = (int64_t)e.nn[0] * e.nn[1] * e.nn[2];
    const int g = (int)std::min<int64_t>(8192, (n + BT - 1) / BT);
    hipLaunchKernelGGL(shared_map_kernel, dim3(g), dim3(BT), 0, s, e, bcmask, map, n);
    return hipGetLastError();
}

template <typename T>
hipError_t launch_cg_assemble_update(CgState* st, int par, double* red, const double* dot_part, int ndot,
                                     const unsigned* map, const SharedEnum& e, int bcmask, const T* part,
                                     int64_t stride, T* r, const T* q, const T* invd, int64_t n, hipStream_t s)
{
    const SharedParts<T> sp{map, part, stride, dot_part, ndot, e, bcmask};
    const dim3 g(grid_update<T>(n)), b(BT);
    if (map)
        hipLaunchKernelGGL((cg_assemble_update_kernel<T, true>), g, b, 0, s, st, par, red, sp, r, q, invd, n);
    else
        hipLaunchKernelGGL((cg_assemble_update_kernel<T, false>), g, b, 0, s, st, par, red, sp, r, q, invd, n);
    return hipGetLastError();
}

template <typename T>
hipError_t launch_cg_pupdate(CgState* st, int par, const double* red, T* x, const T* r, T* p, const T* invd,
                             int64_t n, hipStream_t s)
{
    const int ng = grid_update<T>(n);   // the partials the update wrote
    hipLaunchKernelGGL(cg_pupdate_kernel<T>, dim3(grid_pupdate<T>(n)), dim3(BT), 0, s, st, par, red, ng, x, r, p, invd,
                       n);
    return hipGetLastError();
}

int cg_update_blocks(int64_t n) { return grid_update<double>(n); }

hipError_t launch_cg_batch_step(const CgSystem<double>* sys, const int* owner, int total_blocks, int par, hipStream_t s)
{
    hipLaunchKernelGGL(cg_batch_update_kernel<double>, dim3(total_blocks), dim3(BT), 0, s, sys, owner, par);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(cg_batch_pupdate_kernel<double>, dim3(total_blocks), dim3(BT), 0, s, sys, owner, par);
    return hipGetLastError();
}

#define VPP_INST(T)                                                                                          \
    template hipError_t launch_cg_init<T>(CgState*, double*, const T*, const T*, T*, T*, const T*, int64_t,  \
                                          hipStream_t);                                                      \
    template hipError_t launch_cg_pupdate<T>(CgState*, int, const double*, T*, const T*, T*, const T*, int64_t, \
                                             hipStream_t);                                                       \
    template hipError_t launch_cg_assemble_update<T>(CgState*, int, double*, const double*, int, const unsigned*, \
                                                     const SharedEnum&, int, const T*, int64_t, T*, const T*,        \
                                                     const T*, int64_t, hipStream_t);
VPP_INST(double)
VPP_INST(float)
#undef VPP_INST

// ---------------------------------------------------------------------------
// Deflation space of the mixed-precision solver (Ritz vectors of the first
// FP32 phase and the Galerkin correction in their span).

// One unknown per thread; the recorded residuals are read eight at a time
// (all loads of a group issued before their use).
__global__ void __launch_bounds__(BT) ritz_kernel(const float* __restrict__ hist, int64_t stride, int m,
                                                  const double* __restrict__ C, int k,
                                                  const double* __restrict__ invd, double* __restrict__ W, int64_t n)
{
    constexpr int G = 8;
    for (int64_t i = (int64_t)blockIdx.x * BT + threadIdx.x; i < n; i += (int64_t)gridDim.x * BT) {
        double acc[kMaxDefl];
#pragma unroll
        for (int t = 0; t < kMaxDefl; ++t) acc[t] = 0.0;
        const float* col = hist + (size_t)i;
        for (int j0 = 0; j0 < m; j0 += G) {
            float h[G];
#pragma unroll
            for (int u = 0; u < G; ++u) h[u] = (j0 + u < m) ? col[(size_t)(j0 + u) * (size_t)stride] : 0.0f;
#pragma unroll
            for (int u = 0; u < G; ++u) {
                if (j0 + u >= m) break;
#pragma unroll
                for (int t = 0; t < kMaxDefl; ++t)
                    if (t < k) acc[t] = fma(C[(j0 + u) * k + t], (double)h[u], acc[t]);
            }
        }
        const double di = invd[i];
#pragma unroll
        for (int t = 0; t < kMaxDefl; ++t)
            if (t < k) W[(size_t)t * (size_t)n + (size_t)i] = acc[t] * di;
    }
}

__global__ void __launch_bounds__(BT) multi_dot_kernel(const double* __restrict__ V, int k,
                                                       const double* __restrict__ y, int64_t n, double* red)
{
    double acc[kMaxDefl];
#pragma unroll
    for (int t = 0; t < kMaxDefl; ++t) acc[t] = 0.0;
    for (int64_t i = (int64_t)blockIdx.x * BT + threadIdx.x; i < n; i += (int64_t)gridDim.x * BT) {
        const double yi = y[i];
#pragma unroll
        for (int t = 0; t < kMaxDefl; ++t)
            if (t < k) acc[t] = fma(V[(size_t)t * (size_t)n + (size_t)i], yi, acc[t]);
    }
#pragma unroll
    for (int t = 0; t < kMaxDefl; t += 2) {
        double a = acc[t], b = acc[t + 1];
        block_sum2<BT>(a, b);
        if (threadIdx.x == 0) {
            if (t < k) red[(size_t)t * kMaxRedBlocks + blockIdx.x] = a;
            if (t + 1 < k) red[(size_t)(t + 1) * kMaxRedBlocks + blockIdx.x] = b;
        }
    }
}

__global__ void __launch_bounds__(BT) multi_dot_finish_kernel(const double* red, int k, int ng, double* out)
{
    for (int t = 0; t < k; t += 2) {
        double a = 0.0, b = 0.0;
        for (int i = threadIdx.x; i < ng; i += BT) {
            a += red[(size_t)t * kMaxRedBlocks + i];
            if (t + 1 < k) b += red[(size_t)(t + 1) * kMaxRedBlocks + i];
        }
        block_sum2<BT>(a, b);
        if (threadIdx.x == 0) {
            out[t] = a;
            if (t + 1 < k) out[t + 1] = b;
        }
    }
}

__global__ void __launch_bounds__(BT) defl_update_kernel(double* __restrict__ x, double* __restrict__ r,
                                                         const double* __restrict__ W,
                                                         const double* __restrict__ AW, DeflCoef c, int k,
                                                         int64_t n, double* red)
{
    double s2 = 0.0, unused = 0.0;
    for (int64_t i = (int64_t)blockIdx.x * BT + threadIdx.x; i < n; i += (int64_t)gridDim.x * BT) {
        double xi = x[i], ri = r[i];
#pragma unroll
        for (int t = 0; t < kMaxDefl; ++t)
            if (t < k) {
                xi = fma(c.c[t], W[(size_t)t * (size_t)n + (size_t)i], xi);
                ri = fma(-c.c[t], AW[(size_t)t * (size_t)n + (size_t)i], ri);
            }
        x[i] = xi;
        r[i] = ri;
        s2 += ri * ri;
    }
    block_sum2<BT>(s2, unused);
    write_partials(red, s2, 0.0);
}

hipError_t launch_ritz(const float* hist, int64_t stride, int m, const double* C, int k, const double* invd,
                       double* W, int64_t n, hipStream_t s)
{
    if (k < 1 || k > kMaxDefl) return hipErrorInvalidValue;
    const int64_t want = (n + BT - 1) / BT;
    const int g = (int)(want < 1 ? 1 : (want > 65536 ? 65536 : want));
    hipLaunchKernelGGL(ritz_kernel, dim3(g), dim3(BT), 0, s, hist, stride, m, C, k, invd, W, n);
    return hipGetLastError();
}

hipError_t launch_multi_dot(const double* V, int k, const double* y, int64_t n, double* red, double* out,
                            hipStream_t s)
{
    if (k < 1 || k > kMaxDefl) return hipErrorInvalidValue;
    const int g = grid_for<double>(n);
    hipLaunchKernelGGL(multi_dot_kernel, dim3(g), dim3(BT), 0, s, V, k, y, n, red);
    hipLaunchKernelGGL(multi_dot_finish_kernel, dim3(1), dim3(BT), 0, s, red, k, g, out);
    return hipGetLastError();
}

hipError_t launch_defl_update(double* x, double* r, const double* W, const double* AW, DeflCoef c, int k, int64_t n,
                              double* red, double* rr, hipStream_t s)
{
    if (k < 1 || k > kMaxDefl) return hipErrorInvalidValue;
    const int g = grid_for<double>(n);
    hipLaunchKernelGGL(defl_update_kernel, dim3(g), dim3(BT), 0, s, x, r, W, AW, c, k, n, red);
    hipLaunchKernelGGL(sum_finish_kernel, dim3(1), dim3(BT), 0, s, red, g, rr);
    return hipGetLastError();
}

hipError_t launch_residual(const double* b, const double* q, double* r, int64_t n, double* red, double* rr,
                           hipStream_t s)
{
    const int g = grid_for<double>(n);
    hipLaunchKernelGGL(residual_kernel, dim3(g), dim3(BT), 0, s, b, q, r, n, red);
    hipLaunchKernelGGL(sum_finish_kernel, dim3(1), dim3(BT), 0, s, red, g, rr);
    return hipGetLastError();
}

hipError_t launch_cg_replace32(CgState* st, double* red, const double* r64, double scale, double pscale,
                               float* r32, float* p32, float* x32, const float* invd, int64_t n, hipStream_t s)
{
    const int g = grid_for<float>(n);
    hipLaunchKernelGGL(cg_replace32_kernel, dim3(g), dim3(BT), 0, s, r64, scale, pscale, r32, p32, x32, invd, n,
                       red);
    hipLaunchKernelGGL(cg_resume_kernel, dim3(1), dim3(BT), 0, s, st, red, g);
    return hipGetLastError();
}

static int grid_plain(int64_t n)
{
    const int64_t want = (n + BT - 1) / BT;
    return (int)(want < 2048 ? (want < 1 ? 1 : want) : 2048);
}

hipError_t launch_convert(const double* a, float* b, int64_t n, hipStream_t s)
{
    hipLaunchKernelGGL(convert_kernel, dim3(grid_plain(n)), dim3(BT), 0, s, a, b, n);
    return hipGetLastError();
}

hipError_t launch_promote_add(double* x, const float* d, double scale, int64_t n, hipStream_t s)
{
    hipLaunchKernelGGL(promote_add_kernel, dim3(grid_plain(n)), dim3(BT), 0, s, x, d, scale, n);
    return hipGetLastError();
}

}  // namespace vpp
