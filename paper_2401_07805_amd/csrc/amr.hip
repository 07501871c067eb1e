// Pressure operator on a once-refined mesh with hanging nodes (adaptive
// refinement of Sec. "Numerical framework", one level): kernels.
//
// The unknowns of the two lattices sit in one vector: the coarse lattice
// (entries [0, nc)) and the fine lattice over the whole box (entries [nc, n)).
// Most entries are identity rows (unused nodes of either lattice, constrained
// fine nodes, free unknowns on Dirichlet faces: y = x there, and gathers read
// them as zero), so the operator works on a packed vector: the free unknowns,
// then one value per constrained fine node, sum_p w_p x[src_p] over the nodes of
// the unrefined coarse cell it lies on, then a zero that stands for identity
// rows.  Launches of an apply:
//   expand: the packed vector (gather, constraints evaluated);
//   cells:  every active cell (an unrefined coarse cell, or one of the eight fine
//           cells of a refined one) gathers through a host-built index table and
//           applies the cell operator, plane per thread as apply variant 1 does,
//           a wave per group of cells, with the coefficient stored at set_phi;
//           its results go to a slot each;
//   csum:   every constrained node sums its cells' slots;
//   result: every free unknown sums its cells' slots and, where constrained
//           nodes draw on it, their sums with the same weights (C^T).
// All sums run in a fixed order, no atomics.  In the solver, expand is part of
// the direction update and result of the residual update.
//
// What bounds it: the dependent index -> value loads (three round trips) at 0.5 M
// unknowns, hence lists without weights for the cells' slots and one launch for
// all constrained nodes.  The version this replaces ran one cell per thread on
// the two-lattice vector (constraint lists followed inside the cell, CG vectors
// of 2.4 M entries for 0.5 M unknowns): 32^3 Q2 with 5,064 refined cells 125 us
// per CG iteration, 40 now; the apply alone 85 -> 43 us.
#include "amr.h"

#include <algorithm>

#include "apply_plane.h"
#include "cg_device.h"

namespace vpp {

template <int K>
__device__ __forceinline__ int64_t amr_local(const MeshArgs& m, int64_t base, int a)
{
    constexpr int N = K + 1;
    const int a0 = a % N, a1 = (a / N) % N, a2 = a / (N * N);
    return base + a0 + (int64_t)m.nn[0] * (a1 + (int64_t)m.nn[1] * a2);
}

// Lattice index of local node 0 of cell idx of lattice m.
template <int K>
__device__ __forceinline__ int64_t amr_base(const MeshArgs& m, int idx)
{
    const int cx = idx % m.nc[0], cy = (idx / m.nc[0]) % m.nc[1], cz = idx / (m.nc[0] * m.nc[1]);
    return node_index(m, (int64_t)K * cx, (int64_t)K * cy, (int64_t)K * cz);
}

// Constraint list of local node gl of a cell of lattice FINE (-1: none).
template <bool FINE>
__device__ __forceinline__ int amr_kind(const AmrArgs& a, int64_t gl)
{
    if constexpr (FINE) return a.fkind[gl];
    else return -1;
}

template <int K, int HV>
__device__ __forceinline__ void amr_coefficient(const MeshArgs& m, int64_t base, int64_t off,
                                                const double* __restrict__ phi,
                                                double (&cw)[(K + 1) * (K + 1) * (K + 1)])
{
    constexpr int N3 = (K + 1) * (K + 1) * (K + 1);
#pragma unroll
    for (int q = 0; q < N3; ++q) cw[q] = phi[off + amr_local<K>(m, base, q)];
    sweep3<K, MS, false, 0>(cw);
    sweep3<K, MS, false, 1>(cw);
    sweep3<K, MS, false, 2>(cw);
    coef_weights3<K, HV>(m, cw);
}

// Cells of a workgroup of the cells kernel: four waves of whole cells each.
template <int K>
struct AmrGeo {
    static constexpr int N = K + 1, CG = 64 / N, CB = 4 * CG, BLOCK = 256;
    using G = PlaneGeo<K, CB, 1, 1, true>;
    static_assert(G::CG == CG && G::NG == 4 && G::NTH == BLOCK, "four waves of CG cells");
};

// This thread's cell (index in the list of active cells) and plane.
template <int K>
struct AmrThread {
    using A = AmrGeo<K>;
    int e, ip, offx, offz;
    bool spare;   // repeats its wave's last thread
    __device__ __forceinline__ AmrThread()
    {
        const int w = threadIdx.x / 64, lane = threadIdx.x % 64;
        spare = lane >= A::CG * A::N;
        const int t = spare ? A::CG * A::N - 1 : lane;
        e = blockIdx.x * A::CB + w * A::CG + t / A::N;
        ip = t % A::N;
        offx = w * A::G::GB + t;
        offz = w * A::G::GB + ip * A::G::SZ + (t - ip);
    }
};

// Coefficient factors of every cell at its z-planes, in the threads' order of
// the cells kernel (value q of thread t of workgroup b at (b N^2 + q) 256 + t).
template <int K, int HV>
__global__ void __launch_bounds__(256) amr_coef_kernel(AmrArgs a, const double* __restrict__ phi)
{
    using G = typename AmrGeo<K>::G;
    constexpr int N = G::N, N2 = N * N;
    __shared__ double buf[G::NG * G::GB];
    // a.coef stands in the partials' place of the table
    VPP_BC_BEGIN((const double*)nullptr, (const double*)nullptr, phi, a.coef, (const double*)nullptr, buf, a.n,
                 (int64_t)gridDim.x * N2 * 256, 0, G::NG * G::GB);
    const AmrThread<K> th;
    double cw[N2];
    const bool in = th.e < a.ncells;
    const int code = in ? a.cells[th.e] : 0;
    const MeshArgs& m = code >= 0 ? a.mc : a.mf;
    if (in) {
        const int64_t base = amr_base<K>(m, code >= 0 ? code : -(code + 1)) + (code >= 0 ? 0 : a.nc) + th.ip;
        const int64_t nx = m.nn[0], nxy = (int64_t)m.nn[0] * m.nn[1];
#pragma unroll
        for (int l = 0; l < N; ++l)
#pragma unroll
            for (int j = 0; j < N; ++j) cw[j + N * l] = VPP_LD(&phi[base + nx * j + nxy * l], BC_PHI);
    } else {
#pragma unroll
        for (int q = 0; q < N2; ++q) cw[q] = 0.0;
    }
    sweep2<K, MS, false, 0>(cw);
    sweep2<K, MS, false, 1>(cw);
    put_x<G>(buf + th.offx, cw);
    plane_sync<G>();
    get_z<G>(buf + th.offz, cw);
    sweep2<K, MS, false, 0>(cw);
    double wz = 0.0;
#pragma unroll
    for (int i = 0; i < N; ++i)
        if (th.ip == i) wz = Tab<K>::t.w[i];
#pragma unroll
    for (int q = 0; q < N2; ++q) {
        const double c = coef_scaled<HV>(m, cw[q]) * (wz * (Tab<K>::t.w[q % N] * Tab<K>::t.w[q / N]));
        VPP_ST(&a.coef[((size_t)blockIdx.x * N2 + q) * 256 + threadIdx.x], BC_PART, in ? c : 0.0);
    }
}

// slots := the cell operator on the packed vector ext; with DOT also the
// workgroup's share of x . (A x).
template <int K, bool DOT>
__global__ void __launch_bounds__(256) amr_cells_kernel(AmrArgs a, const double* __restrict__ ext, double* dot_part,
                                                        const int* done)
{
    using G = typename AmrGeo<K>::G;
    constexpr int N = G::N, N2 = N * N;
    __shared__ double buf[G::NG * G::GB];
    // the packed vector as x, the result slots in the partials' place
    VPP_BC_BEGIN(ext, (const double*)nullptr, (const double*)nullptr, a.scratch, dot_part, buf,
                 (int64_t)a.nfree + a.ncon + 2, (int64_t)gridDim.x * N2 * 256, (int64_t)gridDim.x, G::NG * G::GB);
    if (done && *done) return;
    const AmrThread<K> th;
    const size_t at = (size_t)blockIdx.x * N2 * 256 + threadIdx.x;
    int idx[N2];
    double u[N2], cw[N2];
#pragma unroll
    for (int q = 0; q < N2; ++q) idx[q] = a.cidx[at + (size_t)q * 256];
#pragma unroll
    for (int q = 0; q < N2; ++q) cw[q] = a.coef[at + (size_t)q * 256];
#pragma unroll
    for (int q = 0; q < N2; ++q) u[q] = VPP_LD(&ext[idx[q]], BC_X);
    // the spacing ratios of both lattices are the same
    plane_operator<G, K, double, false>(a.mc, buf + th.offx, buf + th.offz, cw, 0.0, u);
    double d = 0.0;
    if (!th.spare) {
#pragma unroll
        for (int q = 0; q < N2; ++q) VPP_ST(&a.scratch[at + (size_t)q * 256], BC_PART, u[q]);
        if constexpr (DOT) {
            // gathered again: held across the operator they cost a wave per SIMD
#pragma unroll
            for (int q = 0; q < N2; ++q) d = fma(VPP_LD(&ext[a.cidx[at + (size_t)q * 256]], BC_X), u[q], d);
        }
    }
    if constexpr (DOT) {
        const double sum = block_sum<256>(d);
        if (threadIdx.x == 0) VPP_ST(&dot_part[blockIdx.x], BC_DOT, sum);
    }
}

// Sum of the slots idx[b .. e): all loaded before any is added, eight at a time;
// past the end the last one is read again, since a load under a condition waits
// for its index by itself (the same in amr_constrained; with
// amr_source_value's, PCG of 0.5 M unknowns at 32^3 Q2 15.5 -> 14.5 ms, 17x14x19 Q3
// 17.8 -> 15.1, 9x10x8 Q4 20.2 -> 16.3).
__device__ __forceinline__ double amr_slot_sum(const double* __restrict__ slots, const unsigned* __restrict__ idx, int b,
                                               int e)
{
    double v = 0.0;
    for (; b < e; b += 8) {
        double t[8];
#pragma unroll
        for (int k = 0; k < 8; ++k) t[k] = slots[idx[min(b + k, e - 1)]];
#pragma unroll
        for (int k = 0; k < 8; ++k)
            if (b + k < e) v += t[k];
    }
    return v;
}

__global__ void __launch_bounds__(BT) amr_csum_kernel(AmrArgs a, const int* done)
{
    if (done && *done) return;
    const int m = blockIdx.x * BT + threadIdx.x;
    if (m < a.ncon) a.csum[m] = amr_slot_sum(a.scratch, a.sidx, a.sptr[m], a.sptr[m + 1]);
}

// Source k (an unknown that constrained nodes draw on, up to a hundred of them)
// by kLanes consecutive lanes: its slots and terms dealt out to the lanes, summed
// by a butterfly; every lane receives (A x) there.  One lane per source would
// follow its terms one after another: 23.5 us for the update of 0.5 M unknowns at
// 32^3 Q2, against 15.0.
constexpr int kLanes = 8;
__device__ __forceinline__ double amr_source_value(const AmrArgs& a, int k, int i)
{
    const int lane = threadIdx.x % kLanes;
    const int f0 = a.fptr[i], f1 = a.fptr[i + 1], t0 = a.tptr[k], t1 = a.tptr[k + 1];
    double v = 0.0;
    for (int j = f0 + lane; j < f1; j += kLanes) v += a.scratch[a.fidx[j]];
    for (int b = t0 + lane; b < t1; b += 4 * kLanes) {
        double w[4], c[4];
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            const int j = min(b + u * kLanes, t1 - 1);
            w[u] = a.tw[j];
            c[u] = a.csum[a.tcon[j]];
        }
#pragma unroll
        for (int u = 0; u < 4; ++u)
            if (b + u * kLanes < t1) v = fma(w[u], c[u], v);
    }
#pragma unroll
    for (int o = kLanes / 2; o > 0; o >>= 1) v += __shfl_xor(v, o);
    return v;
}

// Calls f(i, (A x) at free unknown i) for every free unknown: the plain ones by
// workgroups below g, the sources by the others (amr_source_blocks).
template <typename F>
__device__ __forceinline__ void amr_each_unknown(const AmrArgs& a, int g, F&& f)
{
    if ((int)blockIdx.x < g) {
        for (int i = blockIdx.x * BT + threadIdx.x; i < a.nfree; i += g * BT)
        {
            const int b = a.fptr[i], e = a.fptr[i + 1];
            const bool src = a.issrc[i];
            if (!src) f(i, amr_slot_sum(a.scratch, a.fidx, b, e));
        }
        return;
    }
    const int k = ((blockIdx.x - g) * BT + threadIdx.x) / kLanes;
    const int i = k < a.nsrc ? a.src[k] : -1;
    const double v = i >= 0 ? amr_source_value(a, k, i) : 0.0;
    if (i >= 0 && threadIdx.x % kLanes == 0) f(i, v);
}

// sum_p w_p v(p) over constraint terms p of node m, p's loads batched.
template <typename I, typename F>
__device__ __forceinline__ double amr_constrained(const AmrArgs& a, int m, I&& index, F&& value)
{
    const int p1 = a.cptr[m + 1];
    double s = 0.0;
    for (int b = a.cptr[m]; b < p1; b += 8) {
        double w[8], x[8];
#pragma unroll
        for (int u = 0; u < 8; ++u) {
            const int p = min(b + u, p1 - 1), i = index(p);
            w[u] = a.cw[p];
            x[u] = value(max(i, 0));
            if (i < 0) x[u] = 0.0;
        }
#pragma unroll
        for (int u = 0; u < 8; ++u)
            if (b + u < p1) s = fma(w[u], x[u], s);
    }
    return s;
}

// ext := the packed form of x.
__global__ void __launch_bounds__(BT) amr_expand_kernel(AmrArgs a, const double* __restrict__ x)
{
    const int i = blockIdx.x * BT + threadIdx.x;
    if (i < a.nfree) a.ext[i] = x[a.fent[i]];
    const int m = i - a.nfree;
    if (m >= 0 && m < a.ncon) {
        a.ext[a.nfree + 1 + m] = amr_constrained(
            a, m, [&](int p) { return a.cpk[p] < 0 ? -1 : a.ccol[p]; }, [&](int64_t e) { return x[e]; });
    }
}

// y = x on identity rows (a grid-stride loop of the workgroups below g) and A x
// on the free unknowns.
__global__ void __launch_bounds__(BT) amr_result_kernel(AmrArgs a, int g, const double* __restrict__ x,
                                                        double* __restrict__ y)
{
    if ((int)blockIdx.x < g)
        for (int64_t e = (int64_t)blockIdx.x * BT + threadIdx.x; e < a.n; e += (int64_t)g * BT)
            if (a.ident[e]) y[e] = x[e];
    amr_each_unknown(a, g, [&](int i, double v) { y[a.fent[i]] = v; });
}

// ---------------------------------------------------------------------------
// Jacobi PCG on the packed vector.  All identity rows together are one more
// unknown (index nfree, operator and diagonal 1): their residual stays a
// multiple of the initial one, b - x0 there, so a single entry of the initial
// norm carries them through the recurrence, and the norms, scalars and stop
// decisions are those of the full system.

// r = b - A x, p = D^-1 r (in ext), x packed, and partials of r.r, r.D^-1 r and of
// the identity rows' residual; ext holds x on entry (amr_expand_kernel).
__global__ void __launch_bounds__(BT) amr_cg_init_kernel(AmrArgs a, AmrCg w, int g, const double* __restrict__ b,
                                                         const double* __restrict__ x)
{
    double rr = 0.0, rz = 0.0, id = 0.0, unused = 0.0;
    if ((int)blockIdx.x < g)
        for (int64_t e = (int64_t)blockIdx.x * BT + threadIdx.x; e < a.n; e += (int64_t)g * BT)
            if (a.ident[e]) {
                const double d = b[e] - x[e];
                id += d * d;
            }
    amr_each_unknown(a, g, [&](int i, double v) {
        const int e = a.fent[i];
        const double ri = b[e] - v, zi = ri * a.invd[i];
        w.r[i] = ri;
        w.x[i] = x[e];
        a.ext[i] = zi;
        rr += ri * ri;
        rz += ri * zi;
    });
    block_sum2<BT>(rr, rz);
    __syncthreads();
    block_sum2<BT>(id, unused);
    if (threadIdx.x == 0) {
        w.red[blockIdx.x] = rr;
        w.red[w.nred + blockIdx.x] = rz;
        w.idpart[blockIdx.x] = id;
    }
}

__global__ void __launch_bounds__(BT) amr_cg_init_finish_kernel(AmrArgs a, AmrCg w, int ng)
{
    double rr, rz, id = 0.0, unused = 0.0;
    sum_partials(w.red, ng, rr, rz, w.nred);
    for (int i = threadIdx.x; i < ng; i += BT) id += w.idpart[i];
    __syncthreads();
    block_sum2<BT>(id, unused);
    if (threadIdx.x == 0) {
        const double rho = sqrt(id);
        w.r[a.nfree] = rho;
        a.ext[a.nfree] = rho;
        w.x[a.nfree] = 0.0;
        *w.rho = rho;
        w.st->rr_last = rr + id;
        w.st->rz[0] = rz + id;
    }
}

// Constrained values of p (in ext) from its free entries.
__global__ void __launch_bounds__(BT) amr_constrain_kernel(AmrArgs a)
{
    const int m = blockIdx.x * BT + threadIdx.x;
    if (m >= a.ncon) return;
    a.ext[a.nfree + 1 + m] = amr_constrained(
        a, m, [&](int p) { return a.cpk[p]; }, [&](int i) { return a.ext[i]; });
}

// The residual update, (A p) formed on the way (amr_each_unknown's split).
__global__ void __launch_bounds__(BT) amr_update_kernel(AmrArgs a, AmrCg w, int par, int ndot, int g)
{
    // the identity unknown's own term of p.Ap joins the cells' partials (every
    // workgroup adds it, in the same place of the sum)
    const double pe = a.ext[a.nfree];
    double alpha;
    if (!update_alpha(blockIdx.x, w.st, par, w.dot, ndot, alpha, pe * pe)) return;
    double rr = 0.0, rz = 0.0;
    auto update = [&](int i, double q) {
        const double ri = fma(-alpha, q, w.r[i]);
        w.r[i] = ri;
        rr += ri * ri;
        rz += ri * (ri * a.invd[i]);
    };
    amr_each_unknown(a, g, update);
    if (blockIdx.x == 0 && threadIdx.x == 0) update(a.nfree, pe);
    block_sum2<BT>(rr, rz);
    write_partials(w.red, rr, rz, blockIdx.x, w.nred);
}

// The direction update of the packed vector (workgroups below g), and p's
// constrained values by the same recurrence, C z + beta (C p) (the others).  They
// are not formed from p again: its rounding in C p shrinks and grows with p itself
// (run 1000 iterations past convergence, 32^3 Q2, the residual of the result is 1 to
// 15 10^-16 of b, 8 10^-16 with C p formed anew each time).
__global__ void __launch_bounds__(BT) amr_pupdate_kernel(AmrArgs a, AmrCg w, int par, int ng, int g)
{
    if ((int)blockIdx.x < g) {
        pupdate_body<double>(blockIdx.x, g, w.st, par, w.red, ng, w.x, w.r, a.ext, a.invd, a.nfree + 1, w.nred);
        return;
    }
    const int halt = w.st->halt[par], brk = w.st->breakdown;
    const double rz_par = w.st->rz[par];
    if (halt || brk) return;
    const int m = (blockIdx.x - g) * BT + threadIdx.x;
    double s = 0.0, old = 0.0;
    if (m < a.ncon) {
        old = a.ext[a.nfree + 1 + m];
        s = amr_constrained(
            a, m, [&](int p) { return a.cpk[p]; }, [&](int i) { return w.r[i] * a.invd[i]; });
    }
    double rr, rzn;
    sum_partials(w.red, ng, rr, rzn, w.nred);
    if (m < a.ncon) a.ext[a.nfree + 1 + m] = fma(rzn / rz_par, old, s);
}

// x of the full vector: the free unknowns, and on identity rows the initial
// guess moved by the identity unknown's share of b - x0.
__global__ void __launch_bounds__(BT) amr_unpack_kernel(AmrArgs a, AmrCg w, const double* __restrict__ b,
                                                        double* __restrict__ x)
{
    const double rho = *w.rho;
    const double s = rho > 0.0 ? w.x[a.nfree] / rho : 0.0;
    for (int64_t g = (int64_t)blockIdx.x * BT + threadIdx.x; g < a.n; g += (int64_t)gridDim.x * BT) {
        const int i = a.pidx[g];
        if (i >= 0) x[g] = w.x[i];
        else if (s != 0.0) x[g] = fma(s, b[g] - x[g], x[g]);
    }
}

__global__ void __launch_bounds__(BT) amr_pack_invd_kernel(AmrArgs a, const double* __restrict__ inv64)
{
    for (int i = blockIdx.x * BT + threadIdx.x; i <= a.nfree; i += gridDim.x * BT)
        a.invd[i] = i < a.nfree ? inv64[a.fent[i]] : 1.0;
}

// Diagonal of C^T K_e C for one cell: K_aa from the squared 1D tables for the
// free nodes; for the coarse nodes that constrained nodes of the cell draw on,
// e_i^T K_e e_i with e_i the cell vector of node i's weights, K_e applied by
// the cell operator (each such coarse node once per cell).
template <int K, int HV, bool FINE>
__device__ __forceinline__ void amr_diag_cell(const AmrArgs& a, const MeshArgs& m, int idx, int e,
                                              const double* __restrict__ phi)
{
    constexpr int N3 = (K + 1) * (K + 1) * (K + 1);
    const int64_t base = amr_base<K>(m, idx), off = FINE ? a.nc : 0;
    double cw[N3];
    amr_coefficient<K, HV>(m, base, off, phi, cw);
    {
        double A[N3], Z[N3], Y[N3], out[N3];
#pragma unroll
        for (int q = 0; q < N3; ++q) A[q] = cw[q];
#pragma unroll
        for (int q = 0; q < N3; ++q) Z[q] = A[q];
        sweep3<K, MS2, true, 2>(Z);
#pragma unroll
        for (int q = 0; q < N3; ++q) Y[q] = Z[q];
        sweep3<K, MS2, true, 1>(Y);
        sweep3<K, MD2, true, 0>(Y);
#pragma unroll
        for (int q = 0; q < N3; ++q) out[q] = m.rd[0] * Y[q];
#pragma unroll
        for (int q = 0; q < N3; ++q) Y[q] = Z[q];
        sweep3<K, MD2, true, 1>(Y);
        sweep3<K, MS2, true, 0>(Y);
#pragma unroll
        for (int q = 0; q < N3; ++q) out[q] = fma(m.rd[1], Y[q], out[q]);
        sweep3<K, MD2, true, 2>(A);
        sweep3<K, MS2, true, 1>(A);
        sweep3<K, MS2, true, 0>(A);
#pragma unroll
        for (int q = 0; q < N3; ++q) out[q] = fma(m.rd[2], A[q], out[q]);
#pragma unroll
        for (int q = 0; q < N3; ++q) {
            const int64_t gl = amr_local<K>(m, base, q);
            if (amr_kind<FINE>(a, gl) < 0) a.scratch[(size_t)q * (size_t)a.ncells + (size_t)e] = out[q];
        }
    }
    if constexpr (FINE) {
        // coarse nodes reached through constraints: visit each (node q, term p)
        // pair and handle its coarse node at its first occurrence in that order
        // (the host numbers the slots in the same order)
        int64_t slot = a.nfree_slots + a.soff[e];
        for (int q = 0; q < N3; ++q) {
            const int kq = a.fkind[amr_local<K>(m, base, q)];
            if (kq < 0) continue;
            for (int p = a.cptr[kq]; p < a.cptr[kq + 1]; ++p) {
                const int src = a.ccol[p];
                bool seen = false;
                for (int q2 = 0; q2 <= q && !seen; ++q2) {
                    const int k2 = a.fkind[amr_local<K>(m, base, q2)];
                    if (k2 < 0) continue;
                    const int pend = (q2 == q) ? p : a.cptr[k2 + 1];
                    for (int p2 = a.cptr[k2]; p2 < pend; ++p2)
                        if (a.ccol[p2] == src) seen = true;
                }
                if (seen) continue;
                double ev[N3], kv[N3];
                for (int r = 0; r < N3; ++r) {
                    double w = 0.0;
                    const int kr = a.fkind[amr_local<K>(m, base, r)];
                    if (kr >= 0)
                        for (int p2 = a.cptr[kr]; p2 < a.cptr[kr + 1]; ++p2)
                            if (a.ccol[p2] == src) w += a.cw[p2];
                    ev[r] = w;
                    kv[r] = w;
                }
                cell_operator<K, double>(m, cw, kv);
                double d = 0.0;
                for (int r = 0; r < N3; ++r) d = fma(ev[r], kv[r], d);
                a.scratch[slot++] = d;
            }
        }
    }
}

template <int K, int HV>
__global__ void __launch_bounds__(64) amr_diag_kernel(AmrArgs a, const double* __restrict__ phi)
{
    const int e = blockIdx.x * blockDim.x + threadIdx.x;
    if (e >= a.ncells) return;
    const int code = a.cells[e];
    if (code >= 0) amr_diag_cell<K, HV, false>(a, a.mc, code, e, phi);
    else amr_diag_cell<K, HV, true>(a, a.mf, -(code + 1), e, phi);
}

// diag = 1 on identity rows, else the sum of its cell slots; then the FP64
// and FP32 inverses.
__global__ void amr_fix_diag_kernel(AmrArgs a, double* __restrict__ diag, double* __restrict__ inv64,
                                    float* __restrict__ inv32)
{
    for (int64_t g = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; g < a.n; g += (int64_t)gridDim.x * blockDim.x) {
        double s = 0.0;
        for (int j = a.dptr[g]; j < a.dptr[g + 1]; ++j) s += a.scratch[a.didx[j]];
        const double d = a.ident[g] ? 1.0 : s;
        diag[g] = d;
        inv64[g] = 1.0 / d;
        inv32[g] = (float)(1.0 / d);
    }
}

static int stream_blocks(int64_t n)
{
    const int64_t want = (n + 255) / 256;
    return (int)(want < 8192 ? (want < 1 ? 1 : want) : 8192);
}

#define VPP_AMR_SWITCH(KERNEL, ...)                                                                       \
    switch (k * 4 + a.mc.heaviside) {                                                                     \
    case 8: hipLaunchKernelGGL((KERNEL<2, 0>), dim3(blocks), dim3(64), 0, s, a, __VA_ARGS__); break;    \
    case 9: hipLaunchKernelGGL((KERNEL<2, 1>), dim3(blocks), dim3(64), 0, s, a, __VA_ARGS__); break;    \
    case 10: hipLaunchKernelGGL((KERNEL<2, 2>), dim3(blocks), dim3(64), 0, s, a, __VA_ARGS__); break;   \
    case 11: hipLaunchKernelGGL((KERNEL<2, 3>), dim3(blocks), dim3(64), 0, s, a, __VA_ARGS__); break;   \
    case 12: hipLaunchKernelGGL((KERNEL<3, 0>), dim3(blocks), dim3(64), 0, s, a, __VA_ARGS__); break;   \
    case 13: hipLaunchKernelGGL((KERNEL<3, 1>), dim3(blocks), dim3(64), 0, s, a, __VA_ARGS__); break;   \
    case 14: hipLaunchKernelGGL((KERNEL<3, 2>), dim3(blocks), dim3(64), 0, s, a, __VA_ARGS__); break;   \
    case 15: hipLaunchKernelGGL((KERNEL<3, 3>), dim3(blocks), dim3(64), 0, s, a, __VA_ARGS__); break;   \
    case 16: hipLaunchKernelGGL((KERNEL<4, 0>), dim3(blocks), dim3(64), 0, s, a, __VA_ARGS__); break;   \
    case 17: hipLaunchKernelGGL((KERNEL<4, 1>), dim3(blocks), dim3(64), 0, s, a, __VA_ARGS__); break;   \
    case 18: hipLaunchKernelGGL((KERNEL<4, 2>), dim3(blocks), dim3(64), 0, s, a, __VA_ARGS__); break;   \
    case 19: hipLaunchKernelGGL((KERNEL<4, 3>), dim3(blocks), dim3(64), 0, s, a, __VA_ARGS__); break;   \
    default: return hipErrorInvalidValue;                                                                 \
    }

unsigned long long bounds_count_amr() { return bc_count_here(); }

int amr_cells_per_block(int k) { return k == 2 ? AmrGeo<2>::CB : (k == 3 ? AmrGeo<3>::CB : AmrGeo<4>::CB); }

static int amr_cell_blocks(int k, const AmrArgs& a)
{
    return (a.ncells + amr_cells_per_block(k) - 1) / amr_cells_per_block(k);
}

template <bool DOT>
static hipError_t launch_amr_cells(int k, const AmrArgs& a, double* dot_part, const int* done, hipStream_t s)
{
    const dim3 g(amr_cell_blocks(k, a)), b(256);
    if (g.x == 0) return hipSuccess;
    switch (k) {
    case 2: hipLaunchKernelGGL((amr_cells_kernel<2, DOT>), g, b, 0, s, a, a.ext, dot_part, done); break;
    case 3: hipLaunchKernelGGL((amr_cells_kernel<3, DOT>), g, b, 0, s, a, a.ext, dot_part, done); break;
    case 4: hipLaunchKernelGGL((amr_cells_kernel<4, DOT>), g, b, 0, s, a, a.ext, dot_part, done); break;
    default: return hipErrorInvalidValue;
    }
    return hipGetLastError();
}

static int blocks_of(int64_t n) { return (int)((n + BT - 1) / BT); }

// Workgroups of the sources.
static int amr_source_blocks(const AmrArgs& a) { return blocks_of((int64_t)a.nsrc * kLanes); }

int amr_red_blocks(const AmrArgs& a) { return 768 + amr_source_blocks(a); }

static hipError_t launch_amr_csum(const AmrArgs& a, const int* done, hipStream_t s)
{
    if (a.ncon > 0) hipLaunchKernelGGL(amr_csum_kernel, dim3(blocks_of(a.ncon)), dim3(BT), 0, s, a, done);
    return hipGetLastError();
}

// expand, cells, csum: what every use of A x on a full vector starts with.
static hipError_t launch_amr_parts(int k, const AmrArgs& a, const double* x, hipStream_t s)
{
    hipError_t e;
    const int n = a.nfree + a.ncon;
    if (n > 0) hipLaunchKernelGGL(amr_expand_kernel, dim3(blocks_of(n)), dim3(BT), 0, s, a, x);
    if ((e = hipGetLastError()) != hipSuccess || (e = launch_amr_cells<false>(k, a, nullptr, nullptr, s)) != hipSuccess)
        return e;
    return launch_amr_csum(a, nullptr, s);
}

hipError_t launch_amr_apply(int k, const AmrArgs& a, const double* x, double* y, hipStream_t s)
{
    const hipError_t e = launch_amr_parts(k, a, x, s);
    if (e != hipSuccess) return e;
    const int g = stream_blocks(a.n);
    hipLaunchKernelGGL(amr_result_kernel, dim3(g + amr_source_blocks(a)), dim3(BT), 0, s, a, g, x, y);
    return hipGetLastError();
}

int amr_dot_partials(int k, const AmrArgs& a) { return amr_cell_blocks(k, a); }

hipError_t launch_amr_cg_init(int k, const AmrArgs& a, const AmrCg& w, const double* b, const double* x, hipStream_t s)
{
    hipError_t e = launch_amr_parts(k, a, x, s);
    if (e != hipSuccess) return e;
    const int g = blocks_of(std::min<int64_t>(a.n, 768 * BT)), all = g + amr_source_blocks(a);
    hipLaunchKernelGGL(amr_cg_init_kernel, dim3(all), dim3(BT), 0, s, a, w, g, b, x);
    hipLaunchKernelGGL(amr_cg_init_finish_kernel, dim3(1), dim3(BT), 0, s, a, w, all);
    if (a.ncon > 0) hipLaunchKernelGGL(amr_constrain_kernel, dim3(blocks_of(a.ncon)), dim3(BT), 0, s, a);
    return hipGetLastError();
}

hipError_t launch_amr_cg_step(int k, const AmrArgs& a, const AmrCg& w, int par, hipStream_t s)
{
    hipError_t e;
    const int* done = &w.st->halt[par];
    if ((e = launch_amr_cells<true>(k, a, w.dot, done, s)) != hipSuccess || (e = launch_amr_csum(a, done, s)) != hipSuccess)
        return e;
    const int n = a.nfree + 1, g = std::min(768, blocks_of(n)), all = g + amr_source_blocks(a);
    hipLaunchKernelGGL(amr_update_kernel, dim3(all), dim3(BT), 0, s, a, w, par, amr_dot_partials(k, a), g);
    const int gp = std::min(512, blocks_of((n + 1) / 2));
    hipLaunchKernelGGL(amr_pupdate_kernel, dim3(gp + blocks_of(a.ncon)), dim3(BT), 0, s, a, w, par, all, gp);
    return hipGetLastError();
}

hipError_t launch_amr_unpack(const AmrArgs& a, const AmrCg& w, const double* b, double* x, hipStream_t s)
{
    hipLaunchKernelGGL(amr_unpack_kernel, dim3(stream_blocks(a.n)), dim3(BT), 0, s, a, w, b, x);
    return hipGetLastError();
}

hipError_t launch_amr_coef(int k, const AmrArgs& a, const double* phi, hipStream_t s)
{
    const dim3 g(amr_cell_blocks(k, a)), b(256);
    if (g.x == 0) return hipSuccess;
#define VPP_AMR_COEF(K, HV) hipLaunchKernelGGL((amr_coef_kernel<K, HV>), g, b, 0, s, a, phi)
#define VPP_AMR_COEF_K(K)                            \
    switch (a.mc.heaviside) {                        \
    case 0: VPP_AMR_COEF(K, 0); break;               \
    case 1: VPP_AMR_COEF(K, 1); break;               \
    case 2: VPP_AMR_COEF(K, 2); break;               \
    case 3: VPP_AMR_COEF(K, 3); break;               \
    default: return hipErrorInvalidValue;            \
    }
    switch (k) {
    case 2: VPP_AMR_COEF_K(2) break;
    case 3: VPP_AMR_COEF_K(3) break;
    case 4: VPP_AMR_COEF_K(4) break;
    default: return hipErrorInvalidValue;
    }
#undef VPP_AMR_COEF_K
#undef VPP_AMR_COEF
    return hipGetLastError();
}

hipError_t launch_amr_diag(int k, const AmrArgs& a, const double* phi, double* diag, double* inv64, float* inv32,
                           hipStream_t s)
{
    hipError_t e;
    if (a.ncells > 0) {
        const int blocks = (a.ncells + 63) / 64;
        VPP_AMR_SWITCH(amr_diag_kernel, phi)
        if ((e = hipGetLastError()) != hipSuccess) return e;
    }
    hipLaunchKernelGGL(amr_fix_diag_kernel, dim3(stream_blocks(a.n)), dim3(256), 0, s, a, diag, inv64, inv32);
    hipLaunchKernelGGL(amr_pack_invd_kernel, dim3(stream_blocks(a.nfree + 1)), dim3(BT), 0, s, a, inv64);
    return hipGetLastError();
}

#undef VPP_AMR_SWITCH

}  // namespace vpp
