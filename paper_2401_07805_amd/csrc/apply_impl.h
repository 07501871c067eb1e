// Matrix-free application of the variable-coefficient pressure-Poisson
// operator, y = sum_e R_e^T A_e R_e x (Sec. "Numerical framework"), with
// A_e = sum_q W_q c(phi_h(x_q)) B_q^T B_q evaluated on the fly by sum
// factorisation over the tensor-product Q_k basis and (k+1)^3 Gauss points.
//
// A workgroup owns a tile of TX x TY x TZ cells.  Thread mappings (the
// autotuner picks one per problem and precision):
//   variant 4, cell per thread: all (k+1)^3 values of a cell live in registers,
//              every sweep is register-only; the cell results are exchanged
//              through an LDS slot array without atomics (k = 2);
//   variant 0, cell per thread with the tile's node block accumulated by LDS
//              atomic adds (k = 2);
//   variant 2, half a cell per thread (k = 3): an even/odd lane pair holds a
//              cell's z-planes, z sweeps by DPP lane swaps;
//   variant 1, plane per thread: k+1 threads share a cell, each holding one
//              plane of (k+1)^2 values, an x-plane for the y and z sweeps and a
//              z-plane for the x sweeps, the planes turned through LDS (all k).
// Nodes that only this tile touches are written with plain stores; nodes on
// planes shared with neighbouring tiles are written as per-tile partials and
// summed, in a fixed order, by the assembly kernel (apply_misc.hip), so the
// result does not depend on scheduling.  Dirichlet rows get y_i = x_i
// (identity rows of A_D); Dirichlet columns are dropped by zeroing those
// entries of x at the gather.
#pragma once
#include "kernels.h"
#include "shared_nodes.h"
#include "bounds.h"

namespace vpp {

// Dirichlet faces touched by a cell: bit f set if the cell lies on Dirichlet face f.
__device__ __forceinline__ int cell_dirichlet_faces(const MeshArgs& m, int cx, int cy, int cz)
{
    int f = 0;
    if (cx == 0) f |= 1;
    if (cx == m.nc[0] - 1) f |= 2;
    if (cy == 0) f |= 4;
    if (cy == m.nc[1] - 1) f |= 8;
    if (cz == 0) f |= 16;
    if (cz == m.nc[2] - 1) f |= 32;
    return f & m.bcmask;
}

template <int K>
__device__ __forceinline__ bool local_dirichlet(int faces, int a0, int a1, int a2)
{
    return ((faces & 1) && a0 == 0) || ((faces & 2) && a0 == K) || ((faces & 4) && a1 == 0) ||
           ((faces & 8) && a1 == K) || ((faces & 16) && a2 == 0) || ((faces & 32) && a2 == K);
}

template <int K, typename T, typename S>
__device__ __forceinline__ void gather_cell(const MeshArgs& m, const S* __restrict__ x, int cx, int cy,
                                            int cz, int faces, T (&u)[(K + 1) * (K + 1) * (K + 1)])
{
    constexpr int N = K + 1;
    const int64_t nx = m.nn[0], nxy = (int64_t)m.nn[0] * m.nn[1];
    const int64_t base = node_index(m, (int64_t)K * cx, (int64_t)K * cy, (int64_t)K * cz);
#pragma unroll
    for (int a2 = 0; a2 < N; ++a2)
#pragma unroll
        for (int a1 = 0; a1 < N; ++a1)
#pragma unroll
            for (int a0 = 0; a0 < N; ++a0)
                u[a0 + N * (a1 + N * a2)] = T(VPP_LD(&x[base + a0 + nx * a1 + nxy * a2], BC_IN));
    if (faces) {
#pragma unroll
        for (int a2 = 0; a2 < N; ++a2)
#pragma unroll
            for (int a1 = 0; a1 < N; ++a1)
#pragma unroll
                for (int a0 = 0; a0 < N; ++a0)
                    if (local_dirichlet<K>(faces, a0, a1, a2)) u[a0 + N * (a1 + N * a2)] = T(0);
    }
}

// A wave-uniform 64-bit value moved into scalar registers, so that addresses
// built from it use the scalar-base + 32-bit-lane-offset form of global memory
// instructions (no 64-bit vector address arithmetic per access).
__device__ __forceinline__ int64_t uniform_i64(int64_t v)
{
    const unsigned lo = __builtin_amdgcn_readfirstlane((unsigned)(uint64_t)v);
    const unsigned hi = __builtin_amdgcn_readfirstlane((unsigned)((uint64_t)v >> 32));
    return (int64_t)(((uint64_t)hi << 32) | lo);
}

template <typename S>
__device__ __forceinline__ S* at_byte(S* base, unsigned off)
{
    return reinterpret_cast<S*>(reinterpret_cast<char*>(base) + off);
}
template <typename S>
__device__ __forceinline__ const S* at_byte(const S* base, unsigned off)
{
    return reinterpret_cast<const S*>(reinterpret_cast<const char*>(base) + off);
}

// Gather of a cell's nodal values from a wave-uniform tile base `tb` (node of
// the tile's first cell) and the lane's byte offset `lane_b` of its cell; row
// offsets are uniform, so every load shares one offset register.
template <int K, typename T, typename S>
__device__ __forceinline__ void gather_cell_t(const S* __restrict__ tb, unsigned lane_b, int nx, int nxy, int faces,
                                              T (&u)[(K + 1) * (K + 1) * (K + 1)])
{
    constexpr int N = K + 1;
#pragma unroll
    for (int a2 = 0; a2 < N; ++a2)
#pragma unroll
        for (int a1 = 0; a1 < N; ++a1) {
            // one address per row: its values are adjacent in memory to the compiler
            // too and come as 16-byte loads (k = 2: 36 loads instead of 54 for x and
            // phi; 64^3 Q2 apply 29.4 -> 28.7 us, FP32 29.7 -> 27.7 with cold caches)
            const S* row = at_byte(tb + (nx * a1 + nxy * a2), lane_b);
#pragma unroll
            for (int a0 = 0; a0 < N; ++a0) u[a0 + N * (a1 + N * a2)] = T(VPP_LD(&row[a0], BC_IN));
        }
    if (faces) {
#pragma unroll
        for (int a2 = 0; a2 < N; ++a2)
#pragma unroll
            for (int a1 = 0; a1 < N; ++a1)
#pragma unroll
                for (int a0 = 0; a0 < N; ++a0)
                    if (local_dirichlet<K>(faces, a0, a1, a2)) u[a0 + N * (a1 + N * a2)] = T(0);
    }
}

// Scaled coefficient factor cw_q = c'(phi_h(x_q)) wref_q of a cell from nodal phi.
template <int K, int HV, typename T>
__device__ __forceinline__ void cell_coefficient(const MeshArgs& m, const T* __restrict__ phi, int cx,
                                                 int cy, int cz, T (&cw)[(K + 1) * (K + 1) * (K + 1)])
{
    gather_cell<K>(m, phi, cx, cy, cz, 0, cw);
    sweep3<K, MS, false, 0>(cw);
    sweep3<K, MS, false, 1>(cw);
    sweep3<K, MS, false, 2>(cw);
    coef_weights3<K, HV>(m, cw);
}

// Cell operator on registers: u (nodal values, Dirichlet entries zeroed) is
// replaced by A_e u.
//   forward:  u_q = (S x S x S) u,  g_d = Dc along d of u_q   (collocation derivative)
//   Gauss point: f_d = cw rd[d] g_d
//   backward: v = sum_d Dc_d^T f_d (+ mu hx hy hz wref_q u_q with MASS),
//             A_e u = (S^T x S^T x S^T) v
// The mass term is added where the last derivative pass still holds u_q, so it
// keeps no value alive for longer.
template <int K, typename T, bool MASS = false>
__device__ __forceinline__ void cell_operator(const MeshArgs& m, const T (&cw)[(K + 1) * (K + 1) * (K + 1)],
                                              T (&u)[(K + 1) * (K + 1) * (K + 1)])
{
    constexpr int N = K + 1, N3 = N * N * N;
    sweep3<K, MS, false, 0>(u);
    sweep3<K, MS, false, 1>(u);
    sweep3<K, MS, false, 2>(u);
    T v[N3];
    // rd[0] is 1 by construction (the x spacing is the reference length)
    const T r1 = T(m.rd[1]), r2 = T(m.rd[2]);
#pragma unroll
    for (int i2 = 0; i2 < N; ++i2)
#pragma unroll
        for (int i1 = 0; i1 < N; ++i1) {
            T in[N], g[N], o[N];
#pragma unroll
            for (int a = 0; a < N; ++a) in[a] = u[a + N * (i1 + N * i2)];
            line<K, MDC, false>(in, g);
#pragma unroll
            for (int a = 0; a < N; ++a) g[a] *= cw[a + N * (i1 + N * i2)];
            line<K, MDC, true>(g, o);
#pragma unroll
            for (int a = 0; a < N; ++a) v[a + N * (i1 + N * i2)] = o[a];
        }
#pragma unroll
    for (int i2 = 0; i2 < N; ++i2)
#pragma unroll
        for (int i0 = 0; i0 < N; ++i0) {
            T in[N], g[N], o[N];
#pragma unroll
            for (int a = 0; a < N; ++a) in[a] = u[i0 + N * (a + N * i2)];
            line<K, MDC, false>(in, g);
#pragma unroll
            for (int a = 0; a < N; ++a) g[a] *= cw[i0 + N * (a + N * i2)] * r1;
#pragma unroll
            for (int a = 0; a < N; ++a) o[a] = v[i0 + N * (a + N * i2)];
            line_acc<K, MDC, true>(g, o);
#pragma unroll
            for (int a = 0; a < N; ++a) v[i0 + N * (a + N * i2)] = o[a];
        }
#pragma unroll
    for (int i1 = 0; i1 < N; ++i1)
#pragma unroll
        for (int i0 = 0; i0 < N; ++i0) {
            T in[N], g[N], o[N];
#pragma unroll
            for (int a = 0; a < N; ++a) in[a] = u[i0 + N * (i1 + N * a)];
            line<K, MDC, false>(in, g);
#pragma unroll
            for (int a = 0; a < N; ++a) g[a] *= cw[i0 + N * (i1 + N * a)] * r2;
#pragma unroll
            for (int a = 0; a < N; ++a) o[a] = v[i0 + N * (i1 + N * a)];
            line_acc<K, MDC, true>(g, o);
            if constexpr (MASS) {
                const T ms = T(m.mass);
#pragma unroll
                for (int a = 0; a < N; ++a) o[a] = fma(ms * T(wref<K>(i0, i1, a)), in[a], o[a]);
            }
#pragma unroll
            for (int a = 0; a < N; ++a) v[i0 + N * (i1 + N * a)] = o[a];
        }
    sweep3<K, MS, true, 2>(v);
    sweep3<K, MS, true, 1>(v);
    sweep3<K, MS, true, 0>(v);
#pragma unroll
    for (int a = 0; a < N3; ++a) u[a] = v[a];
}

// ---------------------------------------------------------------------------
// Tile geometry and the write-out of a tile's node block.

struct TileCoord {
    int t[3];      // tile coordinates
    int n0[3];     // first node of the tile's block
    int ext[3];    // valid block extent (nodes) per direction
};

template <int K, int TX, int TY, int TZ>
__device__ __forceinline__ TileCoord tile_coord(const MeshArgs& m, int tile)
{
    TileCoord c;
    c.t[0] = tile % m.ntile[0];
    c.t[1] = (tile / m.ntile[0]) % m.ntile[1];
    c.t[2] = tile / (m.ntile[0] * m.ntile[1]);
    const int T3[3] = {TX, TY, TZ};
#pragma unroll
    for (int d = 0; d < 3; ++d) {
        c.n0[d] = K * T3[d] * c.t[d];
        c.ext[d] = K * min(T3[d], m.nc[d] - T3[d] * c.t[d]) + 1;
    }
    return c;
}

// Workgroup sum of one double per thread (LDS tree in a fixed order, valid for
// any NT including partial waves); the result is returned to thread 0.
template <int NT>
__device__ __forceinline__ double block_sum(double v)
{
    constexpr int P = NT <= 64 ? 64 : (NT <= 128 ? 128 : (NT <= 256 ? 256 : (NT <= 512 ? 512 : 1024)));
    static_assert(NT <= 1024, "workgroup too large");
    __shared__ double red[P];
    __syncthreads();
    red[threadIdx.x] = v;
    for (int i = NT + threadIdx.x; i < P; i += NT) red[i] = 0.0;
    __syncthreads();
#pragma unroll
    for (int s = P / 2; s > 0; s >>= 1) {
        if ((int)threadIdx.x < s) red[threadIdx.x] += red[threadIdx.x + s];
        __syncthreads();
    }
    return red[0];
}

// Write-out by cell ownership: a cell writes the nodes of its block with local
// index a_d in [0, K-1] along each direction, and also a_d = K when it is the
// last cell of the tile along d; every node of the tile block then has exactly
// one writer and all offsets are compile-time except the cell base.
//  - a node only this tile touches: y[g] = value;
//  - a node on a face shared with neighbouring tiles: this tile's partial value
//    goes to part[rank * nshared + f], where f is the node's position in the
//    enumeration of shared nodes (z planes, then y planes, then x planes; see
//    shared_nodes.h) and rank orders the 2, 4 or 8 tiles holding it (lower tile
//    first along each shared direction); the assembly kernel sums them;
//  - a node of a Dirichlet face: y[g] = x[g] (identity row), written by the
//    lowest-index tile that holds it.
// Both f and the rank follow from the tile coordinates and the face flags, with
// no division.  A0 restricts the x index to one plane (plane-per-thread
// kernels); -1 = all.  Returns this thread's share of x . (A x).
template <int K, typename T, int TX, int TY, int TZ, typename Get>
__device__ __forceinline__ double flush_owned_get(const MeshArgs& m, const TileCoord& tc, const Get& get, int lx,
                                                  int ly, int lz, int cx, int cy, int cz, int a0_only,
                                                  const T* __restrict__ x, T* __restrict__ y, T* __restrict__ part,
                                                  int64_t nshared, bool dot)
{
    const int faces = cell_dirichlet_faces(m, cx, cy, cz);
    const bool last[3] = {K * (lx + 1) == tc.ext[0] - 1, K * (ly + 1) == tc.ext[1] - 1, K * (lz + 1) == tc.ext[2] - 1};
    const bool has_lo[3] = {lx == 0 && tc.t[0] > 0, ly == 0 && tc.t[1] > 0, lz == 0 && tc.t[2] > 0};
    const bool has_hi[3] = {last[0] && tc.t[0] < m.ntile[0] - 1, last[1] && tc.t[1] < m.ntile[1] - 1,
                            last[2] && tc.t[2] < m.ntile[2] - 1};
    // 32-bit offsets: nodes relative to the tile's first node, f within the
    // shared-node enumeration (both < 2^31 since N < 2^31)
    const int nx = m.nn[0], nxy = m.nn[0] * m.nn[1];
    const int64_t tile0 = uniform_i64(node_index(m, tc.n0[0], tc.n0[1], tc.n0[2]));
    const T* __restrict__ xt = x + tile0;
    T* __restrict__ yt = y + tile0;
    const int i0 = K * cx, j0 = K * cy, l0 = K * cz;
    const unsigned lane_b = (unsigned)(K * lx + nx * K * ly + nxy * K * lz) * (unsigned)sizeof(T);
    // bases of the shared-node enumeration (z planes, y planes, x planes) for
    // the planes this cell can touch, lower (lo) or upper (hi) face of the tile
    const int t0 = tc.t[0], t1 = tc.t[1], t2 = tc.t[2];
    const int nbx = m.ntile[0] - 1, nby = m.ntile[1] - 1, nbz = m.ntile[2] - 1;
    const int cz_n = nbz * nxy;
    const int cy_n = nby * (m.nn[2] - nbz) * nx;
    const int ny_free = m.nn[1] - nby;
    const int fz = i0 + nx * j0 + nxy * (t2 - 1);                       // + nxy on the upper face
    const int fy = cz_n + i0 + nx * ((t1 - 1) + nby * (l0 - t2));        // + nx on the upper face
    const int fx = cz_n + cy_n + (t0 - 1) + nbx * ((j0 - t1) + ny_free * (l0 - t2));   // + 1 on the upper face
    const unsigned nsh = (unsigned)nshared;   // 8 nshared < 2^32 (checked on the host)
    double dsum = 0.0;
#pragma unroll
    for (int a2 = 0; a2 <= K; ++a2) {
        if (a2 == K && !last[2]) continue;
#pragma unroll
        for (int a1 = 0; a1 <= K; ++a1) {
            if (a1 == K && !last[1]) continue;
#pragma unroll
            for (int a0 = 0; a0 <= K; ++a0) {
                if (a0_only >= 0 && a0 != a0_only) continue;
                if (a0 == K && !last[0]) continue;
                const int row = a0 + nx * a1 + nxy * a2;   // uniform
                const bool lo0 = a0 == 0 && has_lo[0], lo1 = a1 == 0 && has_lo[1], lo2 = a2 == 0 && has_lo[2];
                const bool hi0 = a0 == K && has_hi[0], hi1 = a1 == K && has_hi[1], hi2 = a2 == K && has_hi[2];
                if (faces && local_dirichlet<K>(faces, a0, a1, a2)) {
                    // identity row: every tile holding the node writes the same x
                    const T xv = VPP_LD(at_byte(xt + row, lane_b), BC_X);
                    VPP_ST(at_byte(yt + row, lane_b), BC_Y, xv);
                    if (dot && !(lo0 || lo1 || lo2)) dsum += (double)xv * (double)xv;
                    continue;
                }
                const T v = get(a0, a1, a2, last);
                const bool s0 = lo0 || hi0, s1 = lo1 || hi1, s2 = lo2 || hi2;
                if (s0 || s1 || s2) {
                    int f;
                    if (s2) f = fz + (hi2 ? nxy : 0) + a0 + nx * a1;
                    else if (s1) f = fy + (hi1 ? nx : 0) + a0 + nx * nby * a2;
                    else f = fx + (hi0 ? 1 : 0) + nbx * (a1 + ny_free * a2);
                    const int rank = (lo0 ? 1 : 0) + (s0 ? 2 : 1) * ((lo1 ? 1 : 0) + (s1 ? 2 : 1) * (lo2 ? 1 : 0));
                    VPP_ST(&part[(unsigned)rank * nsh + (unsigned)f], BC_PART, v);
                } else {
                    VPP_ST(at_byte(yt + row, lane_b), BC_Y, v);
                }
                if (dot) dsum += (double)VPP_LD(at_byte(xt + row, lane_b), BC_X) * (double)v;
            }
        }
    }
    return dsum;
}

// flush_owned_get reading the accumulated tile block yb.
template <int K, typename T, int TX, int TY, int TZ>
__device__ __forceinline__ double flush_owned(const MeshArgs& m, const TileCoord& tc, const T* yb, int lx, int ly,
                                              int lz, int cx, int cy, int cz, int a0_only,
                                              const T* __restrict__ x, T* __restrict__ y, T* __restrict__ part,
                                              int64_t nshared, bool dot)
{
    constexpr int BX = K * TX + 1, BY = K * TY + 1;
    const int lbase = K * lx + BX * (K * ly + BY * K * lz);
    auto get = [&](int a0, int a1, int a2, const bool*) { return VPP_LD(&yb[lbase + a0 + BX * (a1 + BY * a2)], BC_SLOT); };
    return flush_owned_get<K, T, TX, TY, TZ>(m, tc, get, lx, ly, lz, cx, cy, cz, a0_only, x, y, part, nshared, dot);
}

template <int K, typename T>
__device__ __forceinline__ void scatter_cell_lds(T* yb, int BX, int BY, int lx, int ly, int lz,
                                                 const T (&u)[(K + 1) * (K + 1) * (K + 1)])
{
    constexpr int N = K + 1;
#pragma unroll
    for (int a2 = 0; a2 < N; ++a2)
#pragma unroll
        for (int a1 = 0; a1 < N; ++a1)
#pragma unroll
            for (int a0 = 0; a0 < N; ++a0)
            {
                T* const cell_node = &yb[(K * lx + a0) + BX * ((K * ly + a1) + BY * (K * lz + a2))];
                if (VPP_OK(cell_node, BC_SLOT)) atomicAdd(cell_node, u[a0 + N * (a1 + N * a2)]);
            }
}

// ---------------------------------------------------------------------------
// Variant 0: one cell per thread, operands gathered straight from global memory,
// one tile per workgroup.

template <int K, typename T, int TX, int TY, int TZ, int HV, bool DOT>
__global__ void __launch_bounds__(TX * TY * TZ) apply_cell_kernel(ApplyArgs<T> a)
{
    constexpr int N = K + 1, N3 = N * N * N, NT = TX * TY * TZ;
    constexpr int BX = K * TX + 1, BY = K * TY + 1, BZ = K * TZ + 1;
    __shared__ T yb[BX * BY * BZ];
    VPP_BC_BEGIN(a.x, a.y, a.phi, a.part, a.dot_part, yb, (int64_t)a.m.nn[0] * a.m.nn[1] * a.m.nn[2],
                 8 * a.nshared, (int64_t)gridDim.x, BX * BY * BZ);
    if (a.done && *a.done) return;
    const MeshArgs& m = a.m;
    const int tile = xcd_tile(blockIdx.x, gridDim.x);
    const TileCoord tc = tile_coord<K, TX, TY, TZ>(m, tile);
    for (int i = threadIdx.x; i < BX * BY * BZ; i += NT) yb[i] = T(0);
    __syncthreads();
    const int lx = threadIdx.x % TX, ly = (threadIdx.x / TX) % TY, lz = threadIdx.x / (TX * TY);
    const int cx = tc.t[0] * TX + lx, cy = tc.t[1] * TY + ly, cz = tc.t[2] * TZ + lz;
    if (cx < m.nc[0] && cy < m.nc[1] && cz < m.nc[2]) {
        T cw[N3], u[N3];
        cell_coefficient<K, HV>(m, a.phi, cx, cy, cz, cw);
        gather_cell<K>(m, a.x, cx, cy, cz, cell_dirichlet_faces(m, cx, cy, cz), u);
        cell_operator<K>(m, cw, u);
        scatter_cell_lds<K>(yb, BX, BY, lx, ly, lz, u);
    }
    __syncthreads();
    double d = 0.0;
    if (cx < m.nc[0] && cy < m.nc[1] && cz < m.nc[2])
        d = flush_owned<K, T, TX, TY, TZ>(m, tc, yb, lx, ly, lz, cx, cy, cz, -1, a.x, a.y, a.part, a.nshared,
                                          DOT);
    if constexpr (DOT) {
        const double s = block_sum<NT>(d);
        if (threadIdx.x == 0) VPP_ST(&a.dot_part[blockIdx.x], BC_DOT, s);
    }
}

// ---------------------------------------------------------------------------
// Write-out of a one-cell-per-thread tile from the slot array in two passes
// with little divergence:
//   pass 1: every cell writes the K^3 nodes with local index a_d < K (its own
//           result from registers plus the slots of the cells below it in the
//           tile) - the same straight-line code for every lane;
//   pass 2: the nodes of the tile block's three upper faces (local index K of
//           the last cells), walked node by node by all threads, whose
//           contributions all lie in slots.
// Each node goes to y (node of this tile only), to the partial array (node on
// a plane shared with a neighbouring tile: part[rank * nshared + f], see
// shared_nodes.h), or is an identity row y = x (Dirichlet node; every tile
// holding it writes the same value).  Only the positions with some a_d = K need
// to be in the slot array.  Returns this thread's share of x . (A x); identity
// rows count once, from the lowest tile holding them.
template <int K>
__device__ __forceinline__ constexpr bool owned_pos(int a0, int a1, int a2)
{
    return a0 < K && a1 < K && a2 < K;
}

// Where the write-out finds a cell's local result (a0, a1, a2) in LDS.  col()
// is the handle of cell c of the tile, zero() that of a column of zeros, which
// stands in for a neighbour cell below the tile.
template <int N, typename T, int NC>
struct ColSlots {   // slot q of cell c at q * (NC + 1) + c
    const T* s;
    __device__ __forceinline__ int col(int c) const { return c; }
    __device__ __forceinline__ int zero() const { return NC; }
    __device__ __forceinline__ T get(int a0, int a1, int a2, int h) const
    {
        return VPP_LD(&s[(a0 + N * (a1 + N * a2)) * (NC + 1) + h], BC_SLOT);
    }
};

// Per-tile data of the upper-face write-out.
template <typename T, typename S>
struct FaceCtx {
    const MeshArgs& m;
    const TileCoord& tc;
    const S& slot;
    const T* __restrict__ xt;
    T* __restrict__ yt;
    T* __restrict__ part;
    unsigned nsh;
    int nx, nxy, nbx, nby, nbz, nyf;
};

// The (cell, local index) pairs of the tile touching block coordinate c along
// one direction: on the face (c == E) only the last cell with index K; else
// cell c / K with index c % K, plus cell c / K - 1 with index K when c is a
// multiple of K above 0 (otherwise the second cell is -1: no contribution).
template <int K>
__device__ __forceinline__ void contributors(int c, bool face, int ncell, int stride, int& cell0, int& q0,
                                             int& cell1, int& q1)
{
    if (face) {
        cell0 = (ncell - 1) * stride;
        q0 = K;
        cell1 = -1;
        q1 = 0;
        return;
    }
    const int q = c / K, r = c - q * K;
    cell0 = q * stride;
    q0 = r;
    cell1 = (r == 0 && q > 0) ? (q - 1) * stride : -1;
    q1 = K;
}

// Writes the nodes of the tile block's upper face normal to direction FACE
// (the two other coordinates strictly below their upper faces for the faces
// written later, so every node is written once: z face first, then y, then x),
// for a tile cut by the mesh's upper boundary (runtime extents); complete
// tiles use upper_face_full.
template <int K, typename T, int TX, int TY, int TZ, int FACE, int NTH, typename S>
__device__ __forceinline__ double upper_face(const FaceCtx<T, S>& f, bool dot)
{
    const int E0 = f.tc.ext[0] - 1;
    const int E1 = f.tc.ext[1] - 1;
    const int E2 = f.tc.ext[2] - 1;
    // extents of the two free coordinates (a, b) of this face
    const int na = FACE == 0 ? E1 + 1 : E0;
    const int nb = FACE == 2 ? E1 : E2 + 1;
    const int count = na * nb;
    const int nc0 = E0 / K, nc1 = E1 / K, nc2 = E2 / K;
    const int t0 = f.tc.t[0], t1 = f.tc.t[1], t2 = f.tc.t[2];
    double dsum = 0.0;
    // the node's x (identity rows copy it, x . Ax needs it) for every
    // iteration of this thread, loaded before the first one; a ragged tile has
    // at most the iterations of a complete one
    constexpr int CMAX = (FACE == 0 ? K * TY + 1 : K * TX) * (FACE == 2 ? K * TY : K * TZ + 1);
    constexpr int MAXIT = (CMAX + NTH - 1) / NTH;
    T xe[MAXIT];
#pragma unroll
    for (int it = 0; it < MAXIT; ++it) {
        const int n = threadIdx.x + it * NTH;
        if (n >= count) break;
        const int ib = n / na, ia = n - ib * na;
        const int c0 = FACE == 0 ? E0 : ia, c1 = FACE == 0 ? ia : (FACE == 1 ? E1 : ib), c2 = FACE == 2 ? E2 : ib;
        xe[it] = VPP_LD(&f.xt[(unsigned)(c0 + f.nx * c1 + f.nxy * c2)], BC_X);
    }
#pragma unroll
    for (int it = 0; it < MAXIT; ++it) {
        const int n = threadIdx.x + it * NTH;
        if (n >= count) break;
        const int ib = n / na, ia = n - ib * na;
        const int c0 = FACE == 0 ? E0 : ia;
        const int c1 = FACE == 0 ? ia : (FACE == 1 ? E1 : ib);
        const int c2 = FACE == 2 ? E2 : ib;
        int x0, p0, x1, p1, y0, r0, y1, r1, z0, s0, z1, s1;
        contributors<K>(c0, FACE == 0, nc0, 1, x0, p0, x1, p1);
        contributors<K>(c1, FACE == 1 || (FACE == 0 && c1 == E1), nc1, TX, y0, r0, y1, r1);
        contributors<K>(c2, FACE == 2 || (FACE != 2 && c2 == E2), nc2, TX * TY, z0, s0, z1, s1);
        auto rd = [&](int cx_, int qx, int cy_, int qy, int cz_, int qz) -> T {
            const bool ok = cx_ >= 0 && cy_ >= 0 && cz_ >= 0;
            return f.slot.get(qx, qy, qz, ok ? f.slot.col(cx_ + cy_ + cz_) : f.slot.zero());
        };
        T v = rd(x0, p0, y0, r0, z0, s0);
        v += rd(x1, p1, y0, r0, z0, s0);
        v += rd(x0, p0, y1, r1, z0, s0);
        v += rd(x1, p1, y1, r1, z0, s0);
        v += rd(x0, p0, y0, r0, z1, s1);
        v += rd(x1, p1, y0, r0, z1, s1);
        v += rd(x0, p0, y1, r1, z1, s1);
        v += rd(x1, p1, y1, r1, z1, s1);
        const int gi = f.tc.n0[0] + c0, gj = f.tc.n0[1] + c1, gl = f.tc.n0[2] + c2;
        const unsigned off = (unsigned)(c0 + f.nx * c1 + f.nxy * c2);
        const bool lo0 = c0 == 0 && t0 > 0, lo1 = c1 == 0 && t1 > 0, lo2 = c2 == 0 && t2 > 0;
        const bool hi0 = c0 == E0 && t0 < f.nbx, hi1 = c1 == E1 && t1 < f.nby, hi2 = c2 == E2 && t2 < f.nbz;
        if (is_dirichlet(f.m, gi, gj, gl)) {
            const T xv = xe[it];
            VPP_ST(&f.yt[off], BC_Y, xv);
            if (dot && !(lo0 || lo1 || lo2)) dsum += (double)xv * (double)xv;
            continue;
        }
        if (lo0 || lo1 || lo2 || hi0 || hi1 || hi2) {
            int64_t fi;
            int rank;
            shared_from_tile(f.m, f.tc.t, lo0, lo1, lo2, hi0, hi1, hi2, gi, gj, gl, fi, rank);
            VPP_ST(&f.part[(unsigned)rank * f.nsh + (unsigned)fi], BC_PART, v);
        } else {
            VPP_ST(&f.yt[off], BC_Y, v);
        }
        if (dot) dsum += (double)xe[it] * (double)v;
    }
    return dsum;
}

// upper_face for a complete tile (compile-time extents), with 32-bit index
// arithmetic and per-tile uniform bases.  Along a direction that is not FACE,
// block coordinate c < E has the pairs (c / K, c % K) when c / K is a cell of
// the tile and (c / K - 1, K) when c % K == 0 and c > 0; on the face (c == E)
// only the second exists.  Along FACE only the last cell with index K holds the
// node, so every node sums at most four slots.
template <int K, typename T, int TX, int TY, int TZ, int FACE, int NTH, typename S>
__device__ __forceinline__ double upper_face_full(const FaceCtx<T, S>& f, const int (&fb)[3], const bool (&dlo)[3],
                                                  const bool (&dhi)[3], bool dot)
{
    constexpr int E0 = K * TX, E1 = K * TY, E2 = K * TZ;
    constexpr int NA = FACE == 0 ? E1 + 1 : E0;
    constexpr int NB = FACE == 2 ? E1 : E2 + 1;
    constexpr int T3[3] = {TX, TY, TZ};
    constexpr int CST[3] = {1, TX, TX * TY};
    const int t0 = f.tc.t[0], t1 = f.tc.t[1], t2 = f.tc.t[2];
    const bool anyd = dlo[0] || dlo[1] || dlo[2] || dhi[0] || dhi[1] || dhi[2];
    const bool hn[3] = {t0 < f.nbx, t1 < f.nby, t2 < f.nbz};   // a tile above along d
    double dsum = 0.0;
    for (int n = threadIdx.x; n < NA * NB; n += NTH) {
        const int ib = n / NA, ia = n - ib * NA;
        const int c[3] = {FACE == 0 ? E0 : ia, FACE == 0 ? ia : (FACE == 1 ? E1 : ib), FACE == 2 ? E2 : ib};
        // slot column and local index of the (up to) two cells along each direction
        int ca[3], cb[3], qa[3];
#pragma unroll
        for (int d = 0; d < 3; ++d) {
            if (d == FACE) {
                ca[d] = -1;
                qa[d] = 0;
                cb[d] = T3[d] - 1;
                continue;
            }
            const int q = c[d] / K, r = c[d] - q * K;
            ca[d] = q < T3[d] ? q : -1;
            qa[d] = r;
            cb[d] = (r == 0 && q > 0) ? q - 1 : -1;
        }
        const unsigned off = (unsigned)(c[0] + f.nx * c[1] + f.nxy * c[2]);
        // on a tile with a Dirichlet face (an identity row copies it) or for
        // x . Ax the node's x is loaded before the slot reads, so its latency
        // overlaps them
        const T xe = (anyd || dot) ? VPP_LD(&f.xt[off], BC_X) : T(0);
        T v = T(0);
#pragma unroll
        for (int s = 0; s < 8; ++s) {
            const bool b0 = s & 1, b1 = (s >> 1) & 1, b2 = (s >> 2) & 1;
            if ((FACE == 0 && !b0) || (FACE == 1 && !b1) || (FACE == 2 && !b2)) continue;
            const int x0 = b0 ? cb[0] : ca[0], x1 = b1 ? cb[1] : ca[1], x2 = b2 ? cb[2] : ca[2];
            const bool ok = x0 >= 0 && x1 >= 0 && x2 >= 0;
            v += f.slot.get(b0 ? K : qa[0], b1 ? K : qa[1], b2 ? K : qa[2],
                            ok ? f.slot.col(x0 * CST[0] + x1 * CST[1] + x2 * CST[2]) : f.slot.zero());
        }
        const bool lo0 = FACE != 0 && c[0] == 0 && t0 > 0;
        const bool lo1 = FACE != 1 && c[1] == 0 && t1 > 0;
        const bool lo2 = FACE != 2 && c[2] == 0 && t2 > 0;
        const bool hi0 = c[0] == E0 && hn[0], hi1 = c[1] == E1 && hn[1], hi2 = c[2] == E2 && hn[2];
        if (anyd && ((dlo[0] && c[0] == 0) || (dhi[0] && c[0] == E0) || (dlo[1] && c[1] == 0) ||
                     (dhi[1] && c[1] == E1) || (dlo[2] && c[2] == 0) || (dhi[2] && c[2] == E2))) {
            const T xv = xe;
            VPP_ST(&f.yt[off], BC_Y, xv);
            if (dot && !(lo0 || lo1 || lo2)) dsum += (double)xv * (double)xv;
            continue;
        }
        const bool s0 = lo0 || hi0, s1 = lo1 || hi1, s2 = lo2 || hi2;
        if (s0 || s1 || s2) {
            int fi;
            if (s2) fi = fb[2] + c[0] + f.nx * c[1] + (hi2 ? f.nxy : 0);
            else if (s1) fi = fb[1] + c[0] + f.nx * ((hi1 ? 1 : 0) + f.nby * c[2]);
            else fi = fb[0] + (hi0 ? 1 : 0) + f.nbx * (c[1] + f.nyf * c[2]);
            const int rank = (lo0 ? 1 : 0) + (s0 ? 2 : 1) * ((lo1 ? 1 : 0) + (s1 ? 2 : 1) * (lo2 ? 1 : 0));
            VPP_ST(&f.part[(unsigned)rank * f.nsh + (unsigned)fi], BC_PART, v);
        } else {
            VPP_ST(&f.yt[off], BC_Y, v);
        }
        if (dot) dsum += (double)xe * (double)v;
    }
    return dsum;
}

// Pass 2 of the write-out: the nodes of the tile block's three upper faces,
// whose contributions all lie in the slot array, walked by NTH threads.
template <int K, typename T, int TX, int TY, int TZ, int NTH, typename S>
__device__ __forceinline__ double upper_faces(const MeshArgs& m, const TileCoord& tc, const S& slot,
                                              const T* __restrict__ x, T* __restrict__ y, T* __restrict__ part,
                                              int64_t nshared, bool dot)
{
    const int nx = m.nn[0], nxy = m.nn[0] * m.nn[1];
    const int64_t tile0 = uniform_i64(node_index(m, tc.n0[0], tc.n0[1], tc.n0[2]));
    const int t0 = tc.t[0], t1 = tc.t[1], t2 = tc.t[2];
    const int nbx = m.ntile[0] - 1, nby = m.ntile[1] - 1, nbz = m.ntile[2] - 1;
    const int cz_n = nbz * nxy;
    const int cy_n = nby * (m.nn[2] - nbz) * nx;
    const int ny_free = m.nn[1] - nby;
    FaceCtx<T, S> fc{m, tc, slot, x + tile0, y + tile0, part, (unsigned)nshared, nx, nxy, nbx, nby, nbz, ny_free};
    double dsum = 0.0;
    const bool full = tc.ext[0] == K * TX + 1 && tc.ext[1] == K * TY + 1 && tc.ext[2] == K * TZ + 1;
    if (full) {
        // shared-node enumeration bases of the tile's planes (lower plane of
        // each family; the upper plane adds nxy, nx or 1)
        const int n0x = tc.n0[0], n0y = tc.n0[1], n0z = tc.n0[2];
        const int fb[3] = {cz_n + cy_n + (t0 - 1) + nbx * ((n0y - t1) + ny_free * (n0z - t2)),
                           cz_n + n0x + nx * ((t1 - 1) + nby * (n0z - t2)), n0x + nx * n0y + nxy * (t2 - 1)};
        const bool dlo[3] = {(m.bcmask & 1) && t0 == 0, (m.bcmask & 4) && t1 == 0, (m.bcmask & 16) && t2 == 0};
        const bool dhi[3] = {(m.bcmask & 2) && t0 == nbx, (m.bcmask & 8) && t1 == nby, (m.bcmask & 32) && t2 == nbz};
        dsum += upper_face_full<K, T, TX, TY, TZ, 2, NTH>(fc, fb, dlo, dhi, dot);
        dsum += upper_face_full<K, T, TX, TY, TZ, 1, NTH>(fc, fb, dlo, dhi, dot);
        dsum += upper_face_full<K, T, TX, TY, TZ, 0, NTH>(fc, fb, dlo, dhi, dot);
    } else {
        dsum += upper_face<K, T, TX, TY, TZ, 2, NTH>(fc, dot);
        dsum += upper_face<K, T, TX, TY, TZ, 1, NTH>(fc, dot);
        dsum += upper_face<K, T, TX, TY, TZ, 0, NTH>(fc, dot);
    }
    return dsum;
}

template <int K, typename T, int TX, int TY, int TZ>
__device__ __forceinline__ double flush_two_pass(const MeshArgs& m, const TileCoord& tc, const T* slot, int cs,
                                                 const T (&u)[(K + 1) * (K + 1) * (K + 1)], bool active, int lx,
                                                 int ly, int lz, int cx, int cy, int cz, const T* __restrict__ x,
                                                 T* __restrict__ y, T* __restrict__ part, int64_t nshared, bool dot)
{
    constexpr int N = K + 1, NT = TX * TY * TZ;
    const int tid = threadIdx.x;
    const int nx = m.nn[0], nxy = m.nn[0] * m.nn[1];
    const int64_t tile0 = uniform_i64(node_index(m, tc.n0[0], tc.n0[1], tc.n0[2]));
    const T* __restrict__ xt = x + tile0;
    T* __restrict__ yt = y + tile0;
    const int t0 = tc.t[0], t1 = tc.t[1], t2 = tc.t[2];
    const int nbx = m.ntile[0] - 1, nby = m.ntile[1] - 1, nbz = m.ntile[2] - 1;
    const int cz_n = nbz * nxy;
    const int cy_n = nby * (m.nn[2] - nbz) * nx;
    const int ny_free = m.nn[1] - nby;
    const unsigned nsh = (unsigned)nshared;
    double dsum = 0.0;

    // ---- pass 1: owned positions of every cell
    if (active) {
        const int zero = NT;
        const int nb0 = lx > 0 ? tid - 1 : zero, nb1 = ly > 0 ? tid - TX : zero, nb2 = lz > 0 ? tid - TX * TY : zero;
        const int nb01 = lx > 0 && ly > 0 ? tid - 1 - TX : zero;
        const int nb02 = lx > 0 && lz > 0 ? tid - 1 - TX * TY : zero;
        const int nb12 = ly > 0 && lz > 0 ? tid - TX - TX * TY : zero;
        const int nb012 = lx > 0 && ly > 0 && lz > 0 ? tid - 1 - TX - TX * TY : zero;
        const bool hl0 = lx == 0 && t0 > 0, hl1 = ly == 0 && t1 > 0, hl2 = lz == 0 && t2 > 0;
        const int faces = cell_dirichlet_faces(m, cx, cy, cz);
        const bool dl0 = faces & 1, dl1 = faces & 4, dl2 = faces & 16;
        const int i0 = K * cx, j0 = K * cy, l0 = K * cz;
        const unsigned lane_b = (unsigned)(K * lx + nx * K * ly + nxy * K * lz) * (unsigned)sizeof(T);
        const int fz = i0 + nx * j0 + nxy * (t2 - 1);
        const int fy = cz_n + i0 + nx * ((t1 - 1) + nby * (l0 - t2));
        const int fx = cz_n + cy_n + (t0 - 1) + nbx * ((j0 - t1) + ny_free * (l0 - t2));
        // x at the owned positions (identity rows on a Dirichlet face copy it,
        // x . Ax needs it), all loads issued together rather than one round
        // trip per row
        T xd[K * K * K];
        if (dot || dl0 || dl1 || dl2) {
#pragma unroll
            for (int a2 = 0; a2 < K; ++a2)
#pragma unroll
                for (int a1 = 0; a1 < K; ++a1) {
                    const T* row = at_byte(xt + (nx * a1 + nxy * a2), lane_b);
#pragma unroll
                    for (int a0 = 0; a0 < K; ++a0) xd[a0 + K * (a1 + K * a2)] = VPP_LD(&row[a0], BC_X);
                }
        }
#pragma unroll
        for (int a2 = 0; a2 < K; ++a2)
#pragma unroll
            for (int a1 = 0; a1 < K; ++a1)
#pragma unroll
                for (int a0 = 0; a0 < K; ++a0) {
                    const bool z0 = a0 == 0, z1 = a1 == 0, z2 = a2 == 0;
                    T v = u[a0 + N * (a1 + N * a2)];
                    if (z0) v += VPP_LD(&slot[(K + N * (a1 + N * a2)) * cs + nb0], BC_SLOT);
                    if (z1) v += VPP_LD(&slot[(a0 + N * (K + N * a2)) * cs + nb1], BC_SLOT);
                    if (z2) v += VPP_LD(&slot[(a0 + N * (a1 + N * K)) * cs + nb2], BC_SLOT);
                    if (z0 && z1) v += VPP_LD(&slot[(K + N * (K + N * a2)) * cs + nb01], BC_SLOT);
                    if (z0 && z2) v += VPP_LD(&slot[(K + N * (a1 + N * K)) * cs + nb02], BC_SLOT);
                    if (z1 && z2) v += VPP_LD(&slot[(a0 + N * (K + N * K)) * cs + nb12], BC_SLOT);
                    if (z0 && z1 && z2) v += VPP_LD(&slot[(K + N * (K + N * K)) * cs + nb012], BC_SLOT);
                    const int row = a0 + nx * a1 + nxy * a2;   // uniform
                    const bool lo0 = z0 && hl0, lo1 = z1 && hl1, lo2 = z2 && hl2;
                    const bool dir = (z0 && dl0) || (z1 && dl1) || (z2 && dl2);
                    if (dir) {
                        const T xv = xd[a0 + K * (a1 + K * a2)];
                        VPP_ST(at_byte(yt + row, lane_b), BC_Y, xv);
                        if (dot && !(lo0 || lo1 || lo2)) dsum += (double)xv * (double)xv;
                        continue;
                    }
                    T* dst = at_byte(yt + row, lane_b);
                    if (lo0 || lo1 || lo2) {
                        const int f = lo2 ? fz + a0 + nx * a1 : (lo1 ? fy + a0 + nx * nby * a2 : fx + nbx * (a1 + ny_free * a2));
                        const int rank = (lo0 ? 1 : 0) + (lo0 ? 2 : 1) * ((lo1 ? 1 : 0) + (lo1 ? 2 : 1) * (lo2 ? 1 : 0));
                        dst = part + ((unsigned)rank * nsh + (unsigned)f);
                    }
                    VPP_ST(dst, BC_OUT, v);
                    if (dot) dsum += (double)xd[a0 + K * (a1 + K * a2)] * (double)v;
                }
    }

    const ColSlots<N, T, NT> slots{slot};
    return dsum + upper_faces<K, T, TX, TY, TZ, NT>(m, tc, slots, x, y, part, nshared, dot);
}

// ---------------------------------------------------------------------------
// Variant 4: one cell per thread, operands gathered straight from global
// memory, and the cell results exchanged through LDS without atomics: every
// cell stores its (k+1)^3 local results in its own column of a slot array
// (slot q of cell c at q * (NT + 1) + c, so a wave's stores and loads hit
// consecutive words), then sums, for each node it owns, the slots of the up to
// eight cells of the tile that touch the node.  Column NT stays zero and stands
// in for a neighbour cell below the tile.


// Body of a workgroup on one tile; dot_out: its partial of x . (A x).
template <int K, typename T, int TX, int TY, int TZ, int HV, bool DOT, bool MASS>
__device__ __forceinline__ void slot_tile(const ApplyArgs<T>& a, int tile, T* slot, double* dot_out)
{
    constexpr int N = K + 1, N3 = N * N * N, NT = TX * TY * TZ, CS = NT + 1;
    const MeshArgs& m = a.m;
    const TileCoord tc = tile_coord<K, TX, TY, TZ>(m, tile);
    const int tid = threadIdx.x;
    const int lx = tid % TX, ly = (tid / TX) % TY, lz = tid / (TX * TY);
    const int cx = tc.t[0] * TX + lx, cy = tc.t[1] * TY + ly, cz = tc.t[2] * TZ + lz;
    const bool active = cx < m.nc[0] && cy < m.nc[1] && cz < m.nc[2];
    for (int q = tid; q < N3; q += NT) VPP_ST(&slot[q * CS + NT], BC_SLOT, T(0));
    T u[N3];
    if (active) {
        const int nx = m.nn[0], nxy = m.nn[0] * m.nn[1];
        const int64_t tile0 = uniform_i64(node_index(m, tc.n0[0], tc.n0[1], tc.n0[2]));
        const unsigned lane_b = (unsigned)(K * lx + nx * K * ly + nxy * K * lz) * (unsigned)sizeof(T);
        T cw[N3];
        gather_cell_t<K>(a.phi + tile0, lane_b, nx, nxy, 0, cw);
        sweep3<K, MS, false, 0>(cw);
        sweep3<K, MS, false, 1>(cw);
        sweep3<K, MS, false, 2>(cw);
        coef_weights3<K, HV>(m, cw);
        gather_cell_t<K>(a.x + tile0, lane_b, nx, nxy, cell_dirichlet_faces(m, cx, cy, cz), u);
        cell_operator<K, T, MASS>(m, cw, u);
#pragma unroll
        for (int q = 0; q < N3; ++q)
            if (!owned_pos<K>(q % N, (q / N) % N, q / (N * N))) VPP_ST(&slot[q * CS + tid], BC_SLOT, u[q]);
    }
    __syncthreads();
    const double d = flush_two_pass<K, T, TX, TY, TZ>(m, tc, slot, CS, u, active, lx, ly, lz, cx, cy, cz, a.x, a.y,
                                                      a.part, a.nshared, DOT);
    if constexpr (DOT) {
        const double s = block_sum<NT>(d);
        if (threadIdx.x == 0) VPP_ST(dot_out, BC_DOT, s);
    }
}

template <int K, typename T, int TX, int TY, int TZ, int HV, bool DOT, bool MASS = false>
__global__ void __launch_bounds__(TX * TY * TZ) apply_slot_kernel(ApplyArgs<T> a)
{
    constexpr int N3 = (K + 1) * (K + 1) * (K + 1), CS = TX * TY * TZ + 1;
    __shared__ T slot[N3 * CS];
    VPP_BC_BEGIN(a.x, a.y, a.phi, a.part, a.dot_part, slot, (int64_t)a.m.nn[0] * a.m.nn[1] * a.m.nn[2],
                 8 * a.nshared, (int64_t)gridDim.x, N3 * CS);
    if (a.done && *a.done) return;
    slot_tile<K, T, TX, TY, TZ, HV, DOT, MASS>(a, xcd_tile(blockIdx.x, gridDim.x), slot, a.dot_part + blockIdx.x);
}

// ---------------------------------------------------------------------------
// Variant 2 (k = 3): half a cell per thread.  The two threads of a cell (an
// even/odd lane pair) hold two z-planes each of the cell's (k+1)^3 values, so a
// thread carries half the register state of the cell-per-thread kernel and
// twice as many waves cover the mesh.  x and y sweeps stay in registers; z
// sweeps combine the pair's planes by DPP lane swaps.  The odd thread stores
// its planes mirrored in z (its local plane j is the cell's plane k - j), which
// makes every z sweep the same compile-time code on both threads: the value
// matrix and the Gauss weights are symmetric under z -> 1 - z, and the
// collocation derivative changes sign, which cancels between the forward and
// the transposed derivative (derivative values exchanged between the two
// threads are negated, since each holds them in its own frame).

template <int K>
constexpr bool z_reflection_ok()
{
    constexpr int N = K + 1;
    for (int q = 0; q < N; ++q) {
        if (Tab<K>::t.w[N - 1 - q] - Tab<K>::t.w[q] > 1e-15 || Tab<K>::t.w[q] - Tab<K>::t.w[N - 1 - q] > 1e-15)
            return false;
        for (int a = 0; a < N; ++a) {
            const double ds = Tab<K>::t.S[N - 1 - q][N - 1 - a] - Tab<K>::t.S[q][a];
            const double dd = Tab<K>::t.Dc[N - 1 - q][N - 1 - a] + Tab<K>::t.Dc[q][a];
            if (ds > 1e-14 || -ds > 1e-14 || dd > 1e-12 || -dd > 1e-12) return false;
        }
    }
    return true;
}
static_assert(z_reflection_ok<3>(), "S even and Dc odd under reflection");

// The partner lane's value (lanes 2i and 2i+1 swapped).
__device__ __forceinline__ double pair_swap(double v)
{
    constexpr int ctrl = 0xB1;   // quad_perm(1, 0, 3, 2)
    const int lo = __builtin_amdgcn_mov_dpp(__double2loint(v), ctrl, 0xF, 0xF, true);
    const int hi = __builtin_amdgcn_mov_dpp(__double2hiint(v), ctrl, 0xF, 0xF, true);
    return __hiloint2double(hi, lo);
}
__device__ __forceinline__ float pair_swap(float v)
{
    return __int_as_float(__builtin_amdgcn_mov_dpp(__float_as_int(v), 0xB1, 0xF, 0xF, true));
}

// z sweep of a 4 x 4 matrix over the pair's planes, in this thread's frame
// (frame planes 0, 1 local; 2, 3 the partner's planes 1, 0).
template <int K, Mat M, bool TR, typename T>
__device__ __forceinline__ void zsweep_pair(T (&v)[2][(K + 1) * (K + 1)])
{
    constexpr int N = K + 1, N2 = N * N;
    static_assert(N == 4, "two planes per thread");
#pragma unroll
    for (int q = 0; q < N2; ++q) {
        const T f[4] = {v[0][q], v[1][q], pair_swap(v[1][q]), pair_swap(v[0][q])};
#pragma unroll
        for (int j = 0; j < 2; ++j) {
            Acc<T> acc;
#pragma unroll
            for (int a = 0; a < 4; ++a) acc.add(TR ? mat<K, M>(a, j) : mat<K, M>(j, a), f[a]);
            v[j][q] = acc.get();
        }
        __builtin_amdgcn_sched_barrier(0);   // one column at a time (register pressure)
    }
}

// Pass 1 of the write-out for a half cell: the owned positions (every index
// below K) of this thread's two planes pl[0], pl[1] (a runtime plane index
// per thread), from its registers plus the slots of the cells below it in the
// tile, as flush_two_pass does for a whole cell.
template <int K, typename T, int TX, int TY, int TZ>
__device__ __forceinline__ double flush_half_owned(const MeshArgs& m, const TileCoord& tc, const T* slot, int cs,
                                                   const T (&v)[2][(K + 1) * (K + 1)], const int (&pl)[2], int lx,
                                                   int ly, int lz, int cx, int cy, int cz, const T* __restrict__ x,
                                                   T* __restrict__ y, T* __restrict__ part, int64_t nshared, bool dot)
{
    constexpr int N = K + 1, NC = TX * TY * TZ;
    const int c = lx + TX * (ly + TY * lz), zero = NC;
    const int nx = m.nn[0], nxy = m.nn[0] * m.nn[1];
    const int64_t tile0 = uniform_i64(node_index(m, tc.n0[0], tc.n0[1], tc.n0[2]));
    const T* __restrict__ xt = x + tile0;
    T* __restrict__ yt = y + tile0;
    const int t0 = tc.t[0], t1 = tc.t[1], t2 = tc.t[2];
    const int nbx = m.ntile[0] - 1, nby = m.ntile[1] - 1, nbz = m.ntile[2] - 1;
    const int cz_n = nbz * nxy;
    const int cy_n = nby * (m.nn[2] - nbz) * nx;
    const int ny_free = m.nn[1] - nby;
    const unsigned nsh = (unsigned)nshared;
    const int nb0 = lx > 0 ? c - 1 : zero, nb1 = ly > 0 ? c - TX : zero, nb2 = lz > 0 ? c - TX * TY : zero;
    const int nb01 = lx > 0 && ly > 0 ? c - 1 - TX : zero;
    const int nb02 = lx > 0 && lz > 0 ? c - 1 - TX * TY : zero;
    const int nb12 = ly > 0 && lz > 0 ? c - TX - TX * TY : zero;
    const int nb012 = lx > 0 && ly > 0 && lz > 0 ? c - 1 - TX - TX * TY : zero;
    const bool hl0 = lx == 0 && t0 > 0, hl1 = ly == 0 && t1 > 0, hl2 = lz == 0 && t2 > 0;
    const int faces = cell_dirichlet_faces(m, cx, cy, cz);
    const bool dl0 = faces & 1, dl1 = faces & 4, dl2 = faces & 16;
    const int i0 = K * cx, j0 = K * cy, l0 = K * cz;
    const unsigned lane_b = (unsigned)(K * lx + nx * K * ly + nxy * K * lz) * (unsigned)sizeof(T);
    const int fz = i0 + nx * j0 + nxy * (t2 - 1);
    const int fy = cz_n + i0 + nx * ((t1 - 1) + nby * (l0 - t2));
    const int fx = cz_n + cy_n + (t0 - 1) + nbx * ((j0 - t1) + ny_free * (l0 - t2));
    auto pos = [](int b0, int b1, int b2) { return b0 + N * (b1 + N * b2); };
    double dsum = 0.0;
    // x at the owned positions (identity rows copy it, x . Ax needs it), all
    // loads issued together rather than one round trip per row
    T xd[2][K * K];
    if (dot || dl0 || dl1 || dl2) {
#pragma unroll
        for (int j = 0; j < 2; ++j) {
            if (pl[j] >= K) continue;
#pragma unroll
            for (int a1 = 0; a1 < K; ++a1) {
                const T* row = at_byte(xt + (nx * a1 + nxy * pl[j]), lane_b);
#pragma unroll
                for (int a0 = 0; a0 < K; ++a0) xd[j][a0 + K * a1] = VPP_LD(&row[a0], BC_X);
            }
        }
    }
#pragma unroll
    for (int j = 0; j < 2; ++j) {
        const int a2 = pl[j];
        if (a2 >= K) continue;
        const bool z2 = a2 == 0;
#pragma unroll
        for (int a1 = 0; a1 < K; ++a1)
#pragma unroll
            for (int a0 = 0; a0 < K; ++a0) {
                const bool z0 = a0 == 0, z1 = a1 == 0;
                T val = v[j][a0 + N * a1];
                if (z0) val += VPP_LD(&slot[pos(K, a1, a2) * cs + nb0], BC_SLOT);
                if (z1) val += VPP_LD(&slot[pos(a0, K, a2) * cs + nb1], BC_SLOT);
                if (z2) val += VPP_LD(&slot[pos(a0, a1, K) * cs + nb2], BC_SLOT);
                if (z0 && z1) val += VPP_LD(&slot[pos(K, K, a2) * cs + nb01], BC_SLOT);
                if (z0 && z2) val += VPP_LD(&slot[pos(K, a1, K) * cs + nb02], BC_SLOT);
                if (z1 && z2) val += VPP_LD(&slot[pos(a0, K, K) * cs + nb12], BC_SLOT);
                if (z0 && z1 && z2) val += VPP_LD(&slot[pos(K, K, K) * cs + nb012], BC_SLOT);
                const int row = a0 + nx * a1 + nxy * a2;
                const bool lo0 = z0 && hl0, lo1 = z1 && hl1, lo2 = z2 && hl2;
                if ((z0 && dl0) || (z1 && dl1) || (z2 && dl2)) {
                    const T xv = xd[j][a0 + K * a1];
                    VPP_ST(at_byte(yt + row, lane_b), BC_Y, xv);
                    if (dot && !(lo0 || lo1 || lo2)) dsum += (double)xv * (double)xv;
                    continue;
                }
                T* dst = at_byte(yt + row, lane_b);
                if (lo0 || lo1 || lo2) {
                    const int f = lo2 ? fz + a0 + nx * a1
                                      : (lo1 ? fy + a0 + nx * nby * a2 : fx + nbx * (a1 + ny_free * a2));
                    const int rank = (lo0 ? 1 : 0) + (lo0 ? 2 : 1) * ((lo1 ? 1 : 0) + (lo1 ? 2 : 1) * (lo2 ? 1 : 0));
                    dst = part + ((unsigned)rank * nsh + (unsigned)f);
                }
                VPP_ST(dst, BC_OUT, val);
                if (dot) dsum += (double)xd[j][a0 + K * a1] * (double)val;
            }
    }
    return dsum;
}

template <int K, typename T, int TX, int TY, int TZ, int HV, bool DOT>
__global__ void __launch_bounds__(2 * TX * TY * TZ) apply_half_kernel(ApplyArgs<T> a)
{
    static_assert(K == 3, "two z-planes per thread");
    constexpr int N = K + 1, N2 = N * N, N3 = N2 * N, NC = TX * TY * TZ, NTH = 2 * NC, CS = NC + 1;
    __shared__ T slot[N3 * CS];
    VPP_BC_BEGIN(a.x, a.y, a.phi, a.part, a.dot_part, slot, (int64_t)a.m.nn[0] * a.m.nn[1] * a.m.nn[2],
                 8 * a.nshared, (int64_t)gridDim.x, N3 * CS);
    if (a.done && *a.done) return;
    const MeshArgs& m = a.m;
    const int tile = xcd_tile(blockIdx.x, gridDim.x);
    const TileCoord tc = tile_coord<K, TX, TY, TZ>(m, tile);
    const int tid = threadIdx.x, c = tid >> 1, hz = tid & 1;
    const int lx = c % TX, ly = (c / TX) % TY, lz = c / (TX * TY);
    const int cx = tc.t[0] * TX + lx, cy = tc.t[1] * TY + ly, cz = tc.t[2] * TZ + lz;
    const bool active = cx < m.nc[0] && cy < m.nc[1] && cz < m.nc[2];
    for (int q = tid; q < N3; q += NTH) VPP_ST(&slot[q * CS + NC], BC_SLOT, T(0));
    // cell plane of local plane j
    const int pl[2] = {hz ? K : 0, hz ? K - 1 : 1};
    T v[2][N2];
    if (active) {
        const int nx = m.nn[0], nxy = m.nn[0] * m.nn[1];
        const int64_t tile0 = uniform_i64(node_index(m, tc.n0[0], tc.n0[1], tc.n0[2]));
        const int faces = cell_dirichlet_faces(m, cx, cy, cz);
        T cw[2][N2], u[2][N2];
#pragma unroll
        for (int j = 0; j < 2; ++j) {
            const unsigned lane_b =
                (unsigned)(K * lx + nx * K * ly + nxy * (K * lz + pl[j])) * (unsigned)sizeof(T);
#pragma unroll
            for (int a1 = 0; a1 < N; ++a1) {
                const T* prow = at_byte(a.phi + tile0 + nx * a1, lane_b);
                const T* xrow = at_byte(a.x + tile0 + nx * a1, lane_b);
#pragma unroll
                for (int a0 = 0; a0 < N; ++a0) {
                    cw[j][a0 + N * a1] = VPP_LD(&prow[a0], BC_PHI);
                    u[j][a0 + N * a1] = VPP_LD(&xrow[a0], BC_X);
                }
            }
        }
        // Dirichlet entries zeroed after every load has been issued (zeroing
        // inside the load loop made each group of loads wait for the last)
        if (faces) {
#pragma unroll
            for (int j = 0; j < 2; ++j)
#pragma unroll
                for (int a1 = 0; a1 < N; ++a1)
#pragma unroll
                    for (int a0 = 0; a0 < N; ++a0)
                        if (local_dirichlet<K>(faces, a0, a1, pl[j])) u[j][a0 + N * a1] = T(0);
        }
        // coefficient at the Gauss points of the two planes (frame plane j is
        // Gauss plane j or k - j, with the same weight)
#pragma unroll
        for (int j = 0; j < 2; ++j) {
            sweep2<K, MS, false, 0>(cw[j]);
            sweep2<K, MS, false, 1>(cw[j]);
        }
        zsweep_pair<K, MS, false>(cw);
#pragma unroll
        for (int j = 0; j < 2; ++j)
#pragma unroll
            for (int q = 0; q < N2; ++q) cw[j][q] = coef_scaled<HV>(m, cw[j][q]) * T(wref<K>(q % N, q / N, j));
        // operand at the Gauss points
#pragma unroll
        for (int j = 0; j < 2; ++j) {
            sweep2<K, MS, false, 0>(u[j]);
            sweep2<K, MS, false, 1>(u[j]);
        }
        zsweep_pair<K, MS, false>(u);
        const T r1 = T(m.rd[1]), r2 = T(m.rd[2]);
        // x and y derivative lines within the planes
#pragma unroll
        for (int j = 0; j < 2; ++j) {
#pragma unroll
            for (int i1 = 0; i1 < N; ++i1) {
                T in[N], g[N], o[N];
#pragma unroll
                for (int b = 0; b < N; ++b) in[b] = u[j][b + N * i1];
                line<K, MDC, false>(in, g);
#pragma unroll
                for (int b = 0; b < N; ++b) g[b] *= cw[j][b + N * i1];
                line<K, MDC, true>(g, o);
#pragma unroll
                for (int b = 0; b < N; ++b) v[j][b + N * i1] = o[b];
            }
#pragma unroll
            for (int i0 = 0; i0 < N; ++i0) {
                T in[N], g[N], o[N];
#pragma unroll
                for (int b = 0; b < N; ++b) in[b] = u[j][i0 + N * b];
                line<K, MDC, false>(in, g);
#pragma unroll
                for (int b = 0; b < N; ++b) g[b] *= cw[j][i0 + N * b] * r1;
#pragma unroll
                for (int b = 0; b < N; ++b) o[b] = v[j][i0 + N * b];
                line_acc<K, MDC, true>(g, o);
#pragma unroll
                for (int b = 0; b < N; ++b) v[j][i0 + N * b] = o[b];
            }
        }
        // z derivative lines across the pair
#pragma unroll
        for (int q = 0; q < N2; ++q) {
            const T f[4] = {u[0][q], u[1][q], pair_swap(u[1][q]), pair_swap(u[0][q])};
            T g[2];
#pragma unroll
            for (int j = 0; j < 2; ++j) {
                Acc<T> acc;
#pragma unroll
                for (int b = 0; b < 4; ++b) acc.add(mat<K, MDC>(j, b), f[b]);
                g[j] = acc.get() * (cw[j][q] * r2);
            }
            // the derivative is odd under the mirror: the partner's values
            // change sign in this thread's frame
            const T h[4] = {g[0], g[1], -pair_swap(g[1]), -pair_swap(g[0])};
#pragma unroll
            for (int j = 0; j < 2; ++j) {
                T s = v[j][q];
#pragma unroll
                for (int b = 0; b < 4; ++b) {
                    const double cf = mat<K, MDC>(b, j);
                    if (cf != 0.0) s = fma(T(cf), h[b], s);
                }
                v[j][q] = s;
            }
            __builtin_amdgcn_sched_barrier(0);
        }
        // transposed value sweeps
        zsweep_pair<K, MS, true>(v);
#pragma unroll
        for (int j = 0; j < 2; ++j) {
            sweep2<K, MS, true, 1>(v[j]);
            sweep2<K, MS, true, 0>(v[j]);
        }
        // non-owned positions (some index K) go to the slot array
#pragma unroll
        for (int j = 0; j < 2; ++j)
#pragma unroll
            for (int q = 0; q < N2; ++q) {
                const int a0 = q % N, a1 = q / N;
                if (a0 == K || a1 == K || pl[j] == K) VPP_ST(&slot[(a0 + N * (a1 + N * pl[j])) * CS + c], BC_SLOT, v[j][q]);
            }
    }
    __syncthreads();
    double dsum = 0.0;
    if (active)
        dsum = flush_half_owned<K, T, TX, TY, TZ>(m, tc, slot, CS, v, pl, lx, ly, lz, cx, cy, cz, a.x, a.y, a.part,
                                                  a.nshared, DOT);
    const ColSlots<N, T, NC> slots{slot};
    dsum += upper_faces<K, T, TX, TY, TZ, NTH>(m, tc, slots, a.x, a.y, a.part, a.nshared, DOT);
    if constexpr (DOT) {
        const double sum = block_sum<NTH>(dsum);
        if (threadIdx.x == 0) VPP_ST(&a.dot_part[blockIdx.x], BC_DOT, sum);
    }
}

}  // namespace vpp
