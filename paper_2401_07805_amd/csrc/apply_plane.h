// Plane-per-thread kernels: the tile machinery of apply variant 1 (thread
// mapping, turns of a cell's planes through LDS, write-out) and that kernel.
#pragma once
#include "apply_impl.h"

namespace vpp {

// ---------------------------------------------------------------------------
// Variant 1: one plane of a cell per thread.  The k+1 threads of a cell hold
// its x-planes for the y and z sweeps and its z-planes for the x sweeps, so
// every sweep is register-only with compile-time tables; in between, the
// cell's values turn over through LDS, one write and one read per value and
// turn.  The z derivative is taken on the x-planes (before the x
// interpolation, which commutes with it), so five turns do: phi, u and its z
// derivative there, their two fluxes back.  (A direct x sweep out of LDS reads
// k+1 values per result: 600 instead of 250 LDS accesses per thread at k = 4.)
//
// Groups: for k = 3 and 4 a wave holds 64 / (k+1) whole cells (all 64 lanes at
// k = 3, 60 at k = 4; the spare lanes repeat the group's last thread), so the
// turns stay inside a wave and need no barrier: the LDS accesses of one wave
// complete in order.  At k = 2 a wave would leave a lane idle and tiles would
// be multiples of 21 cells, so the workgroup is one group with barriers.
//
// Layout of a group's buffer: value (x, y, z) of the group's cell c at
// z SZ + y SY + c (k+1) + x.  Writing or reading x-planes touches consecutive
// words over the lanes; z-planes do as well since SZ = 1 mod 32.  The columns
// past the group's last cell are zeros (a neighbour below the tile), which
// lets the write-out use the same buffer as its slot array.

template <int K, int TX, int TY, int TZ, bool W = (K >= 3)>
struct PlaneGeo {
    static constexpr int N = K + 1, NC = TX * TY * TZ;
    static constexpr bool WAVE = W;                      // groups are waves
    static constexpr int CG = WAVE ? 64 / N : NC;        // cells per group
    static constexpr int NG = (NC + CG - 1) / CG;
    static constexpr int NTH = WAVE ? 64 * NG : N * NC;  // threads per workgroup
    static constexpr int SY = N * CG + N;
    static constexpr int SZ = N * SY + (33 - (N * SY) % 32) % 32;
    static constexpr int GB = N * SZ;                    // words per group
    static_assert(SZ % 32 == 1 && SZ >= N * SY, "conflict-free turns");
};

template <typename G, typename T>
struct PlaneSlots {
    const T* s;
    __device__ __forceinline__ int col(int c) const { return G::NG == 1 ? c * G::N : c / G::CG * G::GB + c % G::CG * G::N; }
    __device__ __forceinline__ int zero() const { return G::CG * G::N; }
    __device__ __forceinline__ T get(int a0, int a1, int a2, int h) const
    {
        return VPP_LD(&s[a2 * G::SZ + a1 * G::SY + a0 + h], BC_SLOT);
    }
};

// Orders the LDS accesses of a group: across the workgroup, or inside a wave
// (whose LDS accesses complete in program order: only the compiler must keep it).
template <typename G>
__device__ __forceinline__ void plane_sync()
{
    if constexpr (G::WAVE) {
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
        __builtin_amdgcn_wave_barrier();
        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
    } else {
        __syncthreads();
    }
}

// This thread's x-plane (v[y + N z]) or z-plane (v[x + N y]) to and from the
// group's buffer; px, pz: the buffer at this thread's plane.
template <typename G, typename T>
__device__ __forceinline__ void put_x(T* px, const T (&v)[G::N * G::N])
{
#pragma unroll
    for (int l = 0; l < G::N; ++l)
#pragma unroll
        for (int j = 0; j < G::N; ++j) VPP_ST(&px[l * G::SZ + j * G::SY], BC_SLOT, v[j + G::N * l]);
}
template <typename G, typename T>
__device__ __forceinline__ void get_x(const T* px, T (&v)[G::N * G::N])
{
#pragma unroll
    for (int l = 0; l < G::N; ++l)
#pragma unroll
        for (int j = 0; j < G::N; ++j) v[j + G::N * l] = VPP_LD(&px[l * G::SZ + j * G::SY], BC_SLOT);
}
template <typename G, typename T>
__device__ __forceinline__ void put_z(T* pz, const T (&v)[G::N * G::N])
{
#pragma unroll
    for (int j = 0; j < G::N; ++j)
#pragma unroll
        for (int i = 0; i < G::N; ++i) VPP_ST(&pz[j * G::SY + i], BC_SLOT, v[i + G::N * j]);
}
template <typename G, typename T>
__device__ __forceinline__ void get_z(const T* pz, T (&v)[G::N * G::N])
{
#pragma unroll
    for (int j = 0; j < G::N; ++j)
#pragma unroll
        for (int i = 0; i < G::N; ++i) v[i + G::N * j] = VPP_LD(&pz[j * G::SY + i], BC_SLOT);
}

// out += the transposed 1D table along direction DIR of a plane (v[first + N second]).
template <int K, Mat M, int DIR, typename T>
__device__ __forceinline__ void plane_add_lines(const T (&f)[(K + 1) * (K + 1)], T (&out)[(K + 1) * (K + 1)])
{
    constexpr int N = K + 1, st = DIR == 0 ? 1 : N, so = DIR == 0 ? N : 1;
#pragma unroll
    for (int i = 0; i < N; ++i) {
        T g[N], o[N];
#pragma unroll
        for (int b = 0; b < N; ++b) {
            g[b] = f[i * so + b * st];
            o[b] = out[i * so + b * st];
        }
        line_acc<K, M, true>(g, o);
#pragma unroll
        for (int b = 0; b < N; ++b) out[i * so + b * st] = o[b];
    }
}

// This thread's place: its cell, plane and buffer positions.
template <int K, int TX, int TY, int TZ>
struct PlaneThread {
    using G = PlaneGeo<K, TX, TY, TZ>;
    TileCoord tc;
    int ip;              // its x-plane, and its z-plane after a turn
    int lx, ly, lz;      // cell in the tile
    int cx, cy, cz;      // cell in the mesh
    bool in;             // the cell lies in the mesh
    bool spare;          // repeats the group's last thread: writes nothing out
    int offx, offz;      // its planes in the workgroup's buffer

    __device__ __forceinline__ PlaneThread(const MeshArgs& m, int tile) : tc(tile_coord<K, TX, TY, TZ>(m, tile))
    {
        const int tid = threadIdx.x;
        const int group = G::WAVE ? tid / 64 : 0;
        const int gl = G::WAVE ? tid % 64 : tid;
        const int gcells = min(G::CG, G::NC - group * G::CG);
        spare = gl >= gcells * G::N;
        const int t = spare ? gcells * G::N - 1 : gl;
        const int c = group * G::CG + t / G::N;
        ip = t % G::N;
        lx = c % TX;
        ly = (c / TX) % TY;
        lz = c / (TX * TY);
        cx = tc.t[0] * TX + lx;
        cy = tc.t[1] * TY + ly;
        cz = tc.t[2] * TZ + lz;
        in = cx < m.nc[0] && cy < m.nc[1] && cz < m.nc[2];
        offx = group * G::GB + t;
        offz = group * G::GB + ip * G::SZ + (t - ip);
    }

    // The first group's zero columns, which no turn touches.
    template <typename T>
    __device__ __forceinline__ void clear_zero_columns(T* buf) const
    {
        constexpr int N = G::N, N2 = N * N;
        for (int q = threadIdx.x; q < N * N2; q += G::NTH)
            VPP_ST(&buf[q / N2 * G::SZ + q / N % N * G::SY + N * G::CG + q % N], BC_SLOT, T(0));
    }

    // Its x-plane of the nodal field f.
    template <BcBuf B, typename T>
    __device__ __forceinline__ void load(const MeshArgs& m, const T* __restrict__ f, T (&v)[G::N * G::N]) const
    {
        const int nx = m.nn[0], nxy = m.nn[0] * m.nn[1];
        const int64_t tile0 = uniform_i64(node_index(m, tc.n0[0], tc.n0[1], tc.n0[2]));
        const unsigned lane_b = (unsigned)(K * lx + ip + nx * K * ly + nxy * K * lz) * (unsigned)sizeof(T);
#pragma unroll
        for (int l = 0; l < G::N; ++l)
#pragma unroll
            for (int j = 0; j < G::N; ++j)
                v[j + G::N * l] = VPP_LD(at_byte(f + tile0 + (nx * j + nxy * l), lane_b), B);
    }
};

// Write-out of a plane-per-thread tile: every thread writes the nodes of its
// x-plane a0 = ip that its cell owns (indices below K, and K along a direction
// in which it is the tile's last cell), from its registers plus the slots of
// the cells below it in the tile; same destinations as flush_owned_get.  The
// upper x face falls to the threads of plane K, which own nothing else, and the
// upper y and z faces to the waves that hold the last cells: a separate walk
// over the tile's upper faces, as the other variants use, cost a fifth of this
// kernel's vector instructions.
template <int K, typename T, int TX, int TY, int TZ>
__device__ __forceinline__ double flush_plane(const MeshArgs& m, const PlaneThread<K, TX, TY, TZ>& th, const T* buf,
                                              const T (&o)[(K + 1) * (K + 1)], const T* __restrict__ x,
                                              T* __restrict__ y, T* __restrict__ part, int64_t nshared, bool dot)
{
    constexpr int N = K + 1;
    if (!th.in || th.spare) return 0.0;
    const PlaneSlots<PlaneGeo<K, TX, TY, TZ>, T> slot{buf};
    const TileCoord& tc = th.tc;
    const int ip = th.ip, lx = th.lx, ly = th.ly, lz = th.lz, cx = th.cx, cy = th.cy, cz = th.cz;
    const bool last0 = K * (lx + 1) == tc.ext[0] - 1, last1 = K * (ly + 1) == tc.ext[1] - 1;
    const bool last2 = K * (lz + 1) == tc.ext[2] - 1;
    if (ip == K && !last0) return 0.0;
    const int c = lx + TX * (ly + TY * lz), zero = slot.zero();
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
    const bool p0 = ip == 0;
    const bool b0 = p0 && lx > 0, b1 = ly > 0, b2 = lz > 0;
    const int nb0 = b0 ? slot.col(c - 1) : zero, nb1 = b1 ? slot.col(c - TX) : zero;
    const int nb2 = b2 ? slot.col(c - TX * TY) : zero, nb01 = b0 && b1 ? slot.col(c - 1 - TX) : zero;
    const int nb02 = b0 && b2 ? slot.col(c - 1 - TX * TY) : zero;
    const int nb12 = b1 && b2 ? slot.col(c - TX - TX * TY) : zero;
    const int nb012 = b0 && b1 && b2 ? slot.col(c - 1 - TX - TX * TY) : zero;
    const bool lo0 = p0 && lx == 0 && t0 > 0, hl1 = ly == 0 && t1 > 0, hl2 = lz == 0 && t2 > 0;
    const bool hi0 = ip == K && t0 < nbx, hh1 = last1 && t1 < nby, hh2 = last2 && t2 < nbz;
    const bool s0 = lo0 || hi0;
    const int faces = cell_dirichlet_faces(m, cx, cy, cz);
    const bool dir0 = (p0 && (faces & 1)) || (ip == K && (faces & 2));
    const int i0 = K * cx + ip, j0 = K * cy, l0 = K * cz;
    const unsigned lane_b = (unsigned)(K * lx + ip + nx * K * ly + nxy * K * lz) * (unsigned)sizeof(T);
    const int fz = i0 + nx * j0 + nxy * (t2 - 1);
    const int fy = cz_n + i0 + nx * ((t1 - 1) + nby * (l0 - t2));
    const int fx = cz_n + cy_n + (t0 - 1) + (hi0 ? 1 : 0) + nbx * ((j0 - t1) + ny_free * (l0 - t2));
    const int r0 = lo0 ? 1 : 0, m0 = s0 ? 2 : 1;
    double dsum = 0.0;
    // node (ip, a1, a2) with its x (identity rows copy it, x . Ax needs it)
    auto node = [&](int a1, int a2, T xv) {
        const bool z1 = a1 == 0, z2 = a2 == 0;
        T val = o[a1 + N * a2];
        val += slot.get(K, a1, a2, nb0);   // zeros for every plane but the first
        if (z1) val += slot.get(ip, K, a2, nb1);
        if (z2) val += slot.get(ip, a1, K, nb2);
        if (z1) val += slot.get(K, K, a2, nb01);
        if (z2) val += slot.get(K, a1, K, nb02);
        if (z1 && z2) val += slot.get(ip, K, K, nb12);
        if (z1 && z2) val += slot.get(K, K, K, nb012);
        const int row = nx * a1 + nxy * a2;   // uniform
        const bool lo1 = z1 && hl1, lo2 = z2 && hl2;
        const bool hi1 = a1 == K && hh1, hi2 = a2 == K && hh2;
        if (dir0 || (z1 && (faces & 4)) || (a1 == K && (faces & 8)) || (z2 && (faces & 16)) ||
            (a2 == K && (faces & 32))) {
            VPP_ST(at_byte(yt + row, lane_b), BC_Y, xv);
            if (dot && !(lo0 || lo1 || lo2)) dsum += (double)xv * (double)xv;
            return;
        }
        T* dst = at_byte(yt + row, lane_b);
        const bool s1 = lo1 || hi1, s2 = lo2 || hi2;
        if (s0 || s1 || s2) {
            const int f = s2   ? fz + nx * a1 + (hi2 ? nxy : 0)
                          : s1 ? fy + (hi1 ? nx : 0) + nx * nby * a2
                               : fx + nbx * (a1 + ny_free * a2);
            const int rank = r0 + m0 * ((lo1 ? 1 : 0) + (s1 ? 2 : 1) * (lo2 ? 1 : 0));
            dst = part + ((unsigned)rank * nsh + (unsigned)f);
        }
        VPP_ST(dst, BC_OUT, val);
        if (dot) dsum += (double)xv * (double)val;
    };
    const bool need_x = dot || dir0 || faces != 0;
    {
        T xd[K * K];
        if (need_x) {
#pragma unroll
            for (int a2 = 0; a2 < K; ++a2)
#pragma unroll
                for (int a1 = 0; a1 < K; ++a1)
                    xd[a1 + K * a2] = VPP_LD(at_byte(xt + (nx * a1 + nxy * a2), lane_b), BC_X);
        }
#pragma unroll
        for (int a2 = 0; a2 < K; ++a2)
#pragma unroll
            for (int a1 = 0; a1 < K; ++a1) node(a1, a2, xd[a1 + K * a2]);
    }
    if (last1) {
        T xd[K];
        if (need_x) {
#pragma unroll
            for (int a2 = 0; a2 < K; ++a2) xd[a2] = VPP_LD(at_byte(xt + (nx * K + nxy * a2), lane_b), BC_X);
        }
#pragma unroll
        for (int a2 = 0; a2 < K; ++a2) node(K, a2, xd[a2]);
    }
    if (last2) {
        T xd[N];
        if (need_x) {
#pragma unroll
            for (int a1 = 0; a1 < N; ++a1)
                if (a1 < K || last1) xd[a1] = VPP_LD(at_byte(xt + (nx * a1 + nxy * K), lane_b), BC_X);
        }
#pragma unroll
        for (int a1 = 0; a1 < N; ++a1)
            if (a1 < K || last1) node(a1, K, xd[a1]);
    }
    return dsum;
}

// The cell operator on a cell's planes: u (this thread's x-plane of nodal
// values, Dirichlet entries zeroed) is replaced by its x-plane of A_e u; cw: the
// coefficient factors on its z-plane, wz: its z Gauss weight (mass shift only).
template <typename G, int K, typename T, bool MASS>
__device__ __forceinline__ void plane_operator(const MeshArgs& m, T* px, T* pz, const T (&cw)[G::N * G::N], T wz,
                                               T (&u)[G::N * G::N])
{
    constexpr int N = G::N, N2 = N * N;
    // The x and z derivatives either straight from the nodal values (D) or from
    // the interpolated ones (Dc), at as many operations.  D rounds once less,
    // which counts in FP32 (43 x 37 x 29 Q3: 4.6e-8 against 8.0e-8 relative to
    // FP64); in FP64 its additional constants overflow the scalar registers (196
    // v_readlane per thread at k = 3), while FP32 takes them as literals.
    constexpr bool NODAL = sizeof(T) == 4;
    constexpr Mat DER = NODAL ? MD : MDC;
    // operand: y and z interpolation, z derivative; both turn to z-planes
    sweep2<K, MS, false, 0>(u);
    T v[N2];
#pragma unroll
    for (int q = 0; q < N2; ++q) v[q] = u[q];
    sweep2<K, MS, false, 1>(v);
    plane_sync<G>();
    put_x<G>(px, v);
    if constexpr (NODAL) {
        sweep2<K, MD, false, 1>(u);
    } else {
#pragma unroll
        for (int q = 0; q < N2; ++q) u[q] = v[q];
        sweep2<K, MDC, false, 1>(u);
    }
    plane_sync<G>();
    get_z<G>(pz, v);
    plane_sync<G>();
    put_x<G>(px, u);
    // x: u := values at the Gauss points, v := the transposed derivative of the
    // x flux, at the x nodes (NODAL) or Gauss points
    const T r1 = T(m.rd[1]), r2 = T(m.rd[2]);
#pragma unroll
    for (int j = 0; j < N; ++j) {
        T in_[N], g[N], o[N];
#pragma unroll
        for (int b = 0; b < N; ++b) in_[b] = v[b + N * j];
        line<K, MS, false>(in_, o);
        if constexpr (NODAL) line<K, MD, false>(in_, g);
        else line<K, MDC, false>(o, g);
#pragma unroll
        for (int b = 0; b < N; ++b) {
            u[b + N * j] = o[b];
            g[b] *= cw[b + N * j];
        }
        line<K, DER, true>(g, o);
#pragma unroll
        for (int b = 0; b < N; ++b) v[b + N * j] = o[b];
    }
    // y: the transposed derivative of the y flux (+ the mass shift's
    // mu hx hy hz wref u), at the x Gauss points, into u (NODAL) or added to v
#pragma unroll
    for (int i = 0; i < N; ++i) {
        T in_[N], g[N], o[N];
#pragma unroll
        for (int b = 0; b < N; ++b) in_[b] = u[i + N * b];
        line<K, MDC, false>(in_, g);
#pragma unroll
        for (int b = 0; b < N; ++b) g[b] *= cw[i + N * b] * r1;
        if constexpr (NODAL) {
            line<K, MDC, true>(g, o);
        } else {
#pragma unroll
            for (int b = 0; b < N; ++b) o[b] = v[i + N * b];
            line_acc<K, MDC, true>(g, o);
        }
        if constexpr (MASS) {
            const T ms = T(m.mass) * wz;
#pragma unroll
            for (int b = 0; b < N; ++b) o[b] = fma(ms * T(Tab<K>::t.w[i] * Tab<K>::t.w[b]), in_[b], o[b]);
        }
#pragma unroll
        for (int b = 0; b < N; ++b) (NODAL ? u : v)[i + N * b] = o[b];
    }
    if constexpr (NODAL) plane_add_lines<K, MS, 0>(u, v);
    else sweep2<K, MS, true, 0>(v);
    // z flux: back to the x-planes for its transposed derivative
    plane_sync<G>();
    get_z<G>(pz, u);
    sweep2<K, MS, false, 0>(u);
#pragma unroll
    for (int q = 0; q < N2; ++q) u[q] *= cw[q] * r2;
    sweep2<K, MS, true, 0>(u);
    put_z<G>(pz, u);
    plane_sync<G>();
    get_x<G>(px, u);
    plane_sync<G>();
    put_z<G>(pz, v);
    plane_sync<G>();
    get_x<G>(px, v);
    if constexpr (NODAL) {
        sweep2<K, MS, true, 1>(v);
        plane_add_lines<K, MD, 1>(u, v);
    } else {
        plane_add_lines<K, MDC, 1>(u, v);
        sweep2<K, MS, true, 1>(v);
    }
    sweep2<K, MS, true, 0>(v);
#pragma unroll
    for (int q = 0; q < N2; ++q) u[q] = v[q];
}

// Body of a workgroup on one tile; dot_out: its partial of x . (A x).
template <int K, typename T, int TX, int TY, int TZ, int HV, bool DOT, bool MASS>
__device__ __forceinline__ void plane_tile(const ApplyArgs<T>& a, int tile, T* buf, double* dot_out)
{
    using G = PlaneGeo<K, TX, TY, TZ>;
    constexpr int N = G::N, N2 = N * N;
    const MeshArgs& m = a.m;
    const PlaneThread<K, TX, TY, TZ> th(m, tile);
    const int ip = th.ip;
    const bool in = th.in;
    T* const px = buf + th.offx;
    T* const pz = buf + th.offz;
    th.template clear_zero_columns<T>(buf);

    // x-plane of phi and of the operand (zeros past the mesh; Dirichlet entries
    // zeroed after every load has been issued)
    T cw[N2], u[N2];
    if (in) {
        th.template load<BC_PHI>(m, a.phi, cw);
        th.template load<BC_X>(m, a.x, u);
        const int faces = cell_dirichlet_faces(m, th.cx, th.cy, th.cz);
        if (faces) {
#pragma unroll
            for (int l = 0; l < N; ++l)
#pragma unroll
                for (int j = 0; j < N; ++j)
                    if (local_dirichlet<K>(faces, ip, j, l)) u[j + N * l] = T(0);
        }
    } else {
#pragma unroll
        for (int q = 0; q < N2; ++q) cw[q] = u[q] = T(0);
    }

    // coefficient at the Gauss points of this thread's z-plane
    sweep2<K, MS, false, 0>(cw);
    sweep2<K, MS, false, 1>(cw);
    put_x<G>(px, cw);
    plane_sync<G>();
    get_z<G>(pz, cw);
    sweep2<K, MS, false, 0>(cw);
    // At k = 2 the weights' product is rounded to FP32 once, as in the kernels of
    // one cell per thread, which share the degree's default: with wz rounded first
    // the error relative to FP64 was up to 1.3 times theirs (20^3, law 0: 4.0e-8
    // against 3.6e-8; now 3.2e-8) at the same time (24^3: 9.6 us).  k = 3 and 4
    // keep the rounded wz: 1 to 9 % off the error cost up to 2.5 % of the time.
    using W = std::conditional_t<K == 2, double, T>;
    W wz = W(0);
#pragma unroll
    for (int i = 0; i < N; ++i)
        if (ip == i) wz = W(Tab<K>::t.w[i]);
#pragma unroll
    for (int q = 0; q < N2; ++q)
        cw[q] = coef_scaled<HV>(m, cw[q]) * T(wz * W(Tab<K>::t.w[q % N] * Tab<K>::t.w[q / N]));

    plane_operator<G, K, T, MASS>(m, px, pz, cw, T(wz), u);
    // cell results to the slots: the positions this thread has just read
    put_x<G>(px, u);
    __syncthreads();
    const double d = flush_plane<K, T, TX, TY, TZ>(m, th, buf, u, a.x, a.y, a.part, a.nshared, DOT);
    if constexpr (DOT) {
        const double s = block_sum<G::NTH>(d);
        if (threadIdx.x == 0) VPP_ST(dot_out, BC_DOT, s);
    }
}

// The bound of 128 registers: with the mass term the FP64 kernel took 130 at k = 3
// and lost its fourth wave per SIMD (PCG iteration at 48^3 87.9 -> 83.4 us).
template <int K, typename T, int TX, int TY, int TZ, int HV, bool DOT, bool MASS = false>
__global__ void __launch_bounds__((PlaneGeo<K, TX, TY, TZ>::NTH), (K == 3 && MASS && sizeof(T) == 8 ? 4 : 1))
    apply_plane_kernel(ApplyArgs<T> a)
{
    using G = PlaneGeo<K, TX, TY, TZ>;
    __shared__ T buf[G::NG * G::GB];
    VPP_BC_BEGIN(a.x, a.y, a.phi, a.part, a.dot_part, buf, (int64_t)a.m.nn[0] * a.m.nn[1] * a.m.nn[2],
                 8 * a.nshared, (int64_t)gridDim.x, G::NG * G::GB);
    if (a.done && *a.done) return;
    plane_tile<K, T, TX, TY, TZ, HV, DOT, MASS>(a, xcd_tile(blockIdx.x, gridDim.x), buf, a.dot_part + blockIdx.x);
}

}  // namespace vpp
