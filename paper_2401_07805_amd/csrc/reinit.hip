// The operator of the reinitialization step (Eq. reinitialization, semi-implicit
// Euler in pseudo-time; its diagonal and right-hand side are in levelset.hip):
//   A u = (u, v)/dtau + eps ((grad u . n)(grad v . n)),
// n the nodal normal interpolated at the Gauss points as it is, natural
// conditions on every face.  Plane per thread on tiles, like apply variant 1:
// the three normal components and u turn to z-planes, the flux s n (s = eps W
// grad u . n) turns back.
//
// What bounds it: vector instructions (four fields interpolated per apply) at
// two waves per SIMD (k = 3: 96 values per thread live).  The one-cell-per-
// thread kernel (levelset.hip, kept for meshes that the tiles would mostly pad
// or not address: reinit_config) holds 4 (k+1)^3 values per lane, spills at k = 3
// and 4, and writes (k+1)^3 results per cell to memory for a second kernel to
// sum; here the cells of a tile are summed in LDS and only the tile faces go
// through partials, which the CG update assembles.  Operator per iteration of
// the step, both launches before, us: 40x36x27 Q3 133 -> 28, 64^3 Q2 75 -> 45;
// whole step: 39.8 -> 12.3 ms, 18.6 -> 14.0 ms, 24x25x23 Q4 149.5 -> 19.2 ms.
#include "apply_plane.h"
#include "tile_rules.h"

namespace vpp {

namespace {

// This thread's z-plane of the nodal field f at the Gauss points.
template <BcBuf F, int K, int TX, int TY, int TZ>
__device__ __forceinline__ void field_at_gauss(const PlaneThread<K, TX, TY, TZ>& th, const MeshArgs& m,
                                               const double* __restrict__ f, double* px, double* pz,
                                               double (&v)[(K + 1) * (K + 1)])
{
    using G = PlaneGeo<K, TX, TY, TZ>;
    constexpr int N2 = G::N * G::N;
    if (th.in) {
        th.template load<F>(m, f, v);
    } else {
#pragma unroll
        for (int q = 0; q < N2; ++q) v[q] = 0.0;
    }
    sweep2<K, MS, false, 0>(v);
    sweep2<K, MS, false, 1>(v);
    plane_sync<G>();   // the previous turn has been read
    put_x<G>(px, v);
    plane_sync<G>();
    get_z<G>(pz, v);
    sweep2<K, MS, false, 0>(v);
}

template <int K, int TX, int TY, int TZ, bool DOT>
__global__ void __launch_bounds__((PlaneGeo<K, TX, TY, TZ>::NTH)) reinit_plane_kernel(ReinitApplyArgs a)
{
    using G = PlaneGeo<K, TX, TY, TZ>;
    constexpr int N = G::N, N2 = N * N;
    __shared__ double buf[G::NG * G::GB];
    const MeshArgs& m = a.r.g.m;
    VPP_BC_BEGIN(a.x, a.y, (const double*)nullptr, a.part, a.dot_part, buf, (int64_t)m.nn[0] * m.nn[1] * m.nn[2],
                 8 * a.nshared, (int64_t)gridDim.x, G::NG * G::GB);
    VPP_BC_FIELDS(a.r.n0, a.r.n1, a.r.n2, (int64_t)m.nn[0] * m.nn[1] * m.nn[2]);
    if (a.done && *a.done) return;
    const PlaneThread<K, TX, TY, TZ> th(m, xcd_tile(blockIdx.x, gridDim.x));
    double* const px = buf + th.offx;
    double* const pz = buf + th.offz;
    th.template clear_zero_columns<double>(buf);

    double wz = 0.0;
#pragma unroll
    for (int i = 0; i < N; ++i)
        if (th.ip == i) wz = Tab<K>::t.w[i];
    double n0[N2], n1[N2], n2[N2];
    field_at_gauss<BC_N0, K, TX, TY, TZ>(th, m, a.r.n0, px, pz, n0);
    field_at_gauss<BC_N1, K, TX, TY, TZ>(th, m, a.r.n1, px, pz, n1);
    field_at_gauss<BC_N2, K, TX, TY, TZ>(th, m, a.r.n2, px, pz, n2);

    // u and its z derivative on the x-planes, both turned
    double u[N2], s[N2];
    if (th.in) {
        th.template load<BC_X>(m, a.x, u);
    } else {
#pragma unroll
        for (int q = 0; q < N2; ++q) u[q] = 0.0;
    }
    sweep2<K, MS, false, 0>(u);
    sweep2<K, MS, false, 1>(u);
    plane_sync<G>();
    put_x<G>(px, u);
    sweep2<K, MDC, false, 1>(u);
    plane_sync<G>();
    get_z<G>(pz, s);
    plane_sync<G>();
    put_x<G>(px, u);
    plane_sync<G>();
#pragma unroll
    for (int q = 0; q < N2; ++q) u[q] = s[q];
    get_z<G>(pz, s);
    sweep2<K, MS, false, 0>(u);   // u at the Gauss points
    sweep2<K, MS, false, 0>(s);   // its z derivative there
    // s := grad u . n, direction by direction
    const double ih0 = a.r.g.ih[0], ih1 = a.r.g.ih[1], ih2 = a.r.g.ih[2];
#pragma unroll
    for (int q = 0; q < N2; ++q) s[q] *= n2[q] * ih2;
#pragma unroll
    for (int j = 0; j < N; ++j) {
        double in[N], g[N];
#pragma unroll
        for (int b = 0; b < N; ++b) in[b] = u[b + N * j];
        line<K, MDC, false>(in, g);
#pragma unroll
        for (int b = 0; b < N; ++b) s[b + N * j] = fma(n0[b + N * j] * ih0, g[b], s[b + N * j]);
    }
#pragma unroll
    for (int i = 0; i < N; ++i) {
        double in[N], g[N];
#pragma unroll
        for (int b = 0; b < N; ++b) in[b] = u[i + N * b];
        line<K, MDC, false>(in, g);
#pragma unroll
        for (int b = 0; b < N; ++b) s[i + N * b] = fma(n1[i + N * b] * ih1, g[b], s[i + N * b]);
    }
    // mass term in u; s := eps W s; fluxes along x and y added, z turned back
    const double vw = a.r.g.vol * wz;
#pragma unroll
    for (int q = 0; q < N2; ++q) {
        const double w = vw * (Tab<K>::t.w[q % N] * Tab<K>::t.w[q / N]);
        u[q] *= a.r.idtau * w;
        s[q] *= a.r.eps * w;
    }
#pragma unroll
    for (int j = 0; j < N; ++j) {
        double g[N], o[N];
#pragma unroll
        for (int b = 0; b < N; ++b) {
            g[b] = s[b + N * j] * n0[b + N * j] * ih0;
            o[b] = u[b + N * j];
        }
        line_acc<K, MDC, true>(g, o);
#pragma unroll
        for (int b = 0; b < N; ++b) u[b + N * j] = o[b];
    }
#pragma unroll
    for (int i = 0; i < N; ++i) {
        double g[N], o[N];
#pragma unroll
        for (int b = 0; b < N; ++b) {
            g[b] = s[i + N * b] * n1[i + N * b] * ih1;
            o[b] = u[i + N * b];
        }
        line_acc<K, MDC, true>(g, o);
#pragma unroll
        for (int b = 0; b < N; ++b) u[i + N * b] = o[b];
    }
#pragma unroll
    for (int q = 0; q < N2; ++q) s[q] *= n2[q] * ih2;
    sweep2<K, MS, true, 0>(u);
    sweep2<K, MS, true, 0>(s);
    put_z<G>(pz, s);   // the positions this thread read last
    plane_sync<G>();
    get_x<G>(px, s);
    plane_sync<G>();
    put_z<G>(pz, u);
    plane_sync<G>();
    get_x<G>(px, u);
#pragma unroll
    for (int j = 0; j < N; ++j) {
        double g[N], o[N];
#pragma unroll
        for (int b = 0; b < N; ++b) {
            g[b] = s[j + N * b];
            o[b] = u[j + N * b];
        }
        line_acc<K, MDC, true>(g, o);
#pragma unroll
        for (int b = 0; b < N; ++b) u[j + N * b] = o[b];
    }
    sweep2<K, MS, true, 1>(u);
    sweep2<K, MS, true, 0>(u);
    put_x<G>(px, u);
    __syncthreads();
    const double d = flush_plane<K, double, TX, TY, TZ>(m, th, buf, u, a.x, a.y, a.part, a.nshared, DOT);
    if constexpr (DOT) {
        const double sum = block_sum<G::NTH>(d);
        if (threadIdx.x == 0) VPP_ST(&a.dot_part[blockIdx.x], BC_DOT, sum);
    }
}

template <int K, int TX, int TY, int TZ>
hipError_t launch_reinit_tiles(const ReinitApplyArgs& a, hipStream_t s)
{
    const dim3 g(a.r.g.m.ntile[0] * a.r.g.m.ntile[1] * a.r.g.m.ntile[2]);
    const dim3 b(PlaneGeo<K, TX, TY, TZ>::NTH);
    if (a.dot_part) hipLaunchKernelGGL((reinit_plane_kernel<K, TX, TY, TZ, true>), g, b, 0, s, a);
    else hipLaunchKernelGGL((reinit_plane_kernel<K, TX, TY, TZ, false>), g, b, 0, s, a);
    return hipGetLastError();
}

}  // namespace

unsigned long long bounds_count_reinit() { return bc_count_here(); }

int reinit_dot_partials(int k, const MeshArgs& m)
{
    if (reinit_config(k, m).variant == 1) return (int)tile_count64(m);
    const int64_t n = (int64_t)m.nn[0] * m.nn[1] * m.nn[2];
    return (int)std::max<int64_t>(1, std::min<int64_t>(kMaxRedBlocks, (n + 1023) / 1024));
}

hipError_t launch_reinit_apply(int k, const ReinitApplyArgs& a, hipStream_t s)
{
    const MeshArgs& m = a.r.g.m;
    const LaunchCfg c = reinit_config(k, m);
    for (int d = 0; d < 3; ++d)
        if (m.ntile[d] != (m.nc[d] + c.tile[d] - 1) / c.tile[d]) return hipErrorInvalidValue;
    if (c.variant != 1) return launch_reinit_cells(k, a, reinit_dot_partials(k, m), s);
    hipError_t e;
    if (k == 2) e = launch_reinit_tiles<2, 8, 4, 2>(a, s);
    else if (k == 4) e = launch_reinit_tiles<4, 4, 3, 2>(a, s);
    else if (k != 3) return hipErrorInvalidValue;
    else if (c.tile[2] == 2) e = launch_reinit_tiles<3, 4, 4, 2>(a, s);
    else e = launch_reinit_tiles<3, 4, 4, 4>(a, s);
    if (e != hipSuccess || a.tiles_only) return e;
    const AssembleArgs<double> b{m, shared_enum(m, k, c.tile), a.part, a.nshared, a.y, nullptr, 0, nullptr, a.done};
    return launch_assemble<double>(b, s);
}

}  // namespace vpp
