// Diagonal, fill and batched kernels and their launchers.
#include "apply_plane.h"
#include "shared_nodes.h"

namespace vpp {

// ---------------------------------------------------------------------------
// Diagonal: diag_a = sum_q cw_q sum_d rd[d] (dN_a/dxi_d (x_q))^2 (+ the mass
// shift's mu hx hy hz sum_q wref_q N_a(x_q)^2), from squared 1D tables (each
// term is a product of three 1D factors).  Runs once per phi, one launch per
// cell colour (cell_color), adding into the zeroed diagonal without atomics.

template <int K, int HV>
__global__ void __launch_bounds__(64) diag_kernel(MeshArgs m, const double* __restrict__ phi,
                                                   double* __restrict__ diag, CellColor cc)
{
    constexpr int N = K + 1, N3 = N * N * N;
    // phi is gathered by the (instrumented) coefficient helper
    VPP_BC_BEGIN((const double*)nullptr, (const double*)nullptr, phi, (const double*)nullptr,
                 (const double*)nullptr, (const double*)nullptr, (int64_t)m.nn[0] * m.nn[1] * m.nn[2], 0, 0, 0);
    int cx, cy, cz;
    if (!color_cell(cc, (int64_t)blockIdx.x * blockDim.x + threadIdx.x, cx, cy, cz)) return;
    double A[N3], Z[N3], Y[N3], out[N3];
    cell_coefficient<K, HV>(m, phi, cx, cy, cz, A);
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
    if (m.mass != 0.0) {
        // mass shift: mu hx hy hz sum_q wref_q N_a(x_q)^2
#pragma unroll
        for (int q = 0; q < N3; ++q) A[q] = m.mass * wref<K>(q % N, (q / N) % N, q / (N * N));
        sweep3<K, MS2, true, 2>(A);
        sweep3<K, MS2, true, 1>(A);
        sweep3<K, MS2, true, 0>(A);
#pragma unroll
        for (int q = 0; q < N3; ++q) out[q] += A[q];
    }
    const int64_t nx = m.nn[0], nxy = (int64_t)m.nn[0] * m.nn[1];
    const int64_t base = node_index(m, (int64_t)K * cx, (int64_t)K * cy, (int64_t)K * cz);
#pragma unroll
    for (int a2 = 0; a2 < N; ++a2)
#pragma unroll
        for (int a1 = 0; a1 < N; ++a1)
#pragma unroll
            for (int a0 = 0; a0 < N; ++a0)
                diag[base + a0 + nx * a1 + nxy * a2] += out[a0 + N * (a1 + N * a2)];
}

__global__ void fix_diagonal_kernel(MeshArgs m, double* __restrict__ diag, double* __restrict__ inv64,
                                    float* __restrict__ inv32)
{
    const int64_t n = (int64_t)m.nn[0] * m.nn[1] * m.nn[2];
    for (int64_t g = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; g < n;
         g += (int64_t)gridDim.x * blockDim.x) {
        const int i = (int)(g % m.nn[0]), j = (int)((g / m.nn[0]) % m.nn[1]),
                  l = (int)(g / ((int64_t)m.nn[0] * m.nn[1]));
        double d = diag[g];
        if (is_dirichlet(m, i, j, l)) d = 1.0;
        diag[g] = d;
        const double r = 1.0 / d;
        inv64[g] = r;
        inv32[g] = (float)r;
    }
}

template <typename T>
__global__ void fill_kernel(T* __restrict__ p, int64_t n, T v)
{
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += (int64_t)gridDim.x * blockDim.x)
        p[i] = v;
}

// ---------------------------------------------------------------------------
// Host launchers.

template <typename T>
hipError_t launch_fill(T* p, int64_t n, T v, hipStream_t s)
{
    if (n <= 0) return hipSuccess;
    const int64_t want = (n + 255) / 256;
    const int blocks = (int)(want < 8192 ? want : 8192);
    hipLaunchKernelGGL(fill_kernel<T>, dim3(blocks), dim3(256), 0, s, p, n, v);
    return hipGetLastError();
}
template hipError_t launch_fill<double>(double*, int64_t, double, hipStream_t);
template hipError_t launch_fill<float>(float*, int64_t, float, hipStream_t);
template hipError_t launch_fill<int>(int*, int64_t, int, hipStream_t);

hipError_t launch_diag(int k, const MeshArgs& m, const double* phi, double* diag, hipStream_t s)
{
    // one launch per cell colour: the scatter into the nodes needs no atomics
#define VPP_DIAG(K)                                                                                              \
    return for_each_color(m, 64, [&](const CellColor& cc, int blocks) {                                         \
        if (m.heaviside == 0) hipLaunchKernelGGL((diag_kernel<K, 0>), dim3(blocks), dim3(64), 0, s, m, phi, diag, cc); \
        else if (m.heaviside == 1)                                                                               \
            hipLaunchKernelGGL((diag_kernel<K, 1>), dim3(blocks), dim3(64), 0, s, m, phi, diag, cc);            \
        else if (m.heaviside == 2)                                                                               \
            hipLaunchKernelGGL((diag_kernel<K, 2>), dim3(blocks), dim3(64), 0, s, m, phi, diag, cc);            \
        else hipLaunchKernelGGL((diag_kernel<K, 3>), dim3(blocks), dim3(64), 0, s, m, phi, diag, cc);           \
    });
    switch (k) {
    case 2: VPP_DIAG(2)
    case 3: VPP_DIAG(3)
    case 4: VPP_DIAG(4)
    default: return hipErrorInvalidValue;
    }
#undef VPP_DIAG
}

hipError_t launch_fix_diagonal(const MeshArgs& m, double* diag, double* inv64, float* inv32, hipStream_t s)
{
    const int64_t n = (int64_t)m.nn[0] * m.nn[1] * m.nn[2];
    const int64_t want = (n + 255) / 256;
    const int blocks = (int)(want < 8192 ? want : 8192);
    hipLaunchKernelGGL(fix_diagonal_kernel, dim3(blocks), dim3(256), 0, s, m, diag, inv64, inv32);
    return hipGetLastError();
}

// ---------------------------------------------------------------------------
// Assembly of shared-face nodes.  A node lies in one or two tiles along each
// direction (two when it sits on an interior tile boundary); its value is the
// sum of the partial slots of all tiles holding it, taken in a fixed order
// (z, y, x tile index ascending), so the result is deterministic.

// Shared nodes, streamed in the order of their enumeration f, two per thread:
// the value is the sum of the partials the 2, 4 or 8 tiles holding the node
// wrote to part[rank * stride + f], taken in rank order (so the result is
// deterministic).  Every shared node has at least two sharers, so ranks 0 and 1
// are read as 16-byte pairs (stride and f are even).
template <typename T>
struct Pair;
template <>
struct Pair<double> {
    using type = double2;
};
template <>
struct Pair<float> {
    using type = float2;
};

// Nodes f and f + 1 (f even) of the enumeration: their positions and sharer
// counts first (no memory), then every partial of both loaded before any is used.
template <typename T>
__device__ __forceinline__ void assemble_pair(const SharedEnum& e, const MeshArgs& m, const T* __restrict__ part,
                                              int64_t stride, int64_t f, int64_t count, T* __restrict__ y)
{
    using P = typename Pair<T>::type;
    int i0, j0, l0, i1 = 0, j1 = 0, l1 = 0;
    shared_node(e, f, i0, j0, l0);
    const bool has1 = f + 1 < count;
    if (has1) shared_node(e, f + 1, i1, j1, l1);
    const int n0 = is_dirichlet(m, i0, j0, l0) ? 0 : sharer_count(e, i0, j0, l0);
    const int n1 = !has1 || is_dirichlet(m, i1, j1, l1) ? 0 : sharer_count(e, i1, j1, l1);
    const P r0 = VPP_LD(reinterpret_cast<const P*>(part + f), BC_PART);
    const P r1 = VPP_LD(reinterpret_cast<const P*>(part + stride + f), BC_PART);
    T x0[6], x1[6];
#pragma unroll
    for (int c = 2; c < 8; ++c) {
        x0[c - 2] = c < n0 ? VPP_LD(&part[c * stride + f], BC_PART) : T(0);
        x1[c - 2] = c < n1 ? VPP_LD(&part[c * stride + f + 1], BC_PART) : T(0);
    }
    T v0 = r0.x + r1.x, v1 = r0.y + r1.y;
#pragma unroll
    for (int c = 2; c < 8; ++c) {
        if (c < n0) v0 += x0[c - 2];
        if (c < n1) v1 += x1[c - 2];
    }
    if (n0 > 0) VPP_ST(&y[i0 + (int64_t)m.nn[0] * (j0 + (int64_t)m.nn[1] * l0)], BC_Y, v0);
    if (n1 > 0) VPP_ST(&y[i1 + (int64_t)m.nn[0] * (j1 + (int64_t)m.nn[1] * l1)], BC_Y, v1);
}

template <typename T>
__global__ void __launch_bounds__(256) assemble_kernel(AssembleArgs<T> a)
{
    VPP_BC_BEGIN((const T*)nullptr, a.y, (const T*)nullptr, a.part, a.dot_part, (const T*)nullptr,
                 (int64_t)a.m.nn[0] * a.m.nn[1] * a.m.nn[2], 8 * a.nshared, (int64_t)a.ndot, 0);
    if (a.done && *a.done) return;
    if (a.dot && blockIdx.x == 0) {
        // x . y from the per-workgroup partials, summed in a fixed order
        __shared__ double red[256];
        double s = 0.0;
        for (int i = threadIdx.x; i < a.ndot; i += 256) s += VPP_LD(&a.dot_part[i], BC_DOT);
        red[threadIdx.x] = s;
        __syncthreads();
        for (int w = 128; w > 0; w >>= 1) {
            if ((int)threadIdx.x < w) red[threadIdx.x] += red[threadIdx.x + w];
            __syncthreads();
        }
        if (threadIdx.x == 0) *a.dot = red[0];
    }
    const SharedEnum& e = a.e;
    const int64_t count = e.cz + e.cy + e.cx;
    for (int64_t f = 2 * ((int64_t)blockIdx.x * 256 + threadIdx.x); f < count; f += 2 * (int64_t)gridDim.x * 256) {
        assemble_pair(e, a.m, a.part, a.nshared, f, count, a.y);
    }
}

template <typename T>
hipError_t launch_assemble(const AssembleArgs<T>& a, hipStream_t s)
{
    const int64_t want = (a.e.cz + a.e.cy + a.e.cx + 511) / 512;
    const int blocks = (int)(want < 1 ? 1 : (want < 8192 ? want : 8192));
    hipLaunchKernelGGL(assemble_kernel<T>, dim3(blocks), dim3(256), 0, s, a);
    return hipGetLastError();
}
template hipError_t launch_assemble<double>(const AssembleArgs<double>&, hipStream_t);
template hipError_t launch_assemble<float>(const AssembleArgs<float>&, hipStream_t);

int device_cu_count()
{
    static int cached = -1;
    if (cached < 0) {
        int dev = 0, n = 0;
        if (hipGetDevice(&dev) != hipSuccess ||
            hipDeviceGetAttribute(&n, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess || n < 1)
            n = 1;
        cached = n;
    }
    return cached;
}

// ---------------------------------------------------------------------------
// Batched apply: one launch over the (problem, tile, rhs) items of several
// independent meshes, a workgroup each, the items of one tile consecutive (on one
// XCD, so the tile's phi stays in its L2 for the next right-hand side); a second
// launch assembles the shared nodes of every (problem, rhs).
//
// An item runs the single apply's body: cell per thread at k = 2, plane per
// thread at k = 3, with its registers (two waves per SIMD at k = 2).  A
// persistent kernel that pulled tiles from a queue and kept a tile's coefficient
// over its right-hand sides held 421-512 registers, one wave per SIMD: 8 meshes of
// 16^3-64^3 Q2 x 4 right-hand sides 607 us against 430, the apply of a PCG over
// 16 systems of 16^3-40^3 60 against 43; 8 Q3 meshes of 8^3-32^3 x 4 228 against
// 103 (there cell per thread, spilled).

template <int K, int TX, int TY, int TZ>
constexpr int batch_threads()
{
    if constexpr (K == 2) return TX * TY * TZ;
    else return PlaneGeo<K, TX, TY, TZ>::NTH;
}

template <int K, int TX, int TY, int TZ>
constexpr int batch_lds()
{
    if constexpr (K == 2) return (K + 1) * (K + 1) * (K + 1) * (TX * TY * TZ + 1);
    else return PlaneGeo<K, TX, TY, TZ>::NG * PlaneGeo<K, TX, TY, TZ>::GB;
}

// DM & 1: x . Ax partials (batched PCG), DM & 2: mass shift (zero adds exact zeros).
template <int K, int TX, int TY, int TZ, int HV, int DM>
__global__ void __launch_bounds__((batch_threads<K, TX, TY, TZ>())) batch_apply_kernel(BatchArgs a)
{
    constexpr int LDS = batch_lds<K, TX, TY, TZ>();
    constexpr bool dot = (DM & 1) != 0, mass = (DM & 2) != 0;
    __shared__ double slot[LDS];
    const int item = xcd_tile(blockIdx.x, gridDim.x);
    const BatchProblem& P = a.probs[__builtin_amdgcn_readfirstlane(a.owner[item])];
    const int local = item - P.tile_begin, tile = local / P.nrhs, r = local - tile * P.nrhs;   // batch_items' order
    const int rhs = P.rhs_begin + r;
    if (a.st && a.st[rhs].halt[a.par]) return;   // a system that has stopped
    const ApplyArgs<double> t{P.m, a.x[rhs], a.y[rhs], P.phi, a.part + P.part_begin + (int64_t)r * 8 * P.nshared,
                              P.nshared, dot ? a.dot_part + P.dot_begin : nullptr, nullptr, nullptr, true};
    // a tile's partial where its single apply's workgroup puts it: the same sum
    double* const dot_out = t.dot_part + r * P.ntiles + xcd_block(tile, P.ntiles);
    VPP_BC_BEGIN(t.x, t.y, t.phi, t.part, t.dot_part, slot, (int64_t)t.m.nn[0] * t.m.nn[1] * t.m.nn[2],
                 8 * t.nshared, (int64_t)P.nrhs * P.ntiles, LDS);
    if constexpr (K == 2) slot_tile<K, double, TX, TY, TZ, HV, dot, mass>(t, tile, slot, dot_out);
    else plane_tile<K, double, TX, TY, TZ, HV, dot, mass>(t, tile, slot, dot_out);
}

struct BatchAssembleArgs {
    const BatchProblem* probs;
    int nprob;
    double* const* y;
    double* part;
};

// grid.y = (problem, rhs) pair; grid.x strides over that pair's shared nodes.
__global__ void __launch_bounds__(256) batch_assemble_kernel(BatchAssembleArgs a)
{
    int pr = blockIdx.y, pi = 0;
    for (; pi < a.nprob; ++pi) {
        if (pr < a.probs[pi].nrhs) break;
        pr -= a.probs[pi].nrhs;
    }
    if (pi >= a.nprob) return;
    const BatchProblem& P = a.probs[pi];
    const int64_t ns = P.nshared;
    const double* part = a.part + P.part_begin + (int64_t)pr * 8 * ns;
    double* y = a.y[P.rhs_begin + pr];
    VPP_BC_BEGIN((const double*)nullptr, y, (const double*)nullptr, part, (const double*)nullptr,
                 (const double*)nullptr, (int64_t)P.m.nn[0] * P.m.nn[1] * P.m.nn[2], 8 * ns, 0, 0);
    const SharedEnum& e = P.se;
    const int64_t count = e.cz + e.cy + e.cx;
    for (int64_t f = 2 * ((int64_t)blockIdx.x * 256 + threadIdx.x); f < count; f += 2 * (int64_t)gridDim.x * 256)
        assemble_pair(e, P.m, part, ns, f, count, y);
}

#define VPP_BATCH_CONFIGS(X) \
    X(2, 16, 8, 4)           \
    X(2, 32, 4, 4)           \
    X(2, 8, 8, 4)            \
    X(2, 16, 4, 4)           \
    X(2, 8, 4, 4)            \
    X(3, 8, 4, 4)            \
    X(3, 4, 4, 4)

template <int K, int TX, int TY, int TZ, int HV>
static void launch_batch_tiles(const BatchArgs& a, hipStream_t s)
{
    const dim3 g(a.nitems), blk(batch_threads<K, TX, TY, TZ>());
    switch ((a.st ? 1 : 0) | (a.any_mass ? 2 : 0)) {
    case 0: hipLaunchKernelGGL((batch_apply_kernel<K, TX, TY, TZ, HV, 0>), g, blk, 0, s, a); break;
    case 1: hipLaunchKernelGGL((batch_apply_kernel<K, TX, TY, TZ, HV, 1>), g, blk, 0, s, a); break;
    case 2: hipLaunchKernelGGL((batch_apply_kernel<K, TX, TY, TZ, HV, 2>), g, blk, 0, s, a); break;
    default: hipLaunchKernelGGL((batch_apply_kernel<K, TX, TY, TZ, HV, 3>), g, blk, 0, s, a); break;
    }
}

hipError_t launch_batch_apply(const LaunchCfg& c, int k, const BatchArgs& a, int total_rhs, bool tiles_only,
                              hipStream_t s)
{
    if (a.nitems < 1) return hipErrorInvalidValue;
#define VPP_BL(K, TX, TY, TZ)                                                                       \
    if (k == K && c.variant == 4 && c.tile[0] == TX && c.tile[1] == TY && c.tile[2] == TZ) {       \
        if (a.heaviside == 0) launch_batch_tiles<K, TX, TY, TZ, 0>(a, s);                           \
        else launch_batch_tiles<K, TX, TY, TZ, 1>(a, s);                                            \
        hipError_t e = hipGetLastError();                                                           \
        if (e != hipSuccess || tiles_only) return e;                                                \
        BatchAssembleArgs b{a.probs, a.nprob, a.y, a.part};                                         \
        const int64_t want = (a.max_shared + 511) / 512;                                            \
        const unsigned gx = (unsigned)(want < 1 ? 1 : (want < 512 ? want : 512));                   \
        hipLaunchKernelGGL(batch_assemble_kernel, dim3(gx, (unsigned)total_rhs), dim3(256), 0, s, b);  \
        return hipGetLastError();                                                                   \
    }
    VPP_BATCH_CONFIGS(VPP_BL)
#undef VPP_BL
    return hipErrorInvalidValue;
}

bool batch_config_supported(const LaunchCfg& c, int k)
{
#define VPP_BS(K, TX, TY, TZ) \
    if (k == K && c.variant == 4 && c.tile[0] == TX && c.tile[1] == TY && c.tile[2] == TZ) return true;
    VPP_BATCH_CONFIGS(VPP_BS)
#undef VPP_BS
    return false;
}

int list_batch_configs(int k, LaunchCfg* out, int cap)
{
    int n = 0;
#define VPP_BLIST(K, TX, TY, TZ)                                      \
    if (k == K) {                                                     \
        if (n < cap && out) out[n] = LaunchCfg{4, {TX, TY, TZ}};     \
        ++n;                                                          \
    }
    VPP_BATCH_CONFIGS(VPP_BLIST)
#undef VPP_BLIST
    return n;
}

unsigned long long bounds_count_misc() { return bc_count_here(); }

}  // namespace vpp
