// Which kernel configuration a mesh gets (host code, so that the rules are
// checked on the CPU), and what a configuration can address.
#pragma once
#include <algorithm>

#include "kernels.h"

namespace vpp {

inline void set_tiles(MeshArgs& m, const LaunchCfg& c)
{
    for (int d = 0; d < 3; ++d) m.ntile[d] = (m.nc[d] + c.tile[d] - 1) / c.tile[d];
}

inline int64_t tile_count64(const MeshArgs& m) { return (int64_t)m.ntile[0] * m.ntile[1] * m.ntile[2]; }

// Threads of a workgroup of configuration c.
inline int tile_threads(int k, const LaunchCfg& c)
{
    const int cells = c.tile[0] * c.tile[1] * c.tile[2];
    if (c.variant == 1 || (c.variant == 4 && k == 3)) {   // plane per thread (PlaneGeo)
        if (k == 2) return 3 * cells;
        const int per_wave = 64 / (k + 1);
        return 64 * ((cells + per_wave - 1) / per_wave);
    }
    return c.variant == 2 ? 2 * cells : cells;
}

// Largest offset, in values, that a lane adds to its tile's base: the tile
// kernels form it in bytes with 32 bits (gather_cell_t, PlaneThread::load, the
// write-outs; their other terms are 64-bit).  Only cells of the mesh are
// addressed, so a tile deeper than the mesh counts as the mesh.
inline int64_t lane_reach(int k, const MeshArgs& m, const LaunchCfg& c)
{
    const int64_t nx = m.nn[0], nxy = nx * m.nn[1];
    int64_t last[3];
    for (int d = 0; d < 3; ++d) last[d] = (int64_t)k * (std::min(c.tile[d], m.nc[d]) - 1);
    if (c.variant == 2) last[2] += k;   // half-cell lanes start at one of their cell's planes
    return last[0] + k + nx * last[1] + nxy * last[2];
}

// Whether a tile kernel of configuration c addresses all of the mesh: 32-bit
// lane offsets (bytes) and partial indices, below 2^32 threads in a launch.
inline bool tiles_fit(int k, MeshArgs m, const LaunchCfg& c, size_t value_bytes)
{
    constexpr int64_t lim = int64_t(1) << 32;
    set_tiles(m, c);
    return lane_reach(k, m, c) * (int64_t)value_bytes < lim && 8 * shared_stride(m) < lim &&
           tile_count64(m) * tile_threads(k, c) < lim;
}

// The first of the n configurations that fits the mesh, else the first.
inline LaunchCfg first_fit(int k, const MeshArgs& m, const LaunchCfg* c, int n, size_t value_bytes)
{
    for (int i = 0; i < n; ++i)
        if (tiles_fit(k, m, c[i], value_bytes)) return c[i];
    return c[0];
}

inline int64_t cell_count(const MeshArgs& m) { return (int64_t)m.nc[0] * m.nc[1] * m.nc[2]; }

// Kernel configuration of a new problem, by degree, precision and number of
// cells (vpp_tune measures instead).  Measured hot, one apply, us, FP64 / FP32:
//  k = 2: the plane kernel gives a small mesh three times the waves of the
//    cell-per-thread one, each with a third of the serial work (24^3 cells: 11.1
//    against 12.7 / 10.8 against 12.9); a mesh that fills the GPU prefers the
//    latter's fewer LDS accesses (32^3: 12.9 against 13.1 in FP64 but still 11.1
//    against 13.0 in FP32; 48^3: 17.9 against 22.5 / 14.9 against 16.6).
//  k = 3: small tiles until there are enough of them for every CU (20^3: 4x4x2
//    13.6 against 17.3 with 8x4x4), then the fewer shared nodes of 8x4x4 (32^3:
//    19.7 against 20.5, 64^3: 80 against 88 / 52 against 56).
//  k = 4: the same, in multiples of the 12 cells of a wave (16^3: 4x3x2 16.1
//    against 17.6 with 4x4x3; 32^3: 35.4 against 38.9; in FP32 6x4x2 23.1
//    against 24.1 with 4x4x3).
// A wide and shallow box whose lane offsets would pass 32 bits with that tile
// (2576 x 2576 x 4 cells at k = 3, 2048 x 2048 x 3 at k = 4) takes a shallower one.
inline LaunchCfg default_config(int k, bool f32, const MeshArgs& m)
{
    const size_t vb = f32 ? 4 : 8;
    const int64_t ncell = cell_count(m);
    if (k == 2) {
        if (ncell <= (f32 ? 50000 : 20000)) return LaunchCfg{1, {8, 4, 2}};
        const LaunchCfg c[3] = {f32 ? LaunchCfg{4, {16, 8, 4}} : LaunchCfg{4, {8, 8, 4}}, {4, {8, 8, 4}}, {1, {8, 4, 2}}};
        return first_fit(k, m, c, 3, vb);
    }
    if (k == 3) {
        if (ncell <= 16000) return LaunchCfg{1, {4, 4, 2}};
        const LaunchCfg c[2] = {{1, {8, 4, 4}}, {1, {4, 4, 2}}};
        return first_fit(k, m, c, 2, vb);
    }
    if (ncell <= 8000) return LaunchCfg{1, {4, 3, 2}};
    const LaunchCfg c[4] = {f32 ? LaunchCfg{1, {6, 4, 2}} : LaunchCfg{1, {4, 4, 3}}, {1, {4, 3, 2}}, {1, {4, 2, 2}},
                            {1, {4, 4, 1}}};
    return first_fit(k, m, c, 4, vb);
}

// The same with the mass shift, where the configuration in use has no kernel with
// it.  PCG iteration, us: k = 2, 16^3 cells 16.9 with 8x4x4 against 18.9 with
// 16x8x4, 32^3 20.7 against 23.1, 40^3 27.5 against 27.1, 48^3 33.6 against 31.5;
// k = 3, 4x4x4 until 64^3 cells (8^3 19.2 against 21.8 with 8x4x4, 24^3 25.0 against
// 27.8, 48^3 83.4 against 86.5, 64^3 202 against 200).  k = 4 as without: its tiles
// have both kernels (32^3: 4x4x3 65.6 against 71.8 with 4x3x2).
inline LaunchCfg mass_default_config(int k, bool f32, const MeshArgs& m)
{
    const int64_t ncell = cell_count(m);
    if (k == 2) return ncell <= 40000 ? LaunchCfg{4, {8, 4, 4}} : LaunchCfg{4, {16, 8, 4}};
    if (k == 3) return ncell <= 200000 ? LaunchCfg{4, {4, 4, 4}} : LaunchCfg{4, {8, 4, 4}};
    const LaunchCfg c[3] = {default_config(k, f32, m), {1, {4, 3, 2}}, {1, {4, 2, 2}}};
    const int first = c[0].tile[2] == 1 ? 1 : 0;   // 4x4x1 has no kernel with the mass shift
    return first_fit(k, m, c + first, 3 - first, f32 ? 4 : 8);
}

// Configuration of the reinitialization operator: tiles (variant 1), or, where
// they do not address the mesh, one cell per thread into the cell-major scratch
// (variant 0, the whole mesh being one tile: no shared nodes).  Small tiles:
// seven turns per apply, so a workgroup's waves wait for one another often and
// other workgroups fill in (64^3 Q2, whole step: 8x4x2 14.0 ms, 8x4x4 16.3, 8x8x4
// 16.0; 20x17x15 Q3: 4x4x2 5.4, 4x4x4 5.8, 8x4x4 6.5; 24x25x23 Q4: 4x3x2 19.2,
// 4x4x3 19.6).  At k = 3 a large mesh takes 4x4x4 for its fewer shared nodes.
inline LaunchCfg reinit_config(int k, const MeshArgs& m)
{
    const LaunchCfg big{1, {4, 4, 4}};
    const LaunchCfg small = k == 2 ? LaunchCfg{1, {8, 4, 2}} : (k == 3 ? LaunchCfg{1, {4, 4, 2}} : LaunchCfg{1, {4, 3, 2}});
    if (k == 3 && cell_count(m) > 50000 && tiles_fit(k, m, big, 8)) return big;
    if (tiles_fit(k, m, small, 8)) return small;
    return LaunchCfg{0, {m.nc[0], m.nc[1], m.nc[2]}};
}

}  // namespace vpp
