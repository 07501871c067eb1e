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

// Whether c runs the plane-per-thread kernel (plane_per_thread in apply_configs.h).
inline bool plane_variant(int k, const LaunchCfg& c) { return c.variant == 1 || (c.variant == 4 && k == 3); }

// Whether two configurations of degree k are the same kernel under two names.
inline bool same_kernel(int k, const LaunchCfg& a, const LaunchCfg& b)
{
    return a.tile[0] == b.tile[0] && a.tile[1] == b.tile[1] && a.tile[2] == b.tile[2] &&
           (a.variant == b.variant || (plane_variant(k, a) && plane_variant(k, b)));
}

// Threads of a workgroup of configuration c.
inline int tile_threads(int k, const LaunchCfg& c)
{
    const int cells = c.tile[0] * c.tile[1] * c.tile[2];
    if (plane_variant(k, c)) {   // PlaneGeo
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

inline int64_t cell_count(const MeshArgs& m) { return (int64_t)m.nc[0] * m.nc[1] * m.nc[2]; }

// Cells of the mesh's tiles, those past its upper faces included: a thread there
// runs the whole kernel on zeros.
inline int64_t padded_cells(MeshArgs m, const LaunchCfg& c)
{
    set_tiles(m, c);
    return tile_count64(m) * c.tile[0] * c.tile[1] * c.tile[2];
}

// Relative time of a slot of the padded mesh: at k = 4 the tiles that are not made
// of full waves cost more (2x150x150, 2x2x2 at half the slots of 4x4x3 56.1 us
// against 63.6; 90x90x4, 4x4x1 at 1.02 times the slots of 4x3x2 44.1 against 38.3).
inline int slot_cost(int k, const LaunchCfg& c)
{
    if (k != 4) return 100;
    return c.tile[0] == 2 ? 160 : (c.tile[2] == 1 ? 130 : 100);
}

// One of n configurations, preferred ones first: the first that fits the mesh,
// unless it fills the GPU (a tile per CU) and its slots cost a quarter more than a
// later one's.  Below a quarter the larger tile's fewer shared nodes win
// (43x37x29 Q3, FP64 / FP32 us: 8x4x4 26.2 / 19.5 at 1.17 times the slots of 4x4x2,
// 26.8 / 21.0), above it they do not (150x150x5 at 1.33 times 55.7 / 38.0 against
// 48.7 / 33.7, 400x400x1 at 2 times 116.5 / 76.1 against 72.8 / 47.6; Q4 200x200x2,
// 4x4x3 at 1.5 times 73.7 against 65.3 with 4x3x2).
inline LaunchCfg pick_config(int k, const MeshArgs& m, const LaunchCfg* c, int n, size_t value_bytes)
{
    auto cost = [&](int i) { return padded_cells(m, c[i]) * slot_cost(k, c[i]); };
    int best = -1;
    for (int i = 0; i < n; ++i) {
        if (!tiles_fit(k, m, c[i], value_bytes)) continue;
        if (best < 0) {
            best = i;
            continue;
        }
        MeshArgs t = m;
        set_tiles(t, c[best]);
        if (tile_count64(t) > 256 && 4 * cost(best) > 5 * cost(i)) best = i;
    }
    return c[best < 0 ? 0 : best];
}

// Kernel configuration of a new problem, by degree, precision and number of
// cells (vpp_tune measures instead).  Measured hot, one apply, us, FP64 / FP32:
//  k = 2: the plane kernel gives a small mesh three times the waves of the
//    cell-per-thread one, each with a third of the serial work (24^3 cells: 11.1
//    against 12.7 / 10.8 against 12.9); a mesh that fills the GPU prefers the
//    latter's fewer LDS accesses (32^3: 12.9 against 13.1 in FP64 but still 11.1
//    against 13.0 in FP32; 48^3: 17.9 against 22.5 / 14.9 against 16.6).
//  k = 3: small tiles until there are enough of them for every CU (20^3: 4x4x2
//    13.6 against 17.3 with 8x4x4; 24x88x8 16.5 against 17.8, with the sine ramp
//    24.7 against 29.1), then the fewer shared nodes of 8x4x4 (32^3: 19.7 against
//    20.5, 64^3: 80 against 88 / 52 against 56).  A CU holds one workgroup of
//    8x4x4 or the same 128 cells of smaller tiles: while the second round of 8x4x4
//    is less than two thirds full, 4x4x4 fills it better (with the sine ramp,
//    33x30x28: 44.8 / 23.3 with 8x4x4, 30.8 / 18.9 with 4x4x4; 32x36x32: 45.2 /
//    22.2 and 37.8 / 20.7; 36^3: 45.9 / 24.1 and 39.2 / 22.0; but 43x37x29, 1.9
//    rounds: 45.9 / 24.5 and 46.5 / 25.4), and a tile that needs one round only
//    does without it (33x26x34: 4x2x2 31.1, 4x4x4 38.0).
//  k = 4: the same, in multiples of the 12 cells of a wave (16^3: 4x3x2 16.1
//    against 17.6 with 4x4x3; 32^3: 35.4 against 38.9; in FP32 6x4x2 23.1
//    against 24.1 with 4x4x3).
// A thin box takes a tile that its extent fills better (pick_config); at k = 2 the
// plane kernel's per-slot cost, 1.25 times the other's, decides once both pad
// beyond twice the size (1x300x300 in FP64 / FP32: 70.6 / 42.1 against 57.0 / 32.0
// with 8x8x4; 1x1x2000, half the slots: 13.7 against 17.5), and FP32 takes 16x8x4
// up to 1.1 times the slots of 8x8x4 (64^3 18.2 against 20.1; 88^3 at 1.09 times 39.3
// against 39.8, 72^3 at 1.11 28.1 against 26.2, 40x80x80 at 1.2 23.3 against 19.7).
// A wide and shallow box whose lane offsets would pass 32 bits (2576 x 2576 x 4
// cells at k = 3, 2048 x 2048 x 3 at k = 4) takes a shallower tile.
inline LaunchCfg default_config(int k, bool f32, const MeshArgs& m)
{
    const size_t vb = f32 ? 4 : 8;
    const int64_t ncell = cell_count(m);
    if (k == 2) {
        const LaunchCfg plane{1, {8, 4, 2}}, slot{4, {8, 8, 4}};
        const int64_t size = f32 ? 50000 : 20000, pad = padded_cells(m, plane);
        if (ncell <= size && (pad <= 2 * size || 4 * padded_cells(m, slot) > 5 * pad)) return plane;
        const LaunchCfg wide{4, {16, 8, 4}};
        if (f32 && 10 * padded_cells(m, wide) <= 11 * padded_cells(m, slot) && tiles_fit(k, m, wide, vb)) return wide;
        return tiles_fit(k, m, slot, vb) ? slot : plane;
    }
    if (k == 3) {
        if (ncell <= 18000) return LaunchCfg{1, {4, 4, 2}};
        LaunchCfg c[3] = {{1, {8, 4, 4}}, {1, {4, 4, 2}}, {1, {4, 2, 2}}};
        const int64_t round = 256 * 8 * 4 * 4, wide = padded_cells(m, c[0]);
        if (wide > round && 3 * wide <= 5 * round) {
            c[0] = LaunchCfg{4, {4, 4, 4}};
            if (padded_cells(m, c[0]) > round)
                for (int i = 1; i < 3; ++i)
                    if (padded_cells(m, c[i]) <= round) return c[i];
        }
        return pick_config(k, m, c, 3, vb);
    }
    if (ncell <= 8000) {
        const LaunchCfg c[2] = {{1, {4, 3, 2}}, {1, {2, 2, 2}}};
        return pick_config(k, m, c, 2, vb);
    }
    const LaunchCfg c[4] = {f32 ? LaunchCfg{1, {6, 4, 2}} : LaunchCfg{1, {4, 4, 3}}, {1, {4, 3, 2}}, {1, {2, 2, 2}},
                            {1, {4, 4, 1}}};
    return pick_config(k, m, c, 4, vb);
}

// The same with the mass shift, where the configuration in use has no kernel with
// it.  PCG iteration, us: k = 2, 8x4x4 while its tiles are about one a CU (16^3
// cells 16.9 against 18.9 with 16x8x4, 32^3 19.6 against 22.0, 50x12x50 22.3 against
// 27.3), then 16x8x4 (33^3 24.4 and 23.7, 100x2x100 22.5 and 21.1, 48^3 33.6 and
// 31.5), except on a thin box that it pads a quarter more with several tiles a CU
// (1x190x190 43.1 against 74.1, 300x2x300 66.4 against 89.8, 24x90x90 52.2 against
// 62.9; 190x190x1, as many slots either way, 30.4 and 29.4);
// k = 3, 4x4x4 until 64^3 cells (8^3 19.2 against 21.8 with 8x4x4, 24^3 25.0 against
// 27.8, 48^3 83.4 against 86.5, 64^3 202 against 200).  k = 4 as without: its tiles
// have both kernels (32^3: 4x4x3 65.6 against 71.8 with 4x3x2).
inline LaunchCfg mass_default_config(int k, bool f32, const MeshArgs& m)
{
    const int64_t ncell = cell_count(m);
    if (k == 2) {
        const LaunchCfg small{4, {8, 4, 4}}, wide{4, {16, 8, 4}};
        const int64_t pad = padded_cells(m, small), wide_pad = padded_cells(m, wide);
        const bool thin = wide_pad > 256 * 16 * 8 * 4 && 4 * wide_pad > 5 * pad;
        return pad <= 300 * 8 * 4 * 4 || thin || !tiles_fit(k, m, wide, f32 ? 4 : 8) ? small : wide;
    }
    if (k == 3) return ncell <= 200000 ? LaunchCfg{4, {4, 4, 4}} : LaunchCfg{4, {8, 4, 4}};
    const LaunchCfg c[3] = {default_config(k, f32, m), {1, {4, 3, 2}}, {1, {4, 2, 2}}};
    const int first = c[0].tile[2] == 1 ? 1 : 0;   // 4x4x1 has no kernel with the mass shift
    return pick_config(k, m, c + first, 3 - first, f32 ? 4 : 8);
}

// Configuration of the reinitialization operator: tiles (variant 1), or one cell
// per thread into the cell-major scratch (variant 0, the whole mesh being one
// tile: no shared nodes) where they do not address the mesh or would mostly be
// padding.  Small tiles: seven turns per apply, so a workgroup's waves wait for
// one another often and other workgroups fill in (64^3 Q2, whole step: 8x4x2 14.0
// ms, 8x4x4 16.3, 8x8x4 16.0; 20x17x15 Q3: 4x4x2 5.4, 4x4x4 5.8, 8x4x4 6.5;
// 24x25x23 Q4: 4x3x2 19.2, 4x4x3 19.6).  At k = 3 a large mesh takes 4x4x4 for its
// fewer shared nodes (200x200x3 126 us an iteration against 142) unless it pads a
// quarter more (150x150x5 137 against 128, 400x400x1 332 against 232).
// Tiles or cells, us an iteration: k = 2, 300x300x1 52 against 64, 300x1x300 78
// against 63, 1x300x300 130 against 64, 300x2x300 89 against 90, 1x100x100 25
// against 38: a slot costs 3/4 of a cell, and the cell kernel some 15 us more to
// start with.  k = 3, 1x1x20000 155 against 142, 1x200x200 99 against 162; at k = 4
// the tiles are ahead everywhere (1x1x20000, 12 slots a cell: 329 against 415).
inline LaunchCfg reinit_config(int k, const MeshArgs& m)
{
    const LaunchCfg cells{0, {m.nc[0], m.nc[1], m.nc[2]}};
    const LaunchCfg small[3] = {{1, {8, 4, 2}}, {1, {4, 4, 2}}, {1, {4, 3, 2}}};
    const LaunchCfg c[2] = {{1, {4, 4, 4}}, small[k - 2]};
    const int first = k == 3 && cell_count(m) > 50000 ? 0 : 1;
    const LaunchCfg t = pick_config(k, m, c + first, 2 - first, 8);
    if (!tiles_fit(k, m, t, 8)) return cells;
    const int64_t n = cell_count(m), pad = padded_cells(m, t);
    if ((k == 2 && 3 * (pad - 120000) > 4 * n) || (k == 3 && pad - 150000 > 5 * n)) return cells;
    return t;
}

}  // namespace vpp
