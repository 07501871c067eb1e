// Host-side check of the tile rules (tile_rules.h): every configuration that a
// rule picks addresses the mesh with 32-bit lane offsets, shown by walking the
// offsets the kernels form (compiled with hipcc, runs on the CPU only).
#include <algorithm>
#include <cmath>
#include <cstdio>
#include <random>

#include "../../paper_2401_07805_amd/csrc/tile_rules.h"

using namespace vpp;

static int fails = 0, checked = 0;

static MeshArgs mesh(int k, int cx, int cy, int cz)
{
    MeshArgs m{};
    const int nc[3] = {cx, cy, cz};
    for (int d = 0; d < 3; ++d) {
        m.nc[d] = nc[d];
        m.nn[d] = k * nc[d] + 1;
    }
    return m;
}

// The largest byte offset from the tile base over every lane of a full tile (the
// kernels' own expressions), with the cells past the mesh left out.
static unsigned long long largest_offset(int k, const MeshArgs& m, const LaunchCfg& c, int bytes)
{
    const unsigned long long nx = m.nn[0], nxy = nx * m.nn[1];
    unsigned long long worst = 0;
    for (int lz = 0; lz < c.tile[2] && lz < m.nc[2]; ++lz)
        for (int ly = 0; ly < c.tile[1] && ly < m.nc[1]; ++ly)
            for (int lx = 0; lx < c.tile[0] && lx < m.nc[0]; ++lx)
                for (int a = 0; a <= k; ++a) {   // plane of a plane-per-thread lane; pl[j] of a half-cell lane
                    const int px = c.variant == 2 ? 0 : a, pz = c.variant == 2 ? a : 0;
                    const unsigned long long o = (k * lx + px + nx * k * ly + nxy * (k * lz + pz)) * bytes;
                    worst = o > worst ? o : worst;
                }
    return worst;
}

static void expect(bool ok, const char* what, int k, const MeshArgs& m, const LaunchCfg& c)
{
    ++checked;
    if (ok) return;
    if (fails++ < 20)
        std::printf("%s: k=%d %dx%dx%d cells, variant %d tile %dx%dx%d\n", what, k, m.nc[0], m.nc[1], m.nc[2], c.variant,
                    c.tile[0], c.tile[1], c.tile[2]);
}

static bool reaches(int k, const MeshArgs& m, const LaunchCfg& c, int bytes)
{
    return largest_offset(k, m, c, bytes) < (1ull << 32);
}

// Thin boxes: a default's padded cells stay near those of the shallow tile a
// new problem of its degree could take (8x8x4, 4x4x2, 4x2x2) once the tiles fill
// the GPU; the reinitialization operator's cells stay near the mesh's.
static void check_padding(int k, const MeshArgs& m)
{
    const LaunchCfg ref = k == 2 ? LaunchCfg{4, {8, 8, 4}} : (k == 3 ? LaunchCfg{1, {4, 4, 2}} : LaunchCfg{1, {4, 2, 2}});
    for (int f32 = 0; f32 < 2; ++f32) {
        const LaunchCfg c = default_config(k, f32, m);
        MeshArgs t = m;
        set_tiles(t, c);
        if (!tiles_fit(k, m, ref, f32 ? 4 : 8) || tile_count64(t) <= 256) continue;
        // k = 4: 4x2x2 itself is not offered; 4x3x2 has up to 1.5 times its slots
        expect(padded_cells(m, c) <= (k == 4 ? 2.0 : 1.25) * padded_cells(m, ref), "padding", k, m, c);
    }
    const LaunchCfg r = reinit_config(k, m);
    if (r.variant == 1 && k < 4)
        expect(padded_cells(m, r) <= (k == 2 ? 4.0 / 3 : 5.0) * cell_count(m) + (k == 2 ? 120000 : 150000), "reinitialization padding", k, m, r);
}

static void check(int k, const MeshArgs& m)
{
    check_padding(k, m);
    for (int f32 = 0; f32 < 2; ++f32) {
        const int vb = f32 ? 4 : 8;
        const LaunchCfg c = default_config(k, f32, m), ms = mass_default_config(k, f32, m);
        // tiles_fit is exactly "every lane offset, partial index and thread count is in range"
        for (const LaunchCfg& t : {c, ms, LaunchCfg{2, {8, 4, 4}}}) {
            MeshArgs mt = m;
            set_tiles(mt, t);
            const bool in_range = reaches(k, m, t, vb) && 8 * shared_stride(mt) < (1ll << 32) &&
                                  tile_count64(mt) * tile_threads(k, t) < (1ll << 32);
            if (tiles_fit(k, m, t, vb)) expect(in_range, "taken out of range", k, m, t);
            if (k * (t.tile[0] + 1) * 8 < 65536 && in_range) {
                // refused only within the tile's own extent in x of the limit
                const unsigned long long o = largest_offset(k, m, t, vb);
                if (o + 8ull * k < (1ull << 32)) expect(tiles_fit(k, m, t, vb), "refused in range", k, m, t);
            }
        }
        // a mesh that the shallowest tile of its degree addresses gets a configuration that fits
        const LaunchCfg low = k == 2 ? LaunchCfg{1, {8, 4, 2}} : (k == 3 ? LaunchCfg{1, {4, 4, 2}} : LaunchCfg{1, {4, 4, 1}});
        if (tiles_fit(k, m, low, vb)) expect(tiles_fit(k, m, c, vb), "default does not fit", k, m, c);
    }
    const LaunchCfg r = reinit_config(k, m);
    if (r.variant == 1) expect(reaches(k, m, r, 8), "reinitialization tile out of range", k, m, r);
    else {
        MeshArgs t = m;
        set_tiles(t, r);
        expect(tile_count64(t) == 1 && shared_stride(t) == 0, "whole-mesh tile", k, m, r);
    }
}

int main()
{
    // boxes whose offsets pass 2^32 with deep tiles and stay below with shallow ones
    check(3, mesh(3, 2576, 2576, 4));
    check(4, mesh(4, 2048, 2048, 3));
    check(2, mesh(2, 4730, 4730, 4));
    expect(default_config(3, false, mesh(3, 2576, 2576, 4)).tile[2] == 2, "shallow tile", 3, mesh(3, 2576, 2576, 4),
           default_config(3, false, mesh(3, 2576, 2576, 4)));
    expect(default_config(3, true, mesh(3, 2576, 2576, 4)).tile[2] == 4, "FP32 stays deep", 3, mesh(3, 2576, 2576, 4),
           default_config(3, true, mesh(3, 2576, 2576, 4)));
    expect(!tiles_fit(3, mesh(3, 2576, 2576, 4), {1, {8, 4, 4}}, 8), "8x4x4 refused", 3, mesh(3, 2576, 2576, 4), {1, {8, 4, 4}});
    expect(!tiles_fit(4, mesh(4, 2048, 2048, 3), {1, {4, 4, 3}}, 8), "4x4x3 refused", 4, mesh(4, 2048, 2048, 3), {1, {4, 4, 3}});
    // mass shift at k = 2: by the tiles of 8x4x4, thin boxes by padding
    expect(mass_default_config(2, false, mesh(2, 32, 32, 32)).tile[0] == 8, "mass", 2, mesh(2, 32, 32, 32), mass_default_config(2, false, mesh(2, 32, 32, 32)));
    expect(mass_default_config(2, false, mesh(2, 48, 48, 48)).tile[0] == 16, "mass", 2, mesh(2, 48, 48, 48), mass_default_config(2, false, mesh(2, 48, 48, 48)));
    expect(mass_default_config(2, false, mesh(2, 190, 190, 1)).tile[0] == 16, "mass", 2, mesh(2, 190, 190, 1), mass_default_config(2, false, mesh(2, 190, 190, 1)));
    expect(mass_default_config(2, false, mesh(2, 1, 190, 190)).tile[0] == 8, "mass", 2, mesh(2, 1, 190, 190), mass_default_config(2, false, mesh(2, 1, 190, 190)));
    // one kernel under two names
    expect(same_kernel(3, {4, {8, 4, 4}}, {1, {8, 4, 4}}), "same kernel", 3, mesh(3, 1, 1, 1), {1, {8, 4, 4}});
    expect(!same_kernel(2, {4, {8, 4, 2}}, {1, {8, 4, 2}}), "not the same", 2, mesh(2, 1, 1, 1), {1, {8, 4, 2}});
    expect(!same_kernel(3, {2, {8, 4, 4}}, {1, {8, 4, 4}}), "not the same", 3, mesh(3, 1, 1, 1), {2, {8, 4, 4}});
    expect(!same_kernel(3, {1, {4, 4, 2}}, {1, {4, 4, 4}}), "not the same", 3, mesh(3, 1, 1, 1), {1, {4, 4, 4}});
    // thin boxes by their extent
    expect(default_config(3, false, mesh(3, 400, 400, 1)).tile[2] == 2, "thin z", 3, mesh(3, 400, 400, 1), default_config(3, false, mesh(3, 400, 400, 1)));
    expect(default_config(3, false, mesh(3, 1, 200, 200)).tile[0] == 4, "thin x", 3, mesh(3, 1, 200, 200), default_config(3, false, mesh(3, 1, 200, 200)));
    expect(default_config(2, true, mesh(2, 1, 300, 300)).tile[0] == 8, "thin x", 2, mesh(2, 1, 300, 300), default_config(2, true, mesh(2, 1, 300, 300)));
    // k = 3: 8x4x4 would leave CUs idle, in its only round or in the second
    for (int f32 = 0; f32 < 2; ++f32) {
        auto tile = [&](int x, int y, int z, LaunchCfg want) {
            const MeshArgs m = mesh(3, x, y, z);
            const LaunchCfg c = default_config(3, f32, m);
            expect(c.variant == want.variant && std::equal(c.tile, c.tile + 3, want.tile), "rounds", 3, m, c);
        };
        tile(24, 88, 8, {1, {4, 4, 2}});
        tile(32, 32, 32, {1, {8, 4, 4}});
        tile(33, 30, 28, {4, {4, 4, 4}});
        tile(40, 32, 28, {4, {4, 4, 4}});
        tile(36, 36, 36, {4, {4, 4, 4}});
        tile(33, 26, 34, {1, {4, 2, 2}});
        tile(43, 37, 29, {1, {8, 4, 4}});
    }
    expect(reinit_config(2, mesh(2, 1, 300, 300)).variant == 0, "cells", 2, mesh(2, 1, 300, 300), reinit_config(2, mesh(2, 1, 300, 300)));
    // the reinitialization operator where not even its shallow tiles reach
    expect(reinit_config(2, mesh(2, 8200, 8200, 3)).variant == 0, "cells", 2, mesh(2, 8200, 8200, 3), reinit_config(2, mesh(2, 8200, 8200, 3)));
    // random boxes up to 2^31 - 1 nodes, 2^20 - 1 per direction
    std::mt19937_64 g(7);
    for (int t = 0; t < 200000; ++t) {
        const int k = 2 + (int)(g() % 3);
        int nc[3];
        for (int d = 0; d < 3; ++d) {
            const double e = std::uniform_real_distribution<double>(0, 19.99)(g);
            nc[d] = (int)(g() % 3 == 0 ? 1 + g() % 12 : (unsigned long long)(std::pow(2.0, e) / k) + 1);
        }
        const MeshArgs m = mesh(k, nc[0], nc[1], nc[2]);
        if ((double)m.nn[0] * m.nn[1] * m.nn[2] > 2147483647.0) continue;
        check(k, m);
    }
    std::printf("%d checks, %d failures\n", checked, fails);
    return fails != 0;
}
