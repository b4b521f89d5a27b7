// add_image's one pass over an image's levels against the plans' own functions, one by
// one: tiles and chunks of every tile configuration, the multi-level tile grids.
#include <cstdio>
#include <random>

#include "dwt2_batch_plan.h"

using namespace dwt2;

int main() {
    std::mt19937 rng(11);
    int bad = 0;
    for (int rep = 0; rep < 300; ++rep) {
        const int count = 1 + rng() % 6;
        int32_t h[6], w[6];
        int levels = 31;
        for (int i = 0; i < count; ++i) {
            const int bits = 2 + rng() % 29;
            h[i] = 2 + (int32_t)(rng() % ((1u << bits) - 1));
            w[i] = 2 + (int32_t)(rng() % ((1u << (2 + rng() % 29)) - 1));
            int n = 0;
            for (int32_t a = h[i], b = w[i]; a >= 2 && b >= 2; a = (a + 1) / 2, b = (b + 1) / 2) ++n;
            levels = n < levels ? n : levels;
        }
        levels = 1 + rng() % levels;
        for (int cfg = 0; cfg < kNumConfigs; ++cfg) {
            const KernelConfig c = kConfigs[cfg];
            if (c.algo != kAlgoTile) continue;
            BatchSums s{}, one{};
            uint64_t tiles = 0, chunks = 0, by_image = 0;
            for (int i = 0; i < count; ++i) {
                add_image(h[i], w[i], levels, c, true, &s);
                add_image(h[i], w[i], levels, c, false, &one);
                by_image += image_chunks(h[i], levels, core_rows(c));
            }
            for (int l = 0; l < levels; ++l) {
                BatchSums::Level v{};
                for (int i = 0; i < count; ++i) {
                    int32_t hl, wl, tx, ty;
                    level_size(h[i], w[i], l, &hl, &wl);
                    level_tiles(hl, wl, core_cols(c), core_rows(c), &tx, &ty);
                    v.tiles += (uint64_t)tx * (uint64_t)ty;
                    chunks += (uint64_t)chunk_count(ty);
                    if (l + 1 == levels) continue;
                    multi_tile_grid(hl, wl, 2, 32, &tx, &ty);
                    v.tiles32 += (uint64_t)tx * (uint64_t)ty;
                    v.rows32 += (uint64_t)ty;
                    v.cols112 += (uint64_t)tx * (uint64_t)hl;
                    v.cols128 += (uint64_t)(((wl + 1) / 2 + 127) / 128) * (uint64_t)hl;
                    v.samples += (uint64_t)hl * (uint64_t)wl;
                    v.tiles48 += launch_tile_count(h[i], w[i], l, 2, 48, 0, 0);
                    for (int k = 0; k < 2 && l + 3 == levels; ++k)
                        v.tiles3[k] += launch_tile_count(h[i], w[i], l, 3, 48 + 16 * k, 0, 0);
                }
                tiles += v.tiles;
                const BatchSums::Level& g = s.level[l];
                bad += g.tiles != v.tiles || g.tiles32 != v.tiles32 || g.rows32 != v.rows32 || g.cols112 != v.cols112 ||
                       g.cols128 != v.cols128 || g.samples != v.samples || g.tiles48 != v.tiles48 ||
                       g.tiles3[0] != v.tiles3[0] || g.tiles3[1] != v.tiles3[1];
                bad += one.level[l].tiles != v.tiles || one.level[l].tiles32 != 0;
            }
            bad += s.tiles != tiles || s.chunks != chunks || by_image != chunks || one.chunks != chunks;
        }
    }
    std::printf("bad %d\n", bad);
    return bad != 0;
}
