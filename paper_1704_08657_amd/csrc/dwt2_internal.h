// Internal interface between the C ABI layer (dwt2_api.cpp) and the HIP
// kernels (the .hip files).  Not installed; not part of the public ABI.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include "dwt2.h"

namespace dwt2 {

enum Direction : int { kForward = 0, kInverse = 1, kAdjoint = 2 };
// kCdf53: the reversible integer CDF 5/3; kCdf53Real: the real-valued one
enum Wavelet : int { kCdf97 = 0, kCdf53 = 1, kCdf53Real = 2, kDd137 = 3 };
enum Dtype : int { kF32 = 0, kBF16 = 1, kF16 = 2, kI32 = 3 };
// Lifting scheme of a level: the fused non-separable steps, the fused steps
// with the P0/P1 split, the separable steps (the comparison scheme: every
// fused step replaced by its horizontal and its vertical step, a barrier
// each), or the fused steps evaluated as those two factors in registers (one
// barrier per fused step: the horizontal factor never leaves the wave).
// The LDS-plane kernel (kAlgoLds) also runs the non-separable
// polyconvolution: one step N_{P,U} per lifting pair.
enum Scheme : int { kSchemeFused = 0, kSchemeSplit = 1, kSchemeSeparable = 2, kSchemeFactored = 3,
                    kSchemePolyconv = 4 };

// Geometry shared by host planning and the kernels, in blocks of 2x2 pixels.
// A tile (kAlgoTile) has 64 * bpl output columns (bpl blocks per lane) and
// waves * rows - 2 * kHalo output rows; a halo of kHalo blocks on every side
// is recomputed and discarded.  A stream strip (kAlgoStream) has 124 output
// columns.
constexpr int kLanes = 64;
constexpr int kHalo = 2;
constexpr int kStreamCoreBX = 2 * kLanes - 2 * kHalo;     // stream kernel: 124 (halo in the edge lanes)

// Kernel configurations.
//  kAlgoTile:   one work-group = `waves` wave64s stacked vertically, one tile
//               of (64 * bpl) x (waves * rows) blocks held in VGPRs (`rows`
//               block rows and `bpl` block columns per lane, plus a halo
//               pair), one barrier per fused step.
//  kAlgoStream: every wave64 walks down its own column strip of 128 blocks,
//               `rows` block rows of loads in flight ahead of the computation;
//               `waves` strips per work-group; `seg` block rows per segment.
//  kAlgoLds:    the tile with its halo held as the four polyphase planes
//               in LDS (double-buffered), every step a 2-D stencil over them
//               with one barrier; `cx` x `cy` output blocks per work-group of
//               `waves` wave64s.  Runs any step program: fused, separable
//               and polyconvolution schemes, two-tap and four-tap filters.
enum Algo : int { kAlgoTile = 0, kAlgoStream = 1, kAlgoLds = 2 };
struct KernelConfig {
    int algo;
    int waves;
    int rows;
    int seg;
    int bpl;    // kAlgoTile: block columns per lane (2 or 4)
    int cx, cy; // kAlgoLds: output blocks of one work-group tile
};
constexpr KernelConfig kConfigs[] = {
    {kAlgoTile, 4, 4, 0, 2, 0, 0},    {kAlgoTile, 8, 4, 0, 2, 0, 0},    {kAlgoTile, 4, 4, 0, 4, 0, 0},
    {kAlgoTile, 4, 6, 0, 2, 0, 0},    {kAlgoTile, 8, 2, 0, 4, 0, 0},    {kAlgoStream, 4, 8, 64, 2, 0, 0},
    {kAlgoStream, 1, 8, 64, 2, 0, 0}, {kAlgoStream, 4, 8, 32, 2, 0, 0}, {kAlgoLds, 4, 0, 0, 0, 64, 16},
    {kAlgoLds, 4, 0, 0, 0, 32, 32}};
constexpr int kNumConfigs = 10;
constexpr int kDefaultConfig = 0;
constexpr int kLargeConfig = 3;       // levels of 2^25 samples and more
constexpr int kDefaultLdsConfig = 8;
// The four-tap register tile kernel (DD 13/7): a halo of kHalo4 block rows
// above and below a tile.
constexpr int kHalo4 = 3;
// Waves of its work-groups, and the block columns and rows of its taller tile.
constexpr int kWaves4 = 4, kCols4 = 120, kRows4 = 14;
// Tile kernels deal work over the 8 XCDs in chunks of about kRemapRows tile rows;
// the grid is a multiple of 8 chunks.
constexpr int kRemapRows = 2;
// How a list of tiles is dealt: work-groups go round-robin over the 8 XCDs, XCD x
// takes the chunks x, x + 8, ... of consecutive tiles, so that neighbours' halo
// re-reads hit its L2.  The chunk is about `near` tiles, the size that gives every
// XCD as many chunks: with chunks of exactly two tile rows some XCDs had one
// more than others, which a launch of few chunks waits for.  Up to 4096 tiles twice
// that, whose rows the caches hold all the same; up to 1024, which run at once, one
// chunk for each XCD.  Two levels, us, before and now: 8192^2 BF16 74.4 and 68.7, inverse
// 67.1 and 60.4; 4096^2 FP32 28.2 and 25.9, inverse 25.9 and 24.9; 3469 x 5197 adjoint
// 32.6 and 30.1; 8192^2 FP32 105.5 and 106.0; 60 uneven images of 64 ... 2048 152.8 and 146.2.
// A grid beyond `most` work-groups gives way to one chunk for each XCD, of fewer
// than 8 work-groups more than tiles.
struct Deal {
    int64_t chunk, grid;
};
inline Deal deal_tiles(int64_t tiles, int64_t near, int64_t most = 0x7fffffff) {
    if (tiles <= 4096) near *= 2;
    int64_t rounds = tiles > 1024 && tiles > 4 * near ? (tiles + 4 * near) / (8 * near) : 1;
    if (8 * rounds * ((tiles + 8 * rounds - 1) / (8 * rounds)) > most) rounds = 1;
    const int64_t chunk = (tiles + 8 * rounds - 1) / (8 * rounds);
    return {chunk, 8 * rounds * chunk};
}
// A launch is of fewer than 2^32 work-items: the work-groups of `waves` waves it
// may have, and the tiles it is then given (see deal_tiles).
constexpr int64_t max_groups(int waves) { return (((int64_t)1 << 32) - 1) / (waves * kLanes); }
constexpr int64_t max_tiles(int waves) { return max_groups(waves) - 7; }
constexpr int64_t kMaxTiles = max_tiles(1);
static_assert(max_groups(1) <= 0x7fffffff, "tile and work-group numbers fit 32 bits");
// The launches that cover `planes` planes of nt tiles each, as many planes in each
// as it may have: launch(first plane, planes, deal) for one after the other, up to an error.
template <typename F>
inline hipError_t for_each_launch(int64_t nt, int64_t near, int waves, int64_t planes, const F& launch) {
    if (nt < 1 || nt > max_tiles(waves)) return hipErrorInvalidConfiguration;
    const int64_t per = max_tiles(waves) / nt;
    for (int64_t p0 = 0; p0 < planes; p0 += per) {
        const int64_t n = planes - p0 < per ? planes - p0 : per;
        const hipError_t e = launch(p0, (int32_t)n, deal_tiles(nt * n, near, max_groups(waves)));
        if (e != hipSuccess) return e;
    }
    return hipSuccess;
}
// output block rows / columns of one tile (kAlgoTile, kAlgoLds)
constexpr int core_rows(KernelConfig c) { return c.algo == kAlgoLds ? c.cy : c.waves * c.rows - 2 * kHalo; }
constexpr int core_cols(KernelConfig c) { return c.algo == kAlgoLds ? c.cx : kLanes * c.bpl; }

// Whether a launch may have the tiles of one h x w plane on that kernel.  The
// LDS-plane kernel, whose tiles are 16 rows, takes the narrow images up to 2^29
// rows that are beyond.
inline bool taps4_fits(int32_t h, int32_t w) {
    return (int64_t)(((w + 1) / 2 + kCols4 - 1) / kCols4) * (((h + 1) / 2 + kRows4 - 1) / kRows4) <= max_tiles(kWaves4);
}

// One level of a transform.  Forward: `in` is the h x w image of this level,
// `out` the origin of this level's region of the Mallat pyramid (details are
// written there), `out_ll` receives the LL band.  Inverse / adjoint: `in` is
// the pyramid region (details), `in_ll` the LL band, `out` the h x w image.
struct LevelParams {
    const void* in;
    int64_t in_pitch;
    const void* in_ll;
    int64_t in_ll_pitch;
    void* out;
    int64_t out_pitch;
    void* out_ll;
    int64_t out_ll_pitch;
    int32_t h, w;
    int32_t tiles_x, tiles_y;
    int32_t seg_rows;  // kAlgoStream: block rows per segment
    // Plane batch: the launch covers `planes` planes; plane p's buffers
    // start p * (stride) elements after those of plane 0.  Set by the
    // launcher (the tile kernel deals the tiles of all planes as one list,
    // the streaming kernel takes one grid row per plane).
    int64_t in_ps, in_ll_ps, out_ps, out_ll_ps;
    int32_t planes;
    int32_t chunk;     // set by the launcher, see deal_tiles
    // CDF 9/7, a level whose output the call's next level reads (forward:
    // the LL band of every level but the last; inverse / adjoint: the image
    // of every level but the finest): interior tiles store it with ordinary
    // stores, so the next level finds it in the caches; every other store
    // stays nontemporal.  Read by the launcher, which picks the kernel
    // variant.
    int32_t ll_cached;
};

// Two or three consecutive levels in one launch.  Forward: `in` is the h x w
// image of the first level, `out` the pyramid (the details of every level go
// there), `ll` receives the last level's LL band.  Inverse / adjoint: `in` is the
// pyramid, `ll` the last level's LL band, `out` the h x w image.  *_ps: plane strides.
struct PairParams {
    const void* in;
    int64_t in_pitch, in_ps;
    void* out;
    int64_t out_pitch, out_ps;
    void* ll;
    int64_t ll_pitch, ll_ps;
    int32_t h, w;
    int32_t tiles_x, tiles_y;     // set by the launcher, as are planes and chunk
    int32_t planes;
    int32_t chunk;                // see deal_tiles
};

// Its tiles: NW * K block rows of the first level with a halo of kHalo2 above
// and below, 64 lanes of two block columns of which kEdge2 lanes on either side
// are halo.
constexpr int kHalo2 = 6;
constexpr int kEdge2 = 4;
constexpr int kPairCols = (kLanes - 2 * kEdge2) * 2;
inline int64_t pair_tiles(int32_t h, int32_t w, int32_t planes, int rows) {
    const int cy = rows - 2 * kHalo2;
    return (int64_t)(((w + 1) / 2 + kPairCols - 1) / kPairCols) * (((h + 1) / 2 + cy - 1) / cy) * planes;
}
// Tile shape, in block rows of a tile (32: 8 waves x 4 rows, 48: 8 x 6).  Few
// tiles, all on the chip at once (up to 2.5 work-groups of 8 waves on each of 256
// CUs): the shape that takes the least time from load to store, 8 waves x 4 rows
// (1024^2 FP32 forward 7.3 us, 8 x 6: 9.2).  Beyond, 8 x 6 recomputes 12 of 48 rows instead of 12 of 32, which counts where the
// vector units are the limit: 16-bit storage (3 x 8192^2 FP16 inverse 179 us,
// 8 x 4: 200) and one round of tiles (3 x 1081 x 1921 FP32 forward 13.2, 14.5);
// 8 x 4 has 60 registers to 82 and more work-groups on a CU, which counts where
// memory is: 4-byte samples forward (8192^2 106 us, 8 x 6: 115; 4096^2 28.3,
// 29.1) and, inverse and adjoint, from 2^25 samples (inverse 8192^2 103, 108; but
// 4096^2 27.3, 25.6).  Where the lower tiles are no more, the taller ones hold rows
// past the image only (65536 planes of 16^2 FP32, inverse 581 us, 8 x 6: 1069).
inline int pair_rows(Direction dir, size_t es, int64_t tiles32, int64_t tiles48, int64_t samples) {
    if (tiles32 <= 640 || tiles32 <= tiles48) return 32;
    if (es == 2) return 48;
    if (dir == kForward) return tiles48 <= 512 ? 48 : 32;
    return samples >= (1 << 25) ? 32 : 48;
}
// Whether two levels in one launch beat one launch each (both sides measured
// on MI355X, us; two launches first):
//   * a level whose tiles all run at once: always (1024^2 FP32 11.7 / 7.2,
//     inverse 11.6 / 8.0; 192 planes of 64^2 16.0 / 9.6);
//   * larger ones, when 112 columns a tile do not cost half as many tiles
//     again as the one-level kernel's 128 (8192^2 FP32 121 / 106, inverse
//     127 / 103; 3469 x 5197 41 / 33; but 192 planes of 256^2, two tiles for
//     one: 31.4 / 34);
//   * 16-bit storage, forward, up to 2^26 samples: beyond, the recomputed
//     halo costs what the LL band saves (3 x 8192^2 BF16 188 / 193,
//     3 x 4096^2 56 / 53, inverse 198 / 176).
// Never when one plane has more tiles than a launch may.
inline bool pair_pays(Direction dir, Dtype dt, int32_t h, int32_t w, int32_t planes) {
    if (pair_tiles(h, w, planes, 32) <= 640) return true;
    if (pair_tiles(h, w, 1, 32) > max_tiles(8)) return false;
    const int32_t nc = (w + 1) / 2;
    if (2 * ((nc + kPairCols - 1) / kPairCols) >= 3 * ((nc + 2 * kLanes - 1) / (2 * kLanes))) return false;
    return !(dir == kForward && (dt == kBF16 || dt == kF16) && (int64_t)h * w * planes > (1 << 26));
}
// Three levels: tiles of 12 or 16 waves x 4 block rows with a halo of kHalo3
// blocks on every side.
constexpr int kHalo3 = 16;
constexpr int kTripleK = 4;
constexpr int kTripleCols = 2 * kLanes - 2 * kHalo3;
inline int64_t triple_tiles(int32_t h, int32_t w, int32_t planes, int rows) {
    const int cy = rows - 2 * kHalo3;
    return (int64_t)(((w + 1) / 2 + kTripleCols - 1) / kTripleCols) * (((h + 1) / 2 + cy - 1) / cy) * planes;
}
// Block rows of the tiles that take the last three levels in one launch, 0 if
// two launches are faster.  48 (12 waves) while every tile has a CU to itself
// (1024^2 FP32 forward 9.6 us, 64 rows 11.4); then 64 (16 waves), which recompute
// half of a tile instead of two thirds (1500^2 11.9 us, 48 rows 13.9; two launches 14.4), as
// long as they too run alone, forward up to three on two CUs (192 planes of
// 128^2, 384 tiles, 16.7 us, two launches 20.4; 2200^2, 420 tiles, 22.0, 18.6;
// inverse of 1800^2, 290 tiles, 18.8, 17.5).
inline int triple_rows(Direction dir, int64_t tiles48, int64_t tiles64) {
    if (tiles48 <= 256) return 48;
    return tiles64 <= (dir == kForward ? 384 : 256) ? 64 : 0;
}
// Enqueue `levels` (2 or 3) levels with the wavelet's default scheme.
hipError_t launch_pair(Direction dir, Wavelet wav, Dtype dt, int levels, const PairParams& p, int planes,
                       hipStream_t stream);

// The same for DD 13/7 (forward and inverse, two levels): tiles of 48 block rows (8
// waves x 6) or 64 (16 x 4) with a halo of kHalo4x2 above and below and of
// kEdge4x2 lanes of two block columns on either side.
constexpr int kHalo4x2 = 10;
constexpr int kEdge4x2 = 5;
constexpr int kCols4x2 = 2 * (kLanes - 2 * kEdge4x2);
inline int64_t taps4_pair_tiles(int32_t h, int32_t w, int32_t planes, int rows) {
    const int cy = rows - 2 * kHalo4x2;
    return (int64_t)(((w + 1) / 2 + kCols4x2 - 1) / kCols4x2) * (((h + 1) / 2 + cy - 1) / cy) * planes;
}
// Block rows of the tiles that take two levels in one launch, 0 if a launch each is
// faster.  The recomputed halo, half of a tile, is arithmetic, which is what
// bounds the larger levels; where the tiles all run at once, two on a CU, it is hidden by
// what a launch takes from load to store.  us, one launch each / both in one:
// 2048^2, 370 tiles of 48 rows, FP32 16.9 / 14.5, inverse 16.6 / 15.1; 2400^2, 516,
// 18.4 / 19.7; 8192^2 126 / 140.  The taller tiles, of which two fit a CU with
// 16-bit storage only, pay forward: 2800^2 BF16, 416 tiles, 20.7 / 15.8 (inverse 2400^2
// 16.4 / 17.6); 3200^2, 555, 22.6 / 21.9; 3 x 2161 x 3841 40.8 / 37.7, inverse 37.1 / 38.4.
inline int taps4_pair_rows(Direction dir, size_t es, int32_t h, int32_t w, int32_t planes) {
    if (taps4_pair_tiles(h, w, planes, 48) <= 512) return 48;
    return dir == kForward && es == 2 && taps4_pair_tiles(h, w, planes, 64) <= 512 ? 64 : 0;
}
hipError_t launch_taps4_pair(Direction dir, Dtype dt, const PairParams& p, int planes, hipStream_t stream);

// Enqueue one level for `planes` planes (1 <= planes <= kMaxGridPlanes).
// Returns hipSuccess or the launch error.  `cfg` indexes kConfigs;
// tiles_x / tiles_y (and seg_rows) of `p` must follow it: for kAlgoTile the
// tile grid, for kAlgoStream the number of strip groups (ceil(strips /
// waves)) and of segments.
constexpr int kMaxGridPlanes = 65535;
// kSchemeSeparable and kSchemeFactored run on the tile configurations only.
hipError_t launch_level(Direction dir, Wavelet wav, Dtype dt, Scheme scheme, int cfg,
                        const LevelParams& p, int planes, hipStream_t stream);
// The LDS-plane kernel (kConfigs[cfg].algo == kAlgoLds): forward and inverse
// of the float wavelets, fused / separable / polyconvolution schemes.
hipError_t launch_lds(Direction dir, Wavelet wav, Dtype dt, Scheme scheme, int cfg, const LevelParams& p,
                      int planes, hipStream_t stream);
// DD 13/7, forward and inverse, on the four-tap register tile kernel; sets the
// tile grid itself.  The fused steps bit-identical to the LDS-plane kernel, or, for
// 16-bit storage, as their two factors.
hipError_t launch_taps4(Direction dir, Dtype dt, Scheme sch, const LevelParams& p, int planes, hipStream_t stream);

}  // namespace dwt2
