// C ABI of the 2-D lifting DWT library: argument checks, level planning,
// workspace layout and kernel dispatch.  Every check runs on the host before
// the first HIP call, so an invalid call enqueues nothing.
#include <hip/hip_runtime.h>

#include <stdint.h>
#include <string.h>

#include <algorithm>
#include <mutex>
#include <string>
#include <utility>
#include <vector>

#include "dwt2.h"
#include "dwt2_batch_plan.h"
#include "dwt2_internal.h"

static_assert(DWT2_NUM_KERNEL_CONFIGS == dwt2::kNumConfigs, "kernel configuration count in dwt2.h");

namespace {

thread_local std::string g_last_hip_error;

size_t elem_size(int dt) {
    switch (dt) {
        case DWT2_F32: return 4;
        case DWT2_BF16: return 2;
        case DWT2_F16: return 2;
        case DWT2_I32: return 4;
    }
    return 0;
}

constexpr int32_t kMaxSide = 1 << 30;
constexpr int64_t kWsAlign = 256;            // bytes; also the LL pitch granule

int64_t ws_pitch(int32_t w) {                // elements, multiple of 64
    return ((int64_t)w + 63) / 64 * 64;
}

struct Plan {
    int levels;
    int32_t h[32], w[32];                    // size transformed at each level
};

int max_levels(int32_t h, int32_t w) {
    if (h < 2 || w < 2) return 0;
    int n = 0;
    while (h >= 2 && w >= 2) {
        ++n;
        h = (h + 1) / 2;
        w = (w + 1) / 2;
    }
    return n;
}

void plan_levels(int32_t h, int32_t w, int levels, Plan* p) {
    p->levels = levels;
    for (int l = 0; l < levels; ++l) {
        p->h[l] = h;
        p->w[l] = w;
        h = (h + 1) / 2;
        w = (w + 1) / 2;
    }
}

// Two ping-pong buffers per plane for intermediate LL bands: buffer A is large
// enough for any (level 1's), buffer B for any but level 1's.  All planes' A
// buffers come first (plane stride a), then all B buffers (plane stride b); a and
// b are multiples of kWsAlign bytes.
struct WsLayout {
    size_t a, b;        // bytes of one plane's buffer A / B
    size_t off_b;       // offset of the B region
    size_t total;
};

WsLayout ws_layout(const Plan& p, size_t es, int32_t planes) {
    size_t a = 0, b = 0;
    for (int l = 0; l + 1 < p.levels; ++l) {  // LL of level l+1 (0-based l) is kept
        const int32_t he = (p.h[l] + 1) / 2, we = (p.w[l] + 1) / 2;
        const size_t sz = (size_t)he * (size_t)ws_pitch(we) * es;
        if (l % 2 == 0) a = a > sz ? a : sz; else b = b > sz ? b : sz;
    }
    WsLayout L;
    L.a = (a + kWsAlign - 1) / kWsAlign * kWsAlign;
    L.b = (b + kWsAlign - 1) / kWsAlign * kWsAlign;
    L.off_b = L.a * (size_t)planes;
    L.total = L.off_b + L.b * (size_t)planes;
    return L;
}

bool ranges_overlap(const void* a, size_t na, const void* b, size_t nb) {
    if (!na || !nb) return false;
    const uintptr_t x = (uintptr_t)a, y = (uintptr_t)b;
    return x < y + nb && y < x + na;
}

size_t span_bytes(int32_t h, int32_t w, int64_t pitch, size_t es) {
    return ((size_t)(h - 1) * (size_t)pitch + (size_t)w) * es;
}

// Bytes from the first to the last element of `planes` planes.
size_t planes_span_bytes(int32_t planes, int64_t plane_stride, int32_t h, int32_t w, int64_t pitch, size_t es) {
    return (size_t)(planes - 1) * (size_t)plane_stride * es + span_bytes(h, w, pitch, es);
}

// Every tile of a batched call runs in the same launch as the tiles of the
// other images, so no image's destination may overlap another image's
// destination or any image's source (sources may share memory: they are only
// read).  The destination spans are sorted by start; once they are known to
// be disjoint they are also sorted by end, so the only destination that can
// overlap a source [a, b) is the last one starting before b.
bool batch_spans_alias(const dwt2_image* imgs, int count, size_t es) {
    std::vector<std::pair<uintptr_t, uintptr_t>> dst((size_t)count);
    for (int i = 0; i < count; ++i) {
        const uintptr_t a = (uintptr_t)imgs[i].dst;
        dst[(size_t)i] = {a, a + span_bytes(imgs[i].height, imgs[i].width, imgs[i].dst_pitch, es)};
    }
    std::sort(dst.begin(), dst.end());
    for (size_t i = 1; i < dst.size(); ++i)
        if (dst[i].first < dst[i - 1].second) return true;
    for (int i = 0; i < count; ++i) {
        const uintptr_t a = (uintptr_t)imgs[i].src;
        const uintptr_t b = a + span_bytes(imgs[i].height, imgs[i].width, imgs[i].src_pitch, es);
        auto it = std::lower_bound(dst.begin(), dst.end(), std::make_pair(b, (uintptr_t)0));
        if (it != dst.begin() && std::prev(it)->second > a) return true;
    }
    return false;
}

// Kernel configuration selected by the flags (0 in the field = the default:
// the LDS-plane kernel for the polyconvolution, which only it runs, and for
// DD 13/7, where launch_planes() goes by the four-tap kernel first; the register
// tile kernel otherwise).
int config_of(unsigned flags, int wavelet) {
    const unsigned t = (flags & DWT2_FLAG_KERNEL_MASK) >> DWT2_FLAG_KERNEL_SHIFT;
    if (t != 0) return (int)t - 1;
    return (wavelet == DWT2_DD137 || (flags & DWT2_FLAG_POLYCONV)) ? dwt2::kDefaultLdsConfig : dwt2::kDefaultConfig;
}

// Lifting scheme of a call.  Without a scheme flag: the fused steps,
// evaluated directly (T_P, S_U) for 4-byte samples, and for BF16 / FP16
// storage on the tile configurations as their two 1-D factors in registers
// (the same steps and barriers, 8 instead of 11 operations per block and
// step): with half the bytes per pixel that kernel is bound by its
// arithmetic.  DWT2_FLAG_FUSED asks for the direct evaluation everywhere.
dwt2::Scheme scheme_of(unsigned flags, int dtype, int wavelet, bool adjoint) {
    if (flags & DWT2_FLAG_SPLIT) return dwt2::kSchemeSplit;
    if (flags & DWT2_FLAG_SEPARABLE) return dwt2::kSchemeSeparable;
    if (flags & DWT2_FLAG_FACTORED) return dwt2::kSchemeFactored;
    if (flags & DWT2_FLAG_POLYCONV) return dwt2::kSchemePolyconv;
    if (flags & DWT2_FLAG_FUSED) return dwt2::kSchemeFused;
    const bool half = dtype == DWT2_BF16 || dtype == DWT2_F16;
    if (half && !adjoint && (wavelet == DWT2_CDF97 || wavelet == DWT2_CDF53) &&
        dwt2::kConfigs[config_of(flags, wavelet)].algo == dwt2::kAlgoTile)
        return dwt2::kSchemeFactored;
    return dwt2::kSchemeFused;
}

// The persistent forward (DWT2_FLAG_PERSISTENT: every level in one launch)
// runs CDF 9/7 with the fused or split steps on the tile configurations, for
// plane stacks of at most kMaxPersistPlanes planes.
constexpr int32_t kMaxPersistPlanes = 65536;

bool persistent_ok(int wavelet, int dtype, unsigned flags, int32_t planes) {
    return wavelet == DWT2_CDF97 && dtype != DWT2_I32 && planes <= kMaxPersistPlanes &&
           !(flags & (DWT2_FLAG_SEPARABLE | DWT2_FLAG_POLYCONV)) &&
           dwt2::persist_config_supported(config_of(flags, wavelet));
}

// Workspace of a persistent call on `count` images (a plane stack when
// imgs == nullptr: `count` planes of h x w): the work tables and every
// image's LL bands.  The tables depend on the tile shape, so the size is the
// largest over the tile configurations.
size_t persist_bytes(const dwt2_image* imgs, int count, int32_t h, int32_t w, int levels, size_t es) {
    size_t tables = 0;
    for (int cfg = 0; cfg < dwt2::kNumConfigs; ++cfg) {
        if (!dwt2::persist_config_supported(cfg)) continue;
        bool seen = false;                       // tiles of the same height: the same chunks
        for (int k = 0; k < cfg; ++k)
            seen |= dwt2::persist_config_supported(k) &&
                    dwt2::core_rows(dwt2::kConfigs[k]) == dwt2::core_rows(dwt2::kConfigs[cfg]);
        if (seen) continue;
        uint64_t chunks = 0;
        for (int i = 0; i < (imgs ? count : 1); ++i) {
            const uint64_t c = dwt2::image_chunks(imgs ? imgs[i].height : h, levels,
                                                  dwt2::core_rows(dwt2::kConfigs[cfg]));
            chunks += imgs ? c : c * (uint64_t)count;
        }
        const size_t off = dwt2::batch_layout(count, levels, chunks).off_ll;
        tables = tables > off ? tables : off;
    }
    size_t ll = 0;
    if (imgs)
        for (int i = 0; i < count; ++i) ll += dwt2::image_ll_bytes(imgs[i].height, imgs[i].width, levels, es);
    else
        ll = (size_t)count * dwt2::image_ll_bytes(h, w, levels, es);
    return tables + ll;
}

int validate(const void* src, void* dst, int32_t planes, int64_t sps, int64_t dps, int32_t h, int32_t w,
             int64_t sp, int64_t dp, int dtype, int wavelet, int levels, int boundary, unsigned flags,
             const void* ws, size_t ws_bytes, bool adjoint, bool own_ws = false) {
    if (!src || !dst) return DWT2_E_NULL;
    if (planes < 1) return DWT2_E_COUNT;
    if (wavelet != DWT2_CDF97 && wavelet != DWT2_CDF53_REV && wavelet != DWT2_CDF53 && wavelet != DWT2_DD137)
        return DWT2_E_WAVELET;
    if (dtype != DWT2_F32 && dtype != DWT2_BF16 && dtype != DWT2_F16 && dtype != DWT2_I32)
        return DWT2_E_DTYPE;
    if ((wavelet == DWT2_CDF53_REV) != (dtype == DWT2_I32)) return DWT2_E_DTYPE;
    if (boundary != DWT2_SYMMETRIC_WHOLE) return DWT2_E_BOUNDARY;
    if (flags & ~(DWT2_FLAG_SPLIT | DWT2_FLAG_SEPARABLE | DWT2_FLAG_FACTORED | DWT2_FLAG_POLYCONV |
                  DWT2_FLAG_FUSED | DWT2_FLAG_PERSISTENT | DWT2_FLAG_KERNEL_MASK))
        return DWT2_E_FLAGS;
    if (((flags & DWT2_FLAG_KERNEL_MASK) >> DWT2_FLAG_KERNEL_SHIFT) > (unsigned)dwt2::kNumConfigs)
        return DWT2_E_FLAGS;
    if (adjoint && wavelet != DWT2_CDF97) return DWT2_E_WAVELET;
    if ((flags & DWT2_FLAG_SPLIT) && (wavelet == DWT2_CDF53_REV || adjoint)) return DWT2_E_FLAGS;
    // at most one scheme flag; the separable and factored schemes: forward /
    // inverse on tile configurations (the separable one also on LDS-plane
    // configurations); the polyconvolution: CDF 9/7 forward / inverse on
    // LDS-plane configurations
    const unsigned schemes =
        flags & (DWT2_FLAG_SPLIT | DWT2_FLAG_SEPARABLE | DWT2_FLAG_FACTORED | DWT2_FLAG_POLYCONV | DWT2_FLAG_FUSED);
    if (schemes & (schemes - 1)) return DWT2_E_FLAGS;
    const int algo = dwt2::kConfigs[config_of(flags, wavelet)].algo;
    if ((flags & (DWT2_FLAG_SEPARABLE | DWT2_FLAG_FACTORED)) && (adjoint || algo == dwt2::kAlgoStream))
        return DWT2_E_FLAGS;
    if ((flags & DWT2_FLAG_POLYCONV) && wavelet != DWT2_CDF97) return DWT2_E_FLAGS;
    if ((flags & DWT2_FLAG_PERSISTENT) && (adjoint || !persistent_ok(wavelet, dtype, flags, planes)))
        return DWT2_E_FLAGS;
    // the LDS-plane kernel: float wavelets, forward / inverse, fused, separable
    // and polyconvolution schemes; no other configuration runs DD 13/7 or the
    // polyconvolution
    if (algo == dwt2::kAlgoLds &&
        (adjoint || wavelet == DWT2_CDF53_REV || (flags & (DWT2_FLAG_SPLIT | DWT2_FLAG_FACTORED))))
        return DWT2_E_FLAGS;
    if (algo != dwt2::kAlgoLds && (wavelet == DWT2_DD137 || (flags & DWT2_FLAG_POLYCONV))) return DWT2_E_FLAGS;
    if (h < 2 || w < 2 || h > kMaxSide || w > kMaxSide) return DWT2_E_SHAPE;
    if (sp < w || dp < w) return DWT2_E_PITCH;
    // planes of one buffer must not overlap
    const int64_t plane_elems = (int64_t)(h - 1) * sp + w, plane_elems_d = (int64_t)(h - 1) * dp + w;
    if (planes > 1 && (sps < plane_elems || dps < plane_elems_d)) return DWT2_E_PITCH;
    if (levels < 1 || levels > max_levels(h, w)) return DWT2_E_LEVELS;
    size_t need = 0;
    dwt2_workspace_bytes_planes(h, w, levels, (dwt2_dtype)dtype, planes, &need);
    // own_ws: the workspace is the library's scratch array (checked by the caller)
    if (need > 0 && !own_ws && (!ws || ws_bytes < need)) return DWT2_E_WORKSPACE;
    const size_t es = elem_size(dtype);
    const size_t ns = planes_span_bytes(planes, sps, h, w, sp, es), nd = planes_span_bytes(planes, dps, h, w, dp, es);
    if (ranges_overlap(src, ns, dst, nd)) return DWT2_E_ALIAS;
    if (need > 0 && !own_ws && (ranges_overlap(ws, need, src, ns) || ranges_overlap(ws, need, dst, nd)))
        return DWT2_E_ALIAS;
    return DWT2_OK;
}

int report(hipError_t e) {
    if (e == hipSuccess) return DWT2_OK;
    g_last_hip_error = hipGetErrorString(e);
    return DWT2_E_HIP;
}

dwt2::Dtype to_dtype(int d) { return (dwt2::Dtype)d; }
dwt2::Wavelet to_wav(int w) {
    return w == DWT2_CDF97 ? dwt2::kCdf97 : w == DWT2_CDF53 ? dwt2::kCdf53Real : w == DWT2_DD137 ? dwt2::kDd137
                                                                                                  : dwt2::kCdf53;
}

// Work-group grid of one level for kernel configuration `cfg`.
void plan_grid(int cfg, dwt2::LevelParams* lp) {
    const dwt2::KernelConfig c = dwt2::kConfigs[cfg];
    const int32_t nEr = (lp->h + 1) / 2, nEc = (lp->w + 1) / 2;
    if (c.algo != dwt2::kAlgoStream) {
        const int cy = dwt2::core_rows(c);
        const int cx = dwt2::core_cols(c);
        lp->tiles_x = (nEc + cx - 1) / cx;
        lp->tiles_y = (nEr + cy - 1) / cy;
        lp->seg_rows = 0;
    } else {
        const int32_t strips = (nEc + dwt2::kStreamCoreBX - 1) / dwt2::kStreamCoreBX;
        lp->tiles_x = (strips + c.waves - 1) / c.waves;
        lp->tiles_y = (nEr + c.seg - 1) / c.seg;
        lp->seg_rows = c.seg;
    }
}

// Kernel configuration of one level: the one the call names, else the taller
// tile (4 waves x 6 rows: 8 halo rows of 48 image rows instead of 8 of 32) for
// levels of 2^25 samples and more, where the memory system is the limit
// (8192^2 FP32 forward 94.8 us, 4 x 4: 95.6, inverse 96.1 / 97.9; 3 x 8192^2
// BF16 148 / 158), and the shorter one below, where a tile's own time counts
// more (2048^2 9.2 / 8.5; 1024^2 6.9 / 5.9).
int level_config(unsigned flags, int wavelet, int32_t planes, int32_t h, int32_t w) {
    const int cfg = config_of(flags, wavelet);
    if (cfg != dwt2::kDefaultConfig || (flags & DWT2_FLAG_KERNEL_MASK)) return cfg;
    return (int64_t)planes * h * w >= (1 << 25) ? dwt2::kLargeConfig : cfg;
}

// Launch one level for every plane, in grid chunks of at most
// kMaxGridPlanes planes.
int launch_planes(dwt2::Direction dir, int wavelet, int dtype, unsigned flags, int cfg, dwt2::LevelParams lp,
                  int32_t planes, size_t es, hipStream_t s) {
    for (int32_t p0 = 0; p0 < planes; p0 += dwt2::kMaxGridPlanes) {
        const int32_t n = planes - p0 < dwt2::kMaxGridPlanes ? planes - p0 : dwt2::kMaxGridPlanes;
        dwt2::LevelParams q = lp;
        if (p0 > 0) {
            q.in = lp.in ? (const char*)lp.in + (size_t)p0 * (size_t)lp.in_ps * es : nullptr;
            q.in_ll = lp.in_ll ? (const char*)lp.in_ll + (size_t)p0 * (size_t)lp.in_ll_ps * es : nullptr;
            q.out = lp.out ? (char*)lp.out + (size_t)p0 * (size_t)lp.out_ps * es : nullptr;
            q.out_ll = lp.out_ll ? (char*)lp.out_ll + (size_t)p0 * (size_t)lp.out_ll_ps * es : nullptr;
        }
        // DD 13/7 without a named configuration or scheme (or with the fused
        // one), unless its tiles are too many: the four-tap register tile kernel, whose steps are fused for FP32
        // (memory-bound) and factored for 16-bit storage (bound by its arithmetic)
        const bool taps4 = wavelet == DWT2_DD137 && !(flags & ~DWT2_FLAG_FUSED) && dwt2::taps4_fits(lp.h, lp.w);
        const dwt2::Scheme sch4 = flags || dtype == DWT2_F32 ? dwt2::kSchemeFused : dwt2::kSchemeFactored;
        const int rc = taps4 ? report(dwt2::launch_taps4(dir, to_dtype(dtype), sch4, q, n, s))
                             : report(dwt2::launch_level(dir, to_wav(wavelet), to_dtype(dtype),
                                                 scheme_of(flags, dtype, wavelet, dir == dwt2::kAdjoint),
                                                 cfg, q, n, s));
        if (rc) return rc;
    }
    return DWT2_OK;
}

// Whether a level stores the output the next level of the call reads with
// ordinary stores (LevelParams::ll_cached).  It pays from 32 MiB (5 inverse
// levels of 8192^2 FP32: 147.6 us, 151.3 without; smaller outputs stay in the
// Infinity Cache either way) to 128 MiB (16384^2, 2 levels inverse, 256 MiB: 489
// us, 478 without).  A forward LL band of 4-byte samples does not gain
// (5 levels of 8192^2 154.3 with, 151.5 without; 3 planes, 3 levels, 379 and
// 359), one of 16-bit samples does (3 x 8192^2 BF16, 5 levels, 202 and 208).
bool cached_output(dwt2::Direction dir, int32_t planes, int32_t h, int32_t w, size_t es) {
    const uint64_t n = (uint64_t)planes * (uint64_t)h * (uint64_t)w * es;
    return (dir != dwt2::kForward || es == 2) && n >= ((uint64_t)32 << 20) && n <= ((uint64_t)128 << 20);
}

// Levels the launch that starts at level l takes, in a call that names no
// scheme and no kernel configuration: the last three while their tiles all run
// at once (triple_rows), else two where that is the faster way (pair_pays).
int levels_in_launch(dwt2::Direction dir, const Plan& p, int l, int dtype, int wavelet, unsigned flags,
                     int32_t planes) {
    if (flags != 0 || l + 1 >= p.levels) return 1;
    if (wavelet == DWT2_DD137)
        return dwt2::taps4_pair_rows(dir, elem_size(dtype), p.h[l], p.w[l], planes) > 0 ? 2 : 1;
    if (l + 3 == p.levels && dwt2::triple_rows(dir, dwt2::triple_tiles(p.h[l], p.w[l], planes, 48),
                                               dwt2::triple_tiles(p.h[l], p.w[l], planes, 64)) > 0)
        return 3;
    return dwt2::pair_pays(dir, to_dtype(dtype), p.h[l], p.w[l], planes) ? 2 : 1;
}

// Two levels in one launch for a whole batch: the same choice as for a stack of planes
// (levels_in_launch), on the sums over the images.
bool batch_pair_pays(int dtype, const dwt2::BatchSums::Level& st) {
    if (st.tiles32 <= 640) return true;
    if (st.tiles32 > (uint64_t)dwt2::max_tiles(8)) return false;    // more than a launch may have
    if (2 * st.cols112 >= 3 * st.cols128) return false;
    return !(dtype != DWT2_F32 && st.samples > (1 << 26));
}

// Forward: level l reads the LL of level l-1 (src for l = 0) and writes its
// details into dst at the level's region origin (dst itself: every level's
// region starts at (0, 0)), its LL into the workspace or, for the last level,
// into dst.
int run_forward(const void* src, void* dst, int32_t planes, int64_t sps, int64_t dps, int32_t h, int32_t w,
                int64_t sp, int64_t dp, int dtype, int wavelet, int levels, unsigned flags, void* ws,
                hipStream_t s) {
    // one level is one launch either way (and needs no workspace)
    if ((flags & DWT2_FLAG_PERSISTENT) && levels > 1) {
        // without a named configuration the taller tile beyond 2^22 samples (8192^2
        // FP32, 5 levels, 455 us, the lower one 483; 3 x 4096^2 285, 319; but 2048^2 175, 162)
        const bool named = flags & DWT2_FLAG_KERNEL_MASK;
        const int cfg = !named && (int64_t)planes * h * w > (1 << 22) ? dwt2::kLargeConfig : config_of(flags, wavelet);
        dwt2::BatchSums sums{};
        dwt2::add_image(h, w, levels, dwt2::kConfigs[cfg], false, &sums);
        const dwt2::ImageSet S{nullptr, src, dst, sps, dps, sp, dp, h, w};
        const dwt2::BatchLayout L = dwt2::batch_layout(planes, levels, sums.chunks * (uint64_t)planes);
        return report(dwt2::launch_fwd_persistent(to_dtype(dtype), scheme_of(flags, dtype, wavelet, false), cfg, S,
                                                  planes, levels, ws, L, sums.tiles * (uint64_t)planes, s));
    }
    Plan p;
    plan_levels(h, w, levels, &p);
    const size_t es = elem_size(dtype);
    const WsLayout L = ws_layout(p, es, planes);
    char* bufs[2] = {(char*)ws, (char*)ws + L.off_b};
    const int64_t buf_ps[2] = {(int64_t)(L.a / es), (int64_t)(L.b / es)};
    const void* in = src;
    int64_t in_pitch = sp, in_ps = sps;
    int cur = 1;                              // the buffer that holds `in` (none before the first level)
    for (int l = 0; l < levels; ++l) {
        const int n = levels_in_launch(dwt2::kForward, p, l, dtype, wavelet, flags, planes);
        const bool last = l + n == levels;
        // the LL band that leaves this launch: dst, or the buffer the input is
        // not in (A, which holds any band, before B, which holds all but the first)
        cur ^= 1;
        void* const out_ll = last ? dst : (void*)bufs[cur];
        const int64_t out_ll_pitch = last ? dp : ws_pitch((p.w[l + n - 1] + 1) / 2);
        const int64_t out_ll_ps = last ? dps : buf_ps[cur];
        if (n > 1) {
            dwt2::PairParams pp{};
            pp.in = in;
            pp.in_pitch = in_pitch;
            pp.in_ps = in_ps;
            pp.out = dst;
            pp.out_pitch = dp;
            pp.out_ps = dps;
            pp.ll = out_ll;
            pp.ll_pitch = out_ll_pitch;
            pp.ll_ps = out_ll_ps;
            pp.h = p.h[l];
            pp.w = p.w[l];
            const int rc = report(dwt2::launch_pair(dwt2::kForward, to_wav(wavelet), to_dtype(dtype), n, pp, planes, s));
            if (rc) return rc;
            in = out_ll;
            in_pitch = out_ll_pitch;
            in_ps = out_ll_ps;
            l += n - 1;
            continue;
        }
        dwt2::LevelParams lp{};
        lp.h = p.h[l];
        lp.w = p.w[l];
        lp.in = in;
        lp.in_pitch = in_pitch;
        lp.in_ps = in_ps;
        lp.out = dst;
        lp.out_pitch = dp;
        lp.out_ps = dps;
        lp.ll_cached = !last && cached_output(dwt2::kForward, planes, (lp.h + 1) / 2, (lp.w + 1) / 2, es) ? 1 : 0;
        lp.out_ll = out_ll;
        lp.out_ll_pitch = out_ll_pitch;
        lp.out_ll_ps = out_ll_ps;
        const int cfg = level_config(flags, wavelet, planes, lp.h, lp.w);
        plan_grid(cfg, &lp);
        const int rc = launch_planes(dwt2::kForward, wavelet, dtype, flags, cfg, lp, planes, es, s);
        if (rc) return rc;
        in = lp.out_ll;
        in_pitch = lp.out_ll_pitch;
        in_ps = lp.out_ll_ps;
    }
    return DWT2_OK;
}

// Inverse / adjoint: coarsest level first.  Level l reads its LL (src for the
// coarsest level, else the workspace written by level l+1) and its details
// from src, and writes its image into the workspace or, for l = 0, into dst.
int run_backward(dwt2::Direction dir, const void* src, void* dst, int32_t planes, int64_t sps, int64_t dps,
                 int32_t h, int32_t w, int64_t sp, int64_t dp, int dtype, int wavelet, int levels,
                 unsigned flags, void* ws, hipStream_t s) {
    Plan p;
    plan_levels(h, w, levels, &p);
    const size_t es = elem_size(dtype);
    const WsLayout L = ws_layout(p, es, planes);
    char* bufs[2] = {(char*)ws, (char*)ws + L.off_b};
    const int64_t buf_ps[2] = {(int64_t)(L.a / es), (int64_t)(L.b / es)};
    const void* ll = src;
    int64_t ll_pitch = sp, ll_ps = sps;
    // the launches, finest level first; their images, which the next launch
    // reads as its LL band, alternate between the buffers so that the largest
    // (the finest launch's input) lies in A
    int first[32], count = 0;
    for (int l = 0; l < levels; l += levels_in_launch(dir, p, l, dtype, wavelet, flags, planes)) first[count++] = l;
    for (int j = count - 1; j >= 0; --j) {
        const int l = first[j], n = (j + 1 < count ? first[j + 1] : levels) - l;
        const int buf = (j - 1) & 1;
        void* const out = l == 0 ? dst : (void*)bufs[buf];
        const int64_t out_pitch = l == 0 ? dp : ws_pitch(p.w[l]);
        const int64_t out_ps = l == 0 ? dps : buf_ps[buf];
        if (n > 1) {
            dwt2::PairParams pp{};
            pp.in = src;
            pp.in_pitch = sp;
            pp.in_ps = sps;
            pp.out = out;
            pp.out_pitch = out_pitch;
            pp.out_ps = out_ps;
            pp.ll = const_cast<void*>(ll);         // read only
            pp.ll_pitch = ll_pitch;
            pp.ll_ps = ll_ps;
            pp.h = p.h[l];
            pp.w = p.w[l];
            const int rc = report(dwt2::launch_pair(dir, to_wav(wavelet), to_dtype(dtype), n, pp, planes, s));
            if (rc) return rc;
            ll = out;
            ll_pitch = out_pitch;
            ll_ps = out_ps;
            continue;
        }
        dwt2::LevelParams lp{};
        lp.h = p.h[l];
        lp.w = p.w[l];
        lp.in = src;
        lp.in_pitch = sp;
        lp.in_ps = sps;
        lp.in_ll = ll;
        lp.in_ll_pitch = ll_pitch;
        lp.in_ll_ps = ll_ps;
        // the image of level l is the LL of level l-1
        lp.ll_cached = l > 0 && cached_output(dir, planes, p.h[l], p.w[l], es) ? 1 : 0;
        lp.out = out;
        lp.out_pitch = out_pitch;
        lp.out_ps = out_ps;
        const int cfg = level_config(flags, wavelet, planes, lp.h, lp.w);
        plan_grid(cfg, &lp);
        const int rc = launch_planes(dir, wavelet, dtype, flags, cfg, lp, planes, es, s);
        if (rc) return rc;
        ll = lp.out;
        ll_pitch = lp.out_pitch;
        ll_ps = lp.out_ps;
    }
    return DWT2_OK;
}

// Workspace of dwt2_fwd_noalloc: one fixed array per GPU (the code object
// holds it on every device it is loaded on, until the process ends).  Host
// code must not pass `scratch` itself to a kernel or a copy: in host code the
// name is a host-side stand-in, not the device address.  The device address
// is looked up once per device (hipGetSymbolAddress with that device
// current) and kept in g_scratch_ptr.
static __device__ __align__(256) unsigned char scratch[DWT2_SCRATCH_BYTES];

constexpr int kMaxDevices = 64;
std::mutex g_scratch_mu;
void* g_scratch_ptr[kMaxDevices];

int scratch_address(void** out) {
    int dev = 0;
    hipError_t e = hipGetDevice(&dev);
    if (e != hipSuccess) return report(e);
    if (dev < 0 || dev >= kMaxDevices) return report(hipErrorInvalidDevice);
    std::lock_guard<std::mutex> lock(g_scratch_mu);
    if (!g_scratch_ptr[dev]) {
        void* p = nullptr;
        e = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch));
        if (e != hipSuccess) return report(e);
        if (!p) return report(hipErrorInvalidSymbol);
        g_scratch_ptr[dev] = p;
    }
    *out = g_scratch_ptr[dev];
    return DWT2_OK;
}

}  // namespace

extern "C" {

int dwt2_max_levels(int32_t height, int32_t width) { return max_levels(height, width); }

int dwt2_workspace_bytes_planes(int32_t height, int32_t width, int levels, dwt2_dtype dtype, int32_t planes,
                                size_t* bytes) {
    if (!bytes) return DWT2_E_NULL;
    *bytes = 0;
    const size_t es = elem_size(dtype);
    if (!es) return DWT2_E_DTYPE;
    if (planes < 1) return DWT2_E_COUNT;
    if (height < 2 || width < 2 || height > kMaxSide || width > kMaxSide) return DWT2_E_SHAPE;
    if (levels < 1 || levels > max_levels(height, width)) return DWT2_E_LEVELS;
    Plan p;
    plan_levels(height, width, levels, &p);
    size_t n = ws_layout(p, es, planes).total;
    // a float multi-level forward may take the persistent path
    if (levels > 1 && dtype != DWT2_I32 && planes <= kMaxPersistPlanes) {
        const size_t q = persist_bytes(nullptr, planes, height, width, levels, es);
        n = n > q ? n : q;
    }
    *bytes = n;
    return DWT2_OK;
}

int dwt2_workspace_bytes(int32_t height, int32_t width, int levels, dwt2_dtype dtype, size_t* bytes) {
    return dwt2_workspace_bytes_planes(height, width, levels, dtype, 1, bytes);
}

int dwt2_fwd_planes(const void* src, void* dst, int32_t planes, int64_t src_plane_stride, int64_t dst_plane_stride,
                    int32_t height, int32_t width, int64_t src_pitch, int64_t dst_pitch, dwt2_dtype dtype,
                    dwt2_wavelet wavelet, int levels, dwt2_boundary boundary, unsigned flags, void* workspace,
                    size_t workspace_bytes, void* stream) {
    const int rc = validate(src, dst, planes, src_plane_stride, dst_plane_stride, height, width, src_pitch,
                            dst_pitch, dtype, wavelet, levels, boundary, flags, workspace, workspace_bytes, false);
    if (rc) return rc;
    return run_forward(src, dst, planes, src_plane_stride, dst_plane_stride, height, width, src_pitch, dst_pitch,
                       dtype, wavelet, levels, flags, workspace, (hipStream_t)stream);
}

int dwt2_inv_planes(const void* src, void* dst, int32_t planes, int64_t src_plane_stride, int64_t dst_plane_stride,
                    int32_t height, int32_t width, int64_t src_pitch, int64_t dst_pitch, dwt2_dtype dtype,
                    dwt2_wavelet wavelet, int levels, dwt2_boundary boundary, unsigned flags, void* workspace,
                    size_t workspace_bytes, void* stream) {
    if (flags & DWT2_FLAG_PERSISTENT) return DWT2_E_FLAGS;   // a forward-only path
    const int rc = validate(src, dst, planes, src_plane_stride, dst_plane_stride, height, width, src_pitch,
                            dst_pitch, dtype, wavelet, levels, boundary, flags, workspace, workspace_bytes, false);
    if (rc) return rc;
    return run_backward(dwt2::kInverse, src, dst, planes, src_plane_stride, dst_plane_stride, height, width,
                        src_pitch, dst_pitch, dtype, wavelet, levels, flags, workspace, (hipStream_t)stream);
}

int dwt2_adj_planes(const void* src, void* dst, int32_t planes, int64_t src_plane_stride, int64_t dst_plane_stride,
                    int32_t height, int32_t width, int64_t src_pitch, int64_t dst_pitch, dwt2_dtype dtype,
                    dwt2_wavelet wavelet, int levels, dwt2_boundary boundary, unsigned flags, void* workspace,
                    size_t workspace_bytes, void* stream) {
    const int rc = validate(src, dst, planes, src_plane_stride, dst_plane_stride, height, width, src_pitch,
                            dst_pitch, dtype, wavelet, levels, boundary, flags, workspace, workspace_bytes, true);
    if (rc) return rc;
    return run_backward(dwt2::kAdjoint, src, dst, planes, src_plane_stride, dst_plane_stride, height, width,
                        src_pitch, dst_pitch, dtype, wavelet, levels, flags, workspace, (hipStream_t)stream);
}

int dwt2_fwd(const void* src, void* dst, int32_t height, int32_t width, int64_t src_pitch,
             int64_t dst_pitch, dwt2_dtype dtype, dwt2_wavelet wavelet, int levels,
             dwt2_boundary boundary, unsigned flags, void* workspace, size_t workspace_bytes,
             void* stream) {
    return dwt2_fwd_planes(src, dst, 1, 0, 0, height, width, src_pitch, dst_pitch, dtype, wavelet, levels, boundary,
                           flags, workspace, workspace_bytes, stream);
}

int dwt2_inv(const void* src, void* dst, int32_t height, int32_t width, int64_t src_pitch,
             int64_t dst_pitch, dwt2_dtype dtype, dwt2_wavelet wavelet, int levels,
             dwt2_boundary boundary, unsigned flags, void* workspace, size_t workspace_bytes,
             void* stream) {
    return dwt2_inv_planes(src, dst, 1, 0, 0, height, width, src_pitch, dst_pitch, dtype, wavelet, levels, boundary,
                           flags, workspace, workspace_bytes, stream);
}

int dwt2_adj(const void* src, void* dst, int32_t height, int32_t width, int64_t src_pitch,
             int64_t dst_pitch, dwt2_dtype dtype, dwt2_wavelet wavelet, int levels,
             dwt2_boundary boundary, unsigned flags, void* workspace, size_t workspace_bytes,
             void* stream) {
    return dwt2_adj_planes(src, dst, 1, 0, 0, height, width, src_pitch, dst_pitch, dtype, wavelet, levels, boundary,
                           flags, workspace, workspace_bytes, stream);
}

int dwt2_fwd_noalloc(const void* src, void* dst, int32_t height, int32_t width, int64_t src_pitch,
                     int64_t dst_pitch, dwt2_dtype dtype, dwt2_wavelet wavelet, int levels,
                     dwt2_boundary boundary, unsigned flags, void* stream) {
    int rc = validate(src, dst, 1, 0, 0, height, width, src_pitch, dst_pitch, dtype, wavelet, levels, boundary,
                      flags, nullptr, 0, false, /*own_ws=*/true);
    if (rc) return rc;
    size_t need = 0;
    rc = dwt2_workspace_bytes(height, width, levels, dtype, &need);
    if (rc) return rc;
    if (need > DWT2_SCRATCH_BYTES) return DWT2_E_SCRATCH;
    void* ws = nullptr;
    if (need > 0) {                 // one level needs no workspace
        rc = scratch_address(&ws);
        if (rc) return rc;
    }
    return run_forward(src, dst, 1, 0, 0, height, width, src_pitch, dst_pitch, dtype, wavelet, levels, flags, ws,
                       (hipStream_t)stream);
}

int dwt2_kernel_config(int index, int* algorithm, int* waves, int* rows, int* core_cols, int* core_rows) {
    if (index < 0 || index >= dwt2::kNumConfigs) return DWT2_E_FLAGS;
    const dwt2::KernelConfig c = dwt2::kConfigs[index];
    if (algorithm) *algorithm = c.algo;
    if (waves) *waves = c.waves;
    if (rows) *rows = c.rows;
    if (core_cols) *core_cols = c.algo != dwt2::kAlgoStream ? dwt2::core_cols(c) : dwt2::kStreamCoreBX;
    if (core_rows) *core_rows = c.algo != dwt2::kAlgoStream ? dwt2::core_rows(c) : c.seg;
    return DWT2_OK;
}

int dwt2_workspace_bytes_batched(const dwt2_image* images, int count, dwt2_dtype dtype, int levels,
                                 size_t* bytes) {
    if (!bytes || !images) return DWT2_E_NULL;
    *bytes = 0;
    if (count < 1) return DWT2_E_COUNT;
    const size_t es = elem_size(dtype);
    if (!es) return DWT2_E_DTYPE;
    for (int i = 0; i < count; ++i) {
        const dwt2_image& im = images[i];
        if (im.height < 2 || im.width < 2 || im.height > kMaxSide || im.width > kMaxSide) return DWT2_E_SHAPE;
        if (levels < 1 || levels > max_levels(im.height, im.width)) return DWT2_E_LEVELS;
    }
    // one launch per level, two or three: tile tables and ping-pong LL buffers; the
    // persistent launch: work tables and one LL band per level
    const dwt2::LevelBatchLayout L = dwt2::level_batch_layout(count, levels);
    size_t n = L.off_ll;
    for (int i = 0; i < count; ++i) n += dwt2::pingpong_ll_bytes(images[i].height, images[i].width, levels, es);
    const size_t q = persist_bytes(images, count, 0, 0, levels, es);
    *bytes = n > q ? n : q;
    return DWT2_OK;
}

int dwt2_fwd_batched(const dwt2_image* host_images, const dwt2_image* device_images, int count,
                     dwt2_dtype dtype, dwt2_wavelet wavelet, int levels, dwt2_boundary boundary,
                     unsigned flags, void* workspace, size_t workspace_bytes, void* stream) {
    if (!host_images || !device_images || !workspace) return DWT2_E_NULL;
    if (count < 1) return DWT2_E_COUNT;
    if (wavelet != DWT2_CDF97) return DWT2_E_WAVELET;        // batched path: CDF 9/7
    if (dtype != DWT2_F32 && dtype != DWT2_BF16 && dtype != DWT2_F16) return DWT2_E_DTYPE;
    if (boundary != DWT2_SYMMETRIC_WHOLE) return DWT2_E_BOUNDARY;
    if (flags & ~(DWT2_FLAG_SPLIT | DWT2_FLAG_FACTORED | DWT2_FLAG_FUSED | DWT2_FLAG_PERSISTENT |
                  DWT2_FLAG_KERNEL_MASK))
        return DWT2_E_FLAGS;
    {
        const unsigned sch = flags & (DWT2_FLAG_SPLIT | DWT2_FLAG_FACTORED | DWT2_FLAG_FUSED);
        if (sch & (sch - 1)) return DWT2_E_FLAGS;          // at most one scheme
    }
    if (((flags & DWT2_FLAG_KERNEL_MASK) >> DWT2_FLAG_KERNEL_SHIFT) > (unsigned)dwt2::kNumConfigs)
        return DWT2_E_FLAGS;
    // without a named configuration: the taller tile, which measured fastest on
    // batches of uneven images (64 of 32 ... 2048 pixels a side, 5 levels), unless the
    // lower one covers the height of every image (20000 images of 4 ... 16 pixels FP16,
    // 2 levels, persistent: 1.87 ms, now 1.71)
    int cfg = config_of(flags, wavelet);
    if (!(flags & DWT2_FLAG_KERNEL_MASK))
        for (int i = 0; i < count && cfg != dwt2::kLargeConfig; ++i)
            if (host_images[i].height > 2 * dwt2::core_rows(dwt2::kConfigs[dwt2::kDefaultConfig])) cfg = dwt2::kLargeConfig;
    if (!dwt2::persist_config_supported(cfg)) return DWT2_E_FLAGS;
    const size_t es = elem_size(dtype);
    const dwt2::KernelConfig kc = dwt2::kConfigs[cfg];
    dwt2::BatchSums sums{};
    const bool pairs = flags == 0;
    for (int i = 0; i < count; ++i) {
        const dwt2_image& im = host_images[i];
        if (!im.src || !im.dst) return DWT2_E_NULL;
        if (im.height < 2 || im.width < 2 || im.height > kMaxSide || im.width > kMaxSide) return DWT2_E_SHAPE;
        if (im.src_pitch < im.width || im.dst_pitch < im.width) return DWT2_E_PITCH;
        if (levels < 1 || levels > max_levels(im.height, im.width)) return DWT2_E_LEVELS;
        if (ranges_overlap(im.src, span_bytes(im.height, im.width, im.src_pitch, es), im.dst,
                           span_bytes(im.height, im.width, im.dst_pitch, es)))
            return DWT2_E_ALIAS;
        dwt2::add_image(im.height, im.width, levels, kc, pairs, &sums);
    }
    if (batch_spans_alias(host_images, count, es)) return DWT2_E_ALIAS;
    const bool persistent = (flags & DWT2_FLAG_PERSISTENT) && levels > 1;
    // ticket numbers and counters are 32-bit
    for (int l = 0; l < levels; ++l)
        if (sums.level[l].tiles > 0x7fff0000ull) return DWT2_E_SHAPE;
    if (sums.chunks > 0x7fff0000ull) return DWT2_E_SHAPE;
    size_t need = 0;
    const int st = dwt2_workspace_bytes_batched(host_images, count, dtype, levels, &need);
    if (st) return st;
    if (workspace_bytes < need) return DWT2_E_WORKSPACE;
    for (int i = 0; i < count; ++i) {
        const dwt2_image& im = host_images[i];
        if (ranges_overlap(workspace, need, im.src, span_bytes(im.height, im.width, im.src_pitch, es)) ||
            ranges_overlap(workspace, need, im.dst, span_bytes(im.height, im.width, im.dst_pitch, es)))
            return DWT2_E_ALIAS;
    }
    const dwt2::Scheme sch = scheme_of(flags, dtype, wavelet, false);
    if (persistent) {
        const dwt2::ImageSet S{device_images, nullptr, nullptr, 0, 0, 0, 0, 0, 0};
        const dwt2::BatchLayout L = dwt2::batch_layout(count, levels, sums.chunks);
        return report(dwt2::launch_fwd_persistent(to_dtype(dtype), sch, cfg, S, count, levels, workspace, L,
                                                  sums.tiles, (hipStream_t)stream));
    }
    dwt2::BatchLaunches B{};
    uint32_t launch_tiles[32];
    for (int l = 0; l < levels; ++B.n) {
        const dwt2::BatchSums::Level& st = sums.level[l];
        const int rows3 = !pairs || l + 3 != levels ? 0
                          : dwt2::triple_rows(dwt2::kForward, (int64_t)st.tiles3[0], (int64_t)st.tiles3[1]);
        const int n = !pairs || l + 1 >= levels ? 1 : rows3 ? 3 : batch_pair_pays(dtype, st) ? 2 : 1;
        const int rows = n != 2 ? rows3 : dwt2::pair_rows(dwt2::kForward, es, (int64_t)st.tiles32, (int64_t)st.tiles48,
                                                          (int64_t)st.samples);
        if (n == 1 && st.tiles > (uint64_t)dwt2::max_tiles(kc.waves)) return DWT2_E_SHAPE;
        B.first[B.n] = (int8_t)l;
        B.levels[B.n] = (int8_t)n;
        B.rows[B.n] = (int8_t)rows;
        // a chunk of about kRemapRows tile rows of the images' mean width
        const uint64_t near = n == 1 ? (uint64_t)dwt2::kLevelChunk : dwt2::kRemapRows * st.tiles32 / st.rows32;
        B.near[B.n] = near < 16 ? 16 : near > 4096 ? 4096 : (int32_t)near;
        launch_tiles[B.n] = (uint32_t)(n == 1 ? st.tiles : n == 3 ? st.tiles3[rows == 64] : rows == 32 ? st.tiles32 : st.tiles48);
        l += n;
    }
    return report(dwt2::launch_fwd_batched_levels(to_dtype(dtype), sch, cfg, B, device_images, count, levels,
                                                  workspace, launch_tiles, (hipStream_t)stream));
}

int dwt2_workspace_status(const void* header) {
    if (!header) return DWT2_E_NULL;
    return static_cast<const uint32_t*>(header)[0] != 0u ? DWT2_E_TIMEOUT : DWT2_OK;
}

const char* dwt2_status_string(int status) {
    switch (status) {
        case DWT2_OK: return "ok";
        case DWT2_E_NULL: return "null pointer";
        case DWT2_E_SHAPE: return "height and width must be in [2, 2^30]";
        case DWT2_E_LEVELS: return "level count out of range for this shape";
        case DWT2_E_DTYPE: return "dtype not valid for this wavelet";
        case DWT2_E_WAVELET: return "unknown or unsupported wavelet";
        case DWT2_E_BOUNDARY: return "unknown boundary extension";
        case DWT2_E_PITCH: return "pitch smaller than width";
        case DWT2_E_WORKSPACE: return "workspace missing or too small";
        case DWT2_E_ALIAS: return "src, dst and workspace must not overlap";
        case DWT2_E_HIP: return "HIP runtime error";
        case DWT2_E_FLAGS: return "flags not valid for this call";
        case DWT2_E_COUNT: return "image count must be positive";
        case DWT2_E_SCRATCH: return "the call needs more workspace than the library's fixed scratch array";
        case DWT2_E_TIMEOUT: return "a dependency wait of the persistent forward ran out of time: outputs invalid";
    }
    return "unknown status";
}

const char* dwt2_last_hip_error(void) { return g_last_hip_error.c_str(); }

}  // extern "C"
