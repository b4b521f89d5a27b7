// Two or three levels of the transform in one launch: device code (included by
// dwt2_pair_*.hip and dwt2_batched.hip).
#pragma once
#include "dwt2_kernels.inl"

namespace dwt2 {
namespace kern {
namespace pair {

// What one launch per level costs beside the first level's traffic: the LL
// band written and read again (a quarter of the level each way) and, for every
// small level, a launch and one tile's time from load to store.  A tile here
// runs both levels: a lane holds 2 x K blocks of the first level in VGPRs as
// in the one-level tile kernel, so its LL samples are exactly the 1 x K/2 blocks
// of the second level that the lane then holds, without moving a value.
//
// Forward: level 1 on the tile, its details stored, its LL samples (rounded
// to the storage type, as a store would) taken as the blocks of level 2, level
// 2 on them, its four bands stored.  Inverse and adjoint: the mirror image.
//
// The halo is that of both levels, 2 blocks of each: kHalo2 = 6 block rows of
// level 1 above and below, and the columns of kEdge2 lanes on either side,
// which load and compute but do not store: 3 would do, but 4 leave 112 columns,
// whose subband segments (448 bytes of FP32) are whole 64-byte sectors (two levels
// forward take 10 % longer with 3 for 8192^2 FP32, 20 % for 3 x 8192^2 BF16).  Halo
// values come from the neighbouring lane or wave like any others, so a step has no
// halo operands:
// horizontal neighbours are DPP shifts that fold into the adds, vertical ones
// the lane's own rows or one LDS row per wave and step.
//
// Borders.  Level 1 runs on the symmetric extension of its input.  The LL samples
// this gives outside the image are not what level 2 extends them to when a side is
// even, so a border tile passes its LL samples through LDS and each lane takes the
// reflected ones.  Every value is formed by the same operations in the same
// order as by the one-level kernels: the results are theirs bit for bit.

template <typename V, int NW> struct PairLds {
    Vec2<V> t[NW + 1][2][kLanes];     // top block rows (x0, x1) of every wave, for the wave above
    Vec2<V> s[NW + 1][2][kLanes];     // bottom ones (x2, x3), for the wave below
};
// LL samples of a border tile.
template <typename V, int ROWS> struct PairPlane { V p[ROWS][2 * kLanes]; };

// lane i <- lane i + 1 / i - 1 (0 beyond the wave): whole-wave DPP shifts the
// compiler folds into the instruction that uses them.
__device__ __forceinline__ int right1(int v) { return __builtin_amdgcn_update_dpp(0, v, 0x130, 0xf, 0xf, true); }
__device__ __forceinline__ int left1(int v) { return __builtin_amdgcn_update_dpp(0, v, 0x138, 0xf, 0xf, true); }
__device__ __forceinline__ float right1(float v) { return __int_as_float(right1(__float_as_int(v))); }
__device__ __forceinline__ float left1(float v) { return __int_as_float(left1(__float_as_int(v))); }

constexpr bool horizontal_kind(int k) { return k == kSepH || k == kSepHInt || k == kSepHIntInv; }
constexpr bool vertical_kind(int k) { return k == kSepV || k == kSepVInt || k == kSepVIntInv; }

// Predict-shaped step: rows top to bottom, blocks left to right, so every
// operand right of or below a block is still the value before the step.
template <int KIND, int NW, int BPL, int K, typename V>
__device__ __forceinline__ void plus(V (&a)[K][4 * BPL], PairLds<V, NW>& L, int lane, int wv, const Geo& g, float c) {
    V dn[4 * BPL];
#pragma unroll
    for (int i = 0; i < 4 * BPL; ++i) dn[i] = V(0);
    if constexpr (!horizontal_kind(KIND)) {
#pragma unroll
        for (int b = 0; b < BPL; ++b) L.t[wv][b][lane] = Vec2<V>{a[0][4 * b], a[0][4 * b + 1]};
        __syncthreads();
#pragma unroll
        for (int b = 0; b < BPL; ++b) {
            const Vec2<V> v = L.t[wv + 1][b][lane];
            dn[4 * b] = v.a;
            dn[4 * b + 1] = v.b;
        }
    }
#pragma unroll
    for (int r = 0; r < K; ++r) {
        const V(&d)[4 * BPL] = r + 1 < K ? a[r + 1 < K ? r + 1 : r] : dn;
        const V R0 = vertical_kind(KIND) ? V(0) : right1(a[r][0]);
        const V R2 = vertical_kind(KIND) ? V(0) : right1(a[r][2]);
        const V RD0 = vertical_kind(KIND) || horizontal_kind(KIND) ? V(0) : right1(d[0]);
#pragma unroll
        for (int b = 0; b < BPL; ++b)
            plus_block<KIND, false, false>(a[r][4 * b], a[r][4 * b + 1], a[r][4 * b + 2], a[r][4 * b + 3],
                                         b + 1 < BPL ? a[r][4 * ((b + 1) % BPL)] : R0,
                                         b + 1 < BPL ? a[r][4 * ((b + 1) % BPL) + 2] : R2, d[4 * b], d[4 * b + 1],
                                         b + 1 < BPL ? d[4 * ((b + 1) % BPL)] : RD0, g.gcL + b, g.gr0 + r, g, c);
    }
}

// Update-shaped step: rows bottom to top, blocks right to left.
template <int KIND, int NW, int BPL, int K, typename V>
__device__ __forceinline__ void minus(V (&a)[K][4 * BPL], PairLds<V, NW>& L, int lane, int wv, const Geo& g, float c) {
    V up[4 * BPL];
#pragma unroll
    for (int i = 0; i < 4 * BPL; ++i) up[i] = V(0);
    if constexpr (!horizontal_kind(KIND)) {
#pragma unroll
        for (int b = 0; b < BPL; ++b) L.s[wv + 1][b][lane] = Vec2<V>{a[K - 1][4 * b + 2], a[K - 1][4 * b + 3]};
        __syncthreads();
#pragma unroll
        for (int b = 0; b < BPL; ++b) {
            const Vec2<V> v = L.s[wv][b][lane];
            up[4 * b + 2] = v.a;
            up[4 * b + 3] = v.b;
        }
    }
#pragma unroll
    for (int r = K - 1; r >= 0; --r) {
        const V(&u)[4 * BPL] = r > 0 ? a[r > 0 ? r - 1 : 0] : up;
        const V L1 = vertical_kind(KIND) ? V(0) : left1(a[r][4 * BPL - 3]);
        const V L3 = vertical_kind(KIND) ? V(0) : left1(a[r][4 * BPL - 1]);
        const V LU3 = vertical_kind(KIND) || horizontal_kind(KIND) ? V(0) : left1(u[4 * BPL - 1]);
#pragma unroll
        for (int b = BPL - 1; b >= 0; --b)
            minus_block<KIND, false, false>(a[r][4 * b], a[r][4 * b + 1], a[r][4 * b + 2], a[r][4 * b + 3],
                                          b > 0 ? a[r][4 * ((b + BPL - 1) % BPL) + 1] : L1,
                                          b > 0 ? a[r][4 * ((b + BPL - 1) % BPL) + 3] : L3, u[4 * b + 2], u[4 * b + 3],
                                          b > 0 ? u[4 * ((b + BPL - 1) % BPL) + 3] : LU3, g.gcL + b, g.gr0 + r, g, c);
    }
}

template <int BPL, int K, typename V>
__device__ __forceinline__ void scale_bands(V (&a)[K][4 * BPL], float s0, float s3) {
#pragma unroll
    for (int r = 0; r < K; ++r)
#pragma unroll
        for (int b = 0; b < BPL; ++b) {
            a[r][4 * b] *= s0;
            a[r][4 * b + 3] *= s3;
        }
}

// The step program of one level (the same steps as the one-level kernel's
// fused and factored schemes).  Predict- and update-shaped steps alternate
// over both levels, and each shape has its own LDS rows, so the one barrier of
// a step also orders the rows' reuse.
template <int DIR, int WAV, int SCH, int NW, int BPL, int K, typename V>
__device__ __forceinline__ void steps(V (&a)[K][4 * BPL], PairLds<V, NW>& L, int lane, int wv, const Geo& g) {
    static_assert(SCH == kSchemeFused || SCH == kSchemeFactored, "default schemes");
#define DWT2_P(KIND_, c_) plus<KIND_, NW, BPL, K>(a, L, lane, wv, g, (c_));
#define DWT2_M(KIND_, c_) minus<KIND_, NW, BPL, K>(a, L, lane, wv, g, (c_));
    if constexpr (WAV == kCdf53) {
        static_assert(SCH == kSchemeFused, "the integer wavelet's default scheme");
        if constexpr (DIR == kForward) { DWT2_P(kIntFwd, 0.f) DWT2_M(kIntFwd, 0.f) }
        else { DWT2_M(kIntInv, 0.f) DWT2_P(kIntInv, 0.f) }
    } else if constexpr (WAV == kCdf53Real) {
        if constexpr (DIR == kForward) {
            if constexpr (SCH == kSchemeFused) { DWT2_P(kFloat, kP53) DWT2_M(kFloat, kU53) }
            else { DWT2_P(kSepH, kP53) DWT2_P(kSepV, kP53) DWT2_M(kSepH, kU53) DWT2_M(kSepV, kU53) }
            scale_bands<BPL, K>(a, kZeta53Sq, kZeta53SqInv);
        } else {
            scale_bands<BPL, K>(a, kZeta53SqInv, kZeta53Sq);
            if constexpr (SCH == kSchemeFused) { DWT2_M(kFloat, -kU53) DWT2_P(kFloat, -kP53) }
            else { DWT2_M(kSepV, -kU53) DWT2_M(kSepH, -kU53) DWT2_P(kSepV, -kP53) DWT2_P(kSepH, -kP53) }
        }
    } else if constexpr (DIR == kForward) {
        if constexpr (SCH == kSchemeFused) {
            DWT2_P(kFloat, kAlpha) DWT2_M(kFloat, kBeta) DWT2_P(kFloat, kGamma) DWT2_M(kFloat, kDelta)
        } else {
            DWT2_P(kSepH, kAlpha) DWT2_P(kSepV, kAlpha) DWT2_M(kSepH, kBeta) DWT2_M(kSepV, kBeta)
            DWT2_P(kSepH, kGamma) DWT2_P(kSepV, kGamma) DWT2_M(kSepH, kDelta) DWT2_M(kSepV, kDelta)
        }
        scale_bands<BPL, K>(a, kZeta2, kZetaM2);
    } else if constexpr (DIR == kInverse) {
        scale_bands<BPL, K>(a, kZetaM2, kZeta2);
        if constexpr (SCH == kSchemeFused) {
            DWT2_M(kFloat, -kDelta) DWT2_P(kFloat, -kGamma) DWT2_M(kFloat, -kBeta) DWT2_P(kFloat, -kAlpha)
        } else {
            DWT2_M(kSepV, -kDelta) DWT2_M(kSepH, -kDelta) DWT2_P(kSepV, -kGamma) DWT2_P(kSepH, -kGamma)
            DWT2_M(kSepV, -kBeta) DWT2_M(kSepH, -kBeta) DWT2_P(kSepV, -kAlpha) DWT2_P(kSepH, -kAlpha)
        }
    } else {
        scale_bands<BPL, K>(a, kZeta2, kZetaM2);
        DWT2_P(kFloat, kDelta) DWT2_M(kFloat, kGamma) DWT2_P(kFloat, kBeta) DWT2_M(kFloat, kAlpha)
    }
#undef DWT2_P
#undef DWT2_M
}

// The symmetric extension of N positions on either side (fold() takes -6 and
// above; positions further out, which no stored output reads, keep their
// parity and move there).
template <int N>
__device__ __forceinline__ void fold_both(int (&p)[N], int n) {
#pragma unroll
    for (int i = 0; i < N; ++i) p[i] = p[i] < -6 ? -6 + (p[i] & 1) : p[i];
    fold(p, n);
}

// The image rows of a tile (forward): g.cb0 may be negative.
template <typename T, int BPL, int K>
__device__ __forceinline__ void load_image(typename St<T>::V (&a)[K][4 * BPL], const T* in, int64_t pitch, int h,
                                           int w, const Geo& g, bool interior, int lane) {
    using V = typename St<T>::V;
    int rows[2 * K];
#pragma unroll
    for (int i = 0; i < 2 * K; ++i) rows[i] = 2 * g.gr0 + i;
    if (!interior) fold_both(rows, h);
    const int c0 = 2 * g.gcL;
    if (interior || (c0 >= 0 && c0 + 2 * BPL <= w)) {
        const T* const base = in + 2 * g.cb0;
#pragma unroll
        for (int i = 0; i < 2 * K; ++i) {
            V v[2 * BPL];
            load_vec<T, 2 * BPL>(lane_at(base + (int64_t)rows[i] * pitch, (uint32_t)lane * (2 * BPL * sizeof(T))), v);
#pragma unroll
            for (int s = 0; s < 2 * BPL; ++s) a[i >> 1][4 * (s >> 1) + 2 * (i & 1) + (s & 1)] = v[s];
        }
    } else {
        int cols[2 * BPL];
#pragma unroll
        for (int i = 0; i < 2 * BPL; ++i) cols[i] = c0 + i;
        fold_both(cols, w);
#pragma unroll
        for (int i = 0; i < 2 * K; ++i)
#pragma unroll
            for (int s = 0; s < 2 * BPL; ++s)
                a[i >> 1][4 * (s >> 1) + 2 * (i & 1) + (s & 1)] = load_at(in + (int64_t)rows[i] * pitch, cols[s]);
    }
}

template <typename T, int N>
__device__ __forceinline__ void load_band_row(typename St<T>::V (&v)[N], const T* p) {
    if constexpr (N > 1) load_vec<T, N>(p, v);
    else v[0] = St<T>::load(p[0]);
}
template <typename T, int N>
__device__ __forceinline__ void store_band_row(T* p, const typename St<T>::V (&v)[N]) {
    // a wave's row of single 16-bit samples is less than a line: an ordinary
    // store, so that the caches gather the rows' neighbours (3 x 8192^2 BF16,
    // two levels forward, takes 13 % longer with nontemporal ones)
    if constexpr (N > 1) store_vec<T, N>(p, v);
    else if constexpr (sizeof(T) == 4) nt_store1<T>(p, St<T>::store(v[0]));
    else p[0] = St<T>::store(v[0]);
}

// The bands K0 .. 3 of a tile of a pyramid level (h x w; inverse and adjoint), and
// the (folded) positions of a's samples.
template <typename T, int K0, int BPL, int K>
__device__ __forceinline__ void load_bands(typename St<T>::V (&a)[K][4 * BPL], const T* ll, int64_t ll_pitch,
                                           const T* det, int64_t pitch, int h, int w, const Geo& g, bool interior,
                                           int lane, int (&rows)[2 * K], int (&cols)[2 * BPL]) {
    using V = typename St<T>::V;
#pragma unroll
    for (int i = 0; i < 2 * K; ++i) rows[i] = 2 * g.gr0 + i;
    if (!interior) fold_both(rows, h);
#pragma unroll
    for (int i = 0; i < 2 * BPL; ++i) cols[i] = 2 * g.gcL + i;
    if (interior || (cols[0] >= 0 && cols[2 * BPL - 1] < w)) {
#pragma unroll
        for (int r = 0; r < K; ++r)
#pragma unroll
            for (int k = K0; k < 4; ++k) {
                V v[BPL];
                load_band_row<T, BPL>(v, lane_at(subband_row(ll, ll_pitch, det, pitch, g, k,
                                                             rows[2 * r + (k >> 1)] >> 1) + g.cb0,
                                                 (uint32_t)lane * (BPL * sizeof(T))));
#pragma unroll
                for (int b = 0; b < BPL; ++b) a[r][4 * b + k] = v[b];
            }
    } else {
        fold_both(cols, w);
#pragma unroll
        for (int r = 0; r < K; ++r)
#pragma unroll
            for (int k = K0; k < 4; ++k) {
                const T* row = subband_row(ll, ll_pitch, det, pitch, g, k, rows[2 * r + (k >> 1)] >> 1);
#pragma unroll
                for (int b = 0; b < BPL; ++b) a[r][4 * b + k] = load_at(row, cols[2 * b + (k & 1)] >> 1);
            }
    }
}

// Bands K0 .. 3 of the tile's core to a pyramid level (forward).  One body for
// interior and border tiles: with a body each, the compiler gathered the
// samples of every store ahead of the choice (33 more registers at K = 6, two
// work-groups on a CU instead of three).  H: halo
// rows of the tile at this level (NW * K rows).
template <typename T, int K0, int H, int NW, int BPL, int K>
__device__ __forceinline__ void store_bands(typename St<T>::V (&a)[K][4 * BPL], T* ll, int64_t ll_pitch, T* det,
                                            int64_t pitch, const Geo& g, int lane, int wv) {
    using V = typename St<T>::V;
    constexpr bool kBySubband = sizeof(T) == 4;
    T* row[4];
#pragma unroll
    for (int k = K0; k < 4; ++k) row[k] = subband_row(ll, ll_pitch, det, pitch, g, k, g.gr0) + g.cb0;
#pragma unroll
    for (int k0 = K0; k0 < (kBySubband ? 4 : K0 + 1); ++k0)
#pragma unroll
        for (int r = 0; r < K; ++r)
#pragma unroll
            for (int k = (kBySubband ? k0 : K0); k < (kBySubband ? k0 + 1 : 4); ++k) {
                T* const p = lane_at(row[k], (uint32_t)lane * (BPL * sizeof(T)));
                row[k] += k == 0 ? ll_pitch : pitch;
                const int tr = wv * K + r;
                if (tr < H || tr >= NW * K - H) continue;
                if (g.gr0 + r >= (k >= 2 ? g.nOr : g.nEr)) continue;
                V v[BPL];
#pragma unroll
                for (int b = 0; b < BPL; ++b) v[b] = a[r][4 * b + k];
                const int left = ((k & 1) ? g.nOc : g.nEc) - g.gcL;   // samples to the row's end
                if (left >= BPL) {
                    store_band_row<T, BPL>(p, v);
                } else {
#pragma unroll
                    for (int b = 0; b + 1 < BPL; ++b)
                        if (b < left) p[b] = St<T>::store(v[b]);
                }
            }
}

// The tile's core as image rows (inverse and adjoint).
template <typename T, bool BORDER, int H, int NW, int BPL, int K>
__device__ __forceinline__ void store_image(typename St<T>::V (&a)[K][4 * BPL], T* out, int64_t pitch, int h, int w,
                                            const Geo& g, int lane, int wv) {
    using V = typename St<T>::V;
    T* row = out + (int64_t)(2 * g.gr0) * pitch + 2 * g.cb0;
    const int left = w - 2 * g.gcL;
#pragma unroll
    for (int i = 0; i < 2 * K; ++i) {
        T* const p = lane_at(row, (uint32_t)lane * (2 * BPL * sizeof(T)));
        row += pitch;
        const int tr = wv * K + (i >> 1);
        if (tr < H || tr >= NW * K - H) continue;
        if (BORDER && 2 * g.gr0 + i >= h) continue;
        V v[2 * BPL];
#pragma unroll
        for (int s = 0; s < 2 * BPL; ++s) v[s] = a[i >> 1][4 * (s >> 1) + 2 * (i & 1) + (s & 1)];
        if (!BORDER || left >= 2 * BPL) {
            store_vec<T, 2 * BPL>(p, v);
        } else {
#pragma unroll
            for (int s = 0; s + 1 < 2 * BPL; ++s)
                if (s < left) p[s] = St<T>::store(v[s]);
        }
    }
}

__device__ __forceinline__ int clamp_to(int x, int n) { return x < 0 ? 0 : x < n ? x : n - 1; }

// LL samples of a border tile's blocks (inverse and adjoint): each at its
// reflected pixel position of the h x w level, `ll(row, col)` being the block's;
// the adjoint's times f at the ends of an axis and `all` (see scale_edges()).
template <int BPL, int K, bool ADJ, typename V, typename F>
__device__ __forceinline__ void reflect_ll(V (&a)[K][4 * BPL], const Geo& g, int h, int w, float f, float all,
                                           const F& ll) {
    int rows[K], cols[BPL];
#pragma unroll
    for (int i = 0; i < K; ++i) rows[i] = 2 * (g.gr0 + i);
#pragma unroll
    for (int i = 0; i < BPL; ++i) cols[i] = 2 * (g.gcL + i);
    fold_both(rows, h);
    fold_both(cols, w);
#pragma unroll
    for (int r = 0; r < K; ++r)
#pragma unroll
        for (int b = 0; b < BPL; ++b) {
            a[r][4 * b] = ll(rows[r] >> 1, cols[b] >> 1);
            if constexpr (ADJ) {
                a[r][4 * b] *= rows[r] == 0 || rows[r] == h - 1 ? f * all : all;
                a[r][4 * b] *= cols[b] == 0 || cols[b] == w - 1 ? f : 1.f;
            }
        }
}

// What storing a value and loading it again gives.
template <typename T>
__device__ __forceinline__ typename St<T>::V stored(typename St<T>::V v) { return St<T>::load(St<T>::store(v)); }

// Tile (tx, ty) of levels l and l + 1.
template <int DIR, int WAV, typename T, int SCH, int NW, int K>
__device__ __forceinline__ void tile(const PairParams& P, int tx, int ty, PairLds<typename St<T>::V, NW>& L,
                                     PairPlane<typename St<T>::V, NW * K>& S, int lane, int wv) {
    using V = typename St<T>::V;
    static_assert(K % 2 == 0, "a wave's rows are whole blocks of the second level");
    constexpr int R = NW * K, CY = R - 2 * kHalo2, K2 = K / 2;
    Geo g, g2;
    g.nEr = (P.h + 1) >> 1; g.nOr = P.h >> 1;
    g.nEc = (P.w + 1) >> 1; g.nOc = P.w >> 1;
    const int r0 = ty * CY - kHalo2;               // tile's first block row of level 1
    g.cb0 = tx * kPairCols - 2 * kEdge2;
    g.gcL = g.cb0 + 2 * lane;
    g.gr0 = r0 + wv * K;
    const int h2 = g.nEr, w2 = g.nEc;
    g2.nEr = (h2 + 1) >> 1; g2.nOr = h2 >> 1;
    g2.nEc = (w2 + 1) >> 1; g2.nOc = w2 >> 1;
    g2.cb0 = g.cb0 >> 1;
    g2.gcL = g2.cb0 + lane;
    g2.gr0 = g.gr0 >> 1;
    // Waves below both levels' images leave (see below_image), if there are two of
    // them: 65536 planes of 16^2 FP32 forward 623 us, now 477.  One of eight leaving
    // alone cost 4096 planes of 64^2 5 to 8 % (adjoint 96 us for 90).
    auto gone = [&](int v) {
        const int first = r0 + (v < NW - 2 ? v : NW - 2) * K;
        return below_image(first, P.h) && below_image(first >> 1, h2);
    };
    if (gone(wv)) return;
    const bool interior = r0 >= 0 && g.cb0 >= 0 && r0 + R <= g.nOr && g.cb0 + 2 * kLanes <= g.nOc;
    const bool core_lane = lane >= kEdge2 && lane < kLanes - kEdge2;
    V a[K][8], b[K2][4];
    if constexpr (DIR == kForward) {
        load_image<T, 2, K>(a, static_cast<const T*>(P.in), P.in_pitch, P.h, P.w, g, interior, lane);
        steps<DIR, WAV, SCH, NW, 2, K>(a, L, lane, wv, g);
        T* const out = static_cast<T*>(P.out);
        if (core_lane) store_bands<T, 1, kHalo2, NW, 2, K>(a, out, 0, out, P.out_pitch, g, lane, wv);
#pragma unroll
        for (int r = 0; r < K2; ++r)
#pragma unroll
            for (int k = 0; k < 4; ++k) b[r][k] = stored<T>(a[2 * r + (k >> 1)][4 * (k & 1)]);
        if (!interior) {
#pragma unroll
            for (int r = 0; r < K2; ++r)
#pragma unroll
                for (int k = 0; k < 4; ++k) S.p[wv * K + 2 * r + (k >> 1)][2 * lane + (k & 1)] = b[r][k];
            __syncthreads();
            int rows[K], cols[2];
#pragma unroll
            for (int i = 0; i < K; ++i) rows[i] = 2 * g2.gr0 + i;
            cols[0] = 2 * g2.gcL;
            cols[1] = 2 * g2.gcL + 1;
            fold_both(rows, h2);
            fold_both(cols, w2);
#pragma unroll
            for (int r = 0; r < K2; ++r)
#pragma unroll
                for (int k = 0; k < 4; ++k)
                    b[r][k] = S.p[clamp_to(rows[2 * r + (k >> 1)] - r0, R)][clamp_to(cols[k & 1] - g.cb0, 2 * kLanes)];
        }
        steps<DIR, WAV, SCH, NW, 1, K2>(b, L, lane, wv, g2);
        T* const ll = static_cast<T*>(P.ll);
        if (core_lane) store_bands<T, 0, kHalo2 / 2, NW, 1, K2>(b, ll, P.ll_pitch, out, P.out_pitch, g2, lane, wv);
    } else {
        constexpr bool kAdj = DIR == kAdjoint;
        const T* const det = static_cast<const T*>(P.in);
        int rows[2 * K], cols[4], rows2[2 * K2], cols2[2];
        load_bands<T, 0, 1, K2>(b, static_cast<const T*>(P.ll), P.ll_pitch, det, P.in_pitch, h2, w2, g2, interior, lane,
                                rows2, cols2);
        load_bands<T, 1, 2, K>(a, det, P.in_pitch, det, P.in_pitch, P.h, P.w, g, interior, lane, rows, cols);
        float all = 1.f;
        if constexpr (kAdj) {
            if (!interior) {
                all = tile_scale<T, NW>(largest<1, 2>(a, largest<0, 1>(b, V(0))), lane, wv, gone);
                // the columns anew: kept from the load they take 85 registers in all
                // of the 80 that six waves a SIMD may have (8 x 6)
                int gc = g.gcL;
                asm volatile("" : "+v"(gc));
#pragma unroll
                for (int i = 0; i < 4; ++i) cols[i] = 2 * gc + i;
                cols2[0] = gc;
                cols2[1] = gc + 1;
                fold_both(cols, P.w);
                fold_both(cols2, w2);
                scale_edges<0, 4, 1>(b, rows2, cols2, h2, w2, 2.f, all);
                scale_edges<1, 4, 2>(a, rows, cols, P.h, P.w, 2.f, all);
            }
        }
        steps<DIR, WAV, SCH, NW, 1, K2>(b, L, lane, wv, g2);
        if constexpr (kAdj) {
            if (!interior) scale_edges<0, 4, 1>(b, g2, h2, w2, 0.5f, undo(all));
        }
#pragma unroll
        for (int r = 0; r < K2; ++r)
#pragma unroll
            for (int k = 0; k < 4; ++k) a[2 * r + (k >> 1)][4 * (k & 1)] = stored<T>(b[r][k]);
        if (!interior) {
#pragma unroll
            for (int r = 0; r < K; ++r)
#pragma unroll
                for (int c = 0; c < 2; ++c) S.p[wv * K + r][2 * lane + c] = a[r][4 * c];
            __syncthreads();
            reflect_ll<2, K, kAdj>(a, g, P.h, P.w, 2.f, all, [&](int row, int col) -> V {
                return S.p[clamp_to(row - r0, R)][clamp_to(col - g.cb0, 2 * kLanes)];
            });
        }
        steps<DIR, WAV, SCH, NW, 2, K>(a, L, lane, wv, g);
        if constexpr (kAdj) {
            if (!interior) scale_edges<0, 4, 2>(a, g, P.h, P.w, 0.5f, undo(all));
        }
        if (core_lane) {
            T* const out = static_cast<T*>(P.out);
            if (interior) store_image<T, false, kHalo2, NW, 2, K>(a, out, P.out_pitch, P.h, P.w, g, lane, wv);
            else store_image<T, true, kHalo2, NW, 2, K>(a, out, P.out_pitch, P.h, P.w, g, lane, wv);
        }
    }
}

// ---- three levels in one launch ---------------------------------------------
// For the last three levels of small images, where a launch costs more than the
// work: 192 x 256, 3 levels, took a two-level launch of 7.3 us and a one-level
// launch of 6.  Levels l and l + 1 as above; level l + 2 takes its samples from
// LDS, a block a lane (32 blocks across) and a block row a wave, with the
// symmetric extension applied in the read.  The halo is that of three levels, 14
// block rows and columns of level 1, rounded up to whole blocks of level 3.
// Four rows a wave, the fewest that are whole blocks of level 3: what such a
// launch costs is one wave's instructions, each fetched and waited for, so
// 12 waves x 4 rows beat 8 x 6 at the same tile (192 x 256 FP32 forward 9.3 us
// for 10.4, inverse 10.9 for 11.8).
//
// Tile (tx, ty) of levels l, l + 1 and l + 2: NW waves x 4 rows, of which all but
// the halo and kTripleCols block columns are stored.
template <int DIR, int WAV, typename T, int SCH, int NW>
__device__ __forceinline__ void tile3(const PairParams& P, int tx, int ty, PairLds<typename St<T>::V, NW>& L,
                                      PairPlane<typename St<T>::V, NW * kTripleK>& S, int lane, int wv) {
    using V = typename St<T>::V;
    constexpr int K = kTripleK, K2 = K / 2, R = NW * K, R2 = R / 2;
    Geo g, g2, g3;
    const int h2 = (P.h + 1) >> 1, w2 = (P.w + 1) >> 1, h3 = (h2 + 1) >> 1, w3 = (w2 + 1) >> 1;
    g.nEr = h2; g.nOr = P.h >> 1; g.nEc = w2; g.nOc = P.w >> 1;
    g2.nEr = h3; g2.nOr = h2 >> 1; g2.nEc = w3; g2.nOc = w2 >> 1;
    g3.nEr = (h3 + 1) >> 1; g3.nOr = h3 >> 1; g3.nEc = (w3 + 1) >> 1; g3.nOc = w3 >> 1;
    const int r0 = ty * (R - 2 * kHalo3) - kHalo3, c0 = tx * kTripleCols - kHalo3;   // multiples of 4
    g.cb0 = c0;
    g.gcL = c0 + 2 * lane;
    g.gr0 = r0 + wv * K;
    g2.cb0 = c0 / 2;
    g2.gcL = g2.cb0 + lane;
    g2.gr0 = g.gr0 / 2;
    g3.cb0 = c0 / 4;
    g3.gcL = g3.cb0 + lane;
    g3.gr0 = r0 / 4 + wv;
    auto gone = [&](int v) {
        const int first = r0 + v * K;
        return below_image(first, P.h) && below_image(first / 2, h2) && below_image(r0 / 4 + v, h3);
    };
    if (gone(wv)) return;
    const bool interior = r0 >= 0 && c0 >= 0 && r0 + R <= g.nOr && c0 + 2 * kLanes <= g.nOc;
    constexpr int kEl = kHalo3 / 2;                // halo lanes of levels 1 and 2; half as many at level 3
    const bool core_lane = lane >= kEl && lane < kLanes - kEl;
    const bool core_lane3 = lane >= kEl / 2 && lane < kLanes / 2 - kEl / 2;
    V a[K][8], b[K2][4], c[1][4];
    // LL samples of level 1 for level 2 (forward) or back (inverse), see tile()
    auto plane1 = [&](int row, int col) -> V& { return S.p[clamp_to(row - r0, R)][clamp_to(col - c0, 2 * kLanes)]; };
    // those of level 2 for level 3: R2 rows of 64, in the same LDS rows
    auto plane2 = [&](int row, int col) -> V& { return S.p[clamp_to(row - r0 / 2, R2)][clamp_to(col - c0 / 2, kLanes)]; };
    if constexpr (DIR == kForward) {
        load_image<T, 2, K>(a, static_cast<const T*>(P.in), P.in_pitch, P.h, P.w, g, interior, lane);
        steps<DIR, WAV, SCH, NW, 2, K>(a, L, lane, wv, g);
        T* const out = static_cast<T*>(P.out);
        if (core_lane) store_bands<T, 1, kHalo3, NW, 2, K>(a, out, 0, out, P.out_pitch, g, lane, wv);
#pragma unroll
        for (int r = 0; r < K2; ++r)
#pragma unroll
            for (int k = 0; k < 4; ++k) b[r][k] = stored<T>(a[2 * r + (k >> 1)][4 * (k & 1)]);
        if (!interior) {
#pragma unroll
            for (int r = 0; r < K2; ++r)
#pragma unroll
                for (int k = 0; k < 4; ++k) S.p[wv * K + 2 * r + (k >> 1)][2 * lane + (k & 1)] = b[r][k];
            __syncthreads();
            int rows[K], cols[2];
#pragma unroll
            for (int i = 0; i < K; ++i) rows[i] = 2 * g2.gr0 + i;
            cols[0] = 2 * g2.gcL;
            cols[1] = 2 * g2.gcL + 1;
            fold_both(rows, h2);
            fold_both(cols, w2);
#pragma unroll
            for (int r = 0; r < K2; ++r)
#pragma unroll
                for (int k = 0; k < 4; ++k) b[r][k] = plane1(rows[2 * r + (k >> 1)], cols[k & 1]);
        }
        steps<DIR, WAV, SCH, NW, 1, K2>(b, L, lane, wv, g2);
        if (core_lane) store_bands<T, 1, kHalo3 / 2, NW, 1, K2>(b, out, 0, out, P.out_pitch, g2, lane, wv);
        // the reads of plane 1 precede the barriers of level 2's steps
#pragma unroll
        for (int r = 0; r < K2; ++r) S.p[wv * K2 + r][lane] = stored<T>(b[r][0]);
        __syncthreads();
        int rows[2] = {2 * g3.gr0, 2 * g3.gr0 + 1}, cols[2] = {2 * g3.gcL, 2 * g3.gcL + 1};
        fold_both(rows, h3);
        fold_both(cols, w3);
#pragma unroll
        for (int k = 0; k < 4; ++k) c[0][k] = plane2(rows[k >> 1], cols[k & 1]);
        steps<DIR, WAV, SCH, NW, 1, 1>(c, L, lane, wv, g3);
        T* const ll = static_cast<T*>(P.ll);
        if (core_lane3) store_bands<T, 0, kHalo3 / 4, NW, 1, 1>(c, ll, P.ll_pitch, out, P.out_pitch, g3, lane, wv);
    } else {
        constexpr bool kAdj = DIR == kAdjoint;
        const T* const det = static_cast<const T*>(P.in);
        int rows[2 * K], cols[4], rows2[2 * K2], cols2[2], rows3[2], cols3[2];
        load_bands<T, 0, 1, 1>(c, static_cast<const T*>(P.ll), P.ll_pitch, det, P.in_pitch, h3, w3, g3, false, lane,
                               rows3, cols3);
        load_bands<T, 1, 1, K2>(b, det, P.in_pitch, det, P.in_pitch, h2, w2, g2, interior, lane, rows2, cols2);
        load_bands<T, 1, 2, K>(a, det, P.in_pitch, det, P.in_pitch, P.h, P.w, g, interior, lane, rows, cols);
        float all = 1.f;
        if constexpr (kAdj) {
            if (!interior) {
                all = tile_scale<T, NW>(largest<1, 2>(a, largest<1, 1>(b, largest<0, 1>(c, V(0)))), lane, wv, gone);
                scale_edges<0, 4, 1>(c, rows3, cols3, h3, w3, 2.f, all);
                scale_edges<1, 4, 1>(b, rows2, cols2, h2, w2, 2.f, all);
                scale_edges<1, 4, 2>(a, rows, cols, P.h, P.w, 2.f, all);
            }
        }
        steps<DIR, WAV, SCH, NW, 1, 1>(c, L, lane, wv, g3);
        if constexpr (kAdj) {
            if (!interior) scale_edges<0, 4, 1>(c, g3, h3, w3, 0.5f, undo(all));
        }
        if (lane < kLanes / 2) {
#pragma unroll
            for (int k = 0; k < 4; ++k) S.p[2 * wv + (k >> 1)][2 * lane + (k & 1)] = stored<T>(c[0][k]);
        }
        __syncthreads();
        // an interior tile is free of border weights: an end of level 2 or 3 that it
        // holds lies in its halo, further out than its outputs read
        reflect_ll<1, K2, kAdj>(b, g2, h2, w2, interior ? 1.f : 2.f, all, plane2);
        steps<DIR, WAV, SCH, NW, 1, K2>(b, L, lane, wv, g2);
        if constexpr (kAdj) {
            if (!interior) scale_edges<0, 4, 1>(b, g2, h2, w2, 0.5f, undo(all));
        }
#pragma unroll
        for (int r = 0; r < K2; ++r)
#pragma unroll
            for (int k = 0; k < 4; ++k) a[2 * r + (k >> 1)][4 * (k & 1)] = stored<T>(b[r][k]);
        if (!interior) {
            // the reads of plane 2 precede the barriers of level 2's steps
#pragma unroll
            for (int r = 0; r < K; ++r)
#pragma unroll
                for (int q = 0; q < 2; ++q) S.p[wv * K + r][2 * lane + q] = a[r][4 * q];
            __syncthreads();
            reflect_ll<2, K, kAdj>(a, g, P.h, P.w, 2.f, all, plane1);
        }
        steps<DIR, WAV, SCH, NW, 2, K>(a, L, lane, wv, g);
        if constexpr (kAdj) {
            if (!interior) scale_edges<0, 4, 2>(a, g, P.h, P.w, 0.5f, undo(all));
        }
        if (core_lane)
            store_image<T, true, kHalo3, NW, 2, K>(a, static_cast<T*>(P.out), P.out_pitch, P.h, P.w, g, lane, wv);
    }
}

// The calling work-group's tile (tx, ty) and its plane's parameters Q; false past
// the last tile (uniform over the work-group).
template <typename T>
__device__ __forceinline__ bool pick_tile(const PairParams& P, PairParams& Q, int& tx, int& ty) {
    // every kernel argument in one round trip, see fetch_params
    asm volatile("" ::"s"(P.in), "s"(P.in_pitch), "s"(P.in_ps), "s"(P.out), "s"(P.out_pitch), "s"(P.out_ps), "s"(P.ll),
                 "s"(P.ll_pitch), "s"(P.ll_ps), "s"(P.h), "s"(P.w), "s"(P.tiles_x), "s"(P.tiles_y), "s"(P.planes),
                 "s"(P.chunk));
    // XCD remap of the tile list (all planes), as in the one-level kernel
    const int nt = P.tiles_x * P.tiles_y;
    const int j = (int)(blockIdx.x >> 3);
    const int n = ((j / P.chunk) * 8 + (int)(blockIdx.x & 7)) * P.chunk + j % P.chunk;
    if (n >= nt * P.planes) return false;
    const int pl = n / nt;
    const int t = n - pl * nt;
    ty = t / P.tiles_x;
    tx = t - ty * P.tiles_x;
    Q = P;
    Q.in = static_cast<const T*>(P.in) + (int64_t)pl * P.in_ps;
    Q.out = static_cast<T*>(P.out) + (int64_t)pl * P.out_ps;
    Q.ll = static_cast<T*>(P.ll) + (int64_t)pl * P.ll_ps;
    return true;
}

// The adjoint's tiles of 8 x 6 are held to the 80 registers that six waves a SIMD may
// have (83 otherwise: 3 x 2160 x 3840 FP32, two levels, 41.8 us for 37.2).
template <int DIR, int WAV, typename T, int SCH, int NW, int K, int LEVELS = 2>
__global__ void __launch_bounds__(NW * kLanes, DIR == kAdjoint && K == 6 ? 6 : (NW + 3) / 4) pair_kernel(PairParams P) {
    using V = typename St<T>::V;
    __shared__ PairLds<V, NW> L;
    __shared__ PairPlane<V, NW * K> S;
    const int lane = threadIdx.x & (kLanes - 1);
    const int wv = __builtin_amdgcn_readfirstlane(threadIdx.x / kLanes);
    PairParams Q;
    int tx, ty;
    if (!pick_tile<T>(P, Q, tx, ty)) return;
    if constexpr (LEVELS == 3) tile3<DIR, WAV, T, SCH, NW>(Q, tx, ty, L, S, lane, wv);
    else tile<DIR, WAV, T, SCH, NW, K>(Q, tx, ty, L, S, lane, wv);
}

// ---- launch (host) ----------------------------------------------------------
// `kernel` in work-groups of `waves` waves over tiles of cx x cy blocks (halo
// excluded) of the launch's first level.
template <typename T>
hipError_t launch_tiles(void (*kernel)(PairParams), int cx, int cy, int waves, PairParams p, int planes, hipStream_t s) {
    p.tiles_x = ((p.w + 1) / 2 + cx - 1) / cx;
    p.tiles_y = ((p.h + 1) / 2 + cy - 1) / cy;
    // the tiles of all planes; planes beyond what one launch may have go to further ones
    return for_each_launch((int64_t)p.tiles_x * p.tiles_y, (int64_t)kRemapRows * p.tiles_x, waves, planes,
                           [&](int64_t p0, int32_t n, Deal deal) {
        PairParams q = p;
        q.planes = n;
        q.in = static_cast<const T*>(p.in) + p0 * p.in_ps;
        q.out = static_cast<T*>(p.out) + p0 * p.out_ps;
        q.ll = static_cast<T*>(p.ll) + p0 * p.ll_ps;
        q.chunk = (int32_t)deal.chunk;
        hipLaunchKernelGGL(kernel, dim3((unsigned)deal.grid), dim3(waves * kLanes), 0, s, q);
        return hipGetLastError();
    });
}
template <int DIR, int WAV, typename T, int SCH, int NW, int K, int LEVELS = 2>
hipError_t launch_shape(const PairParams& p, int planes, hipStream_t s) {
    return launch_tiles<T>(pair_kernel<DIR, WAV, T, SCH, NW, K, LEVELS>, LEVELS == 3 ? kTripleCols : kPairCols,
                           NW * K - 2 * (LEVELS == 3 ? kHalo3 : kHalo2), NW, p, planes, s);
}

template <int DIR, int WAV, typename T, int SCH>
hipError_t launch(int levels, const PairParams& p, int planes, hipStream_t s) {
    if (levels == 3) {
        const int rows = triple_rows((Direction)DIR, triple_tiles(p.h, p.w, planes, 48), triple_tiles(p.h, p.w, planes, 64));
        if (rows == 48) return launch_shape<DIR, WAV, T, SCH, 12, kTripleK, 3>(p, planes, s);
        return launch_shape<DIR, WAV, T, SCH, 16, kTripleK, 3>(p, planes, s);
    }
    if (pair_rows((Direction)DIR, sizeof(T), pair_tiles(p.h, p.w, planes, 32), pair_tiles(p.h, p.w, planes, 48),
                  (int64_t)p.h * p.w * planes) == 48)
        return launch_shape<DIR, WAV, T, SCH, 8, 6>(p, planes, s);
    return launch_shape<DIR, WAV, T, SCH, 8, 4>(p, planes, s);
}

// The default schemes: fused steps for 4-byte samples and for the adjoint,
// factored ones for 16-bit storage.
template <int DIR, int WAV, typename T>
hipError_t launch_t(int levels, const PairParams& p, int planes, hipStream_t s) {
    return launch<DIR, WAV, T, (sizeof(T) == 4 || DIR == kAdjoint) ? kSchemeFused : kSchemeFactored>(levels, p, planes, s);
}
template <int DIR, int WAV>
hipError_t launch_float(Dtype dt, int levels, const PairParams& p, int planes, hipStream_t s) {
    switch (dt) {
        case kF32: return launch_t<DIR, WAV, float>(levels, p, planes, s);
        case kBF16: return launch_t<DIR, WAV, __hip_bfloat16>(levels, p, planes, s);
        case kF16: return launch_t<DIR, WAV, __half>(levels, p, planes, s);
        default: return hipErrorInvalidValue;
    }
}
template <int DIR>
hipError_t launch_dir(Wavelet wav, Dtype dt, int levels, const PairParams& p, int planes, hipStream_t s) {
    if (levels != 2 && levels != 3) return hipErrorInvalidValue;
    if (wav == kCdf97) return launch_float<DIR, kCdf97>(dt, levels, p, planes, s);
    if constexpr (DIR != kAdjoint) {
        if (wav == kCdf53) return launch_t<DIR, kCdf53, int32_t>(levels, p, planes, s);
        if (wav == kCdf53Real) return launch_float<DIR, kCdf53Real>(dt, levels, p, planes, s);
    }
    return hipErrorInvalidValue;
}

}  // namespace pair
}  // namespace kern
}  // namespace dwt2
