// Register tile kernel for the four-tap steps of DD 13/7 (Section
// "Evaluation"): the predict T_P and update S_U of its one lifting pair, fused or
// as their factors, forward and inverse, FP32 / BF16 / FP16 storage.
//
// Why not the LDS-plane kernel, which also runs them: there every step reads
// about 25 and writes 4 LDS words per block, so LDS bounds it at a quarter of
// the HBM rate.  Here, as in the two-tap tile kernel, a lane holds BPL
// horizontally adjacent blocks for each of its K block rows in VGPRs.  A fused
// step is evaluated as its horizontal sums, which stay inside the wave (DPP),
// and its vertical sums over the lane's own rows; only the two rows below and
// the one above (predict; the mirror image for the update) that belong to
// another wave go through LDS: x0, x1 and the horizontal sum of x0 for the
// predict, x2, x3 and that of x3 for the update.  Every sum is formed in the
// LDS-plane kernel's order, so the results equal that kernel's bit for bit.
//
// The halo is kHalo4 = 3 blocks per side.  Vertically it is recomputed (rows
// of the tile); horizontally it lies in the first and last EL lanes, which load
// and compute but do not store: the four-tap steps need operands three blocks
// away, where the two-tap kernel's packed halo lanes hold two.
//
// 4096^2 FP32, 3 levels forward: 115.6 us a call on the LDS-plane kernel,
// 43.3 on this one; one level of 8192^2 FP32: 300 and 104 forward (5.2 TB/s), 409 and
// 98 inverse (5.5 TB/s): the memory system.  With 16-bit storage the vector units
// bound the fused steps (25 operations per block and step, a quarter of them on
// halo rows), so without a scheme flag it takes their two 1-D factors, 16
// operations (one level of 3 x 2161 x 3841: BF16 forward 27.0, factored 23.5 us,
// inverse 25.8, 22.4; FP16 29.4, 24.3 and 26.7, 23.0).
//
// Tiles touching the image border load the whole-point symmetric extension
// (forward: the reflected pixel; inverse: each subband sample at its
// reflected pixel position).
#include "dwt2_pair.inl"

namespace dwt2 {
namespace kern {
namespace taps4 {

// 4-point Deslauriers-Dubuc predict (offsets -1 .. 2) and update (-2 .. 1).
constexpr float kP[4] = {1.f / 16, -9.f / 16, -9.f / 16, 1.f / 16};
constexpr float kU[4] = {-1.f / 32, 9.f / 32, 9.f / 32, -1.f / 32};
// Scaling (zeta = sqrt(2)): LL * 2, HH * 1/2; exact in FP32.
constexpr float kZ2 = 2.0f, kZ2Inv = 0.5f;

struct Taps { float c0, c1, c2, c3; };
template <bool NEG> constexpr Taps predict_taps() {
    constexpr float s = NEG ? -1.f : 1.f;
    return {s * kP[0], s * kP[1], s * kP[2], s * kP[3]};
}
template <bool NEG> constexpr Taps update_taps() {
    constexpr float s = NEG ? -1.f : 1.f;
    return {s * kU[0], s * kU[1], s * kU[2], s * kU[3]};
}
__device__ __forceinline__ float sum4(Taps t, float a, float b, float c, float d) {
    return fmaf(t.c3, d, fmaf(t.c2, c, fmaf(t.c1, b, t.c0 * a)));
}
// The same over sums that start at zero (the products of two filters).
__device__ __forceinline__ float sum4z(Taps t, float a, float b, float c, float d) {
    return fmaf(t.c3, d, fmaf(t.c2, c, fmaf(t.c1, b, fmaf(t.c0, a, 0.f))));
}

// Component k of block b of the lane's row, -2 <= b < BPL + 2.
template <int BPL>
__device__ __forceinline__ float block_at(const float (&row)[4 * BPL], int b, int k) {
    if (b < -BPL) return from_left(from_left(row[4 * (b + 2 * BPL) + k]));
    if (b < 0) return from_left(row[4 * (b + BPL) + k]);
    if (b < BPL) return row[4 * b + k];
    if (b < 2 * BPL) return from_right(row[4 * (b - BPL) + k]);
    return from_right(from_right(row[4 * (b - 2 * BPL) + k]));
}

// Horizontal sums of component k of one register row: taps at offsets
// FIRST .. FIRST + 3 (FIRST = -1 or -2).
template <int BPL, int FIRST>
__device__ __forceinline__ void row_sums(const float (&row)[4 * BPL], int k, Taps t, float (&s)[BPL]) {
    float x[BPL + 3];                              // blocks FIRST .. BPL + FIRST + 2 of the lane's window
#pragma unroll
    for (int i = 0; i < BPL + 3; ++i) x[i] = block_at<BPL>(row, i + FIRST, k);
#pragma unroll
    for (int b = 0; b < BPL; ++b) s[b] = sum4(t, x[b], x[b + 1], x[b + 2], x[b + 3]);
}

// A row another wave needs: two components and, for the fused steps, the
// horizontal sum of one.
template <int BPL, int SCH> struct EdgeRow {
    float v[SCH == kSchemeFused ? 3 : 2][kLanes][BPL];
};
template <int BPL, int SCH>
__device__ __forceinline__ void put(EdgeRow<BPL, SCH>& E, const float (&row)[4 * BPL], int k0, int lane) {
#pragma unroll
    for (int b = 0; b < BPL; ++b) {
        E.v[0][lane][b] = row[4 * b + k0];
        E.v[1][lane][b] = row[4 * b + k0 + 1];
    }
}
template <int BPL>
__device__ __forceinline__ void put(EdgeRow<BPL, kSchemeFused>& E, const float (&row)[4 * BPL], int k0,
                                    const float (&s)[BPL], int lane) {
    put(E, row, k0, lane);
#pragma unroll
    for (int b = 0; b < BPL; ++b) E.v[2][lane][b] = s[b];
}
template <int BPL, int SCH>
__device__ __forceinline__ void get(const EdgeRow<BPL, SCH>& E, float (&x)[BPL], float (&y)[BPL], int lane) {
#pragma unroll
    for (int b = 0; b < BPL; ++b) {
        x[b] = E.v[0][lane][b];
        y[b] = E.v[1][lane][b];
    }
}
template <int BPL>
__device__ __forceinline__ void get(const EdgeRow<BPL, kSchemeFused>& E, float (&x)[BPL], float (&y)[BPL],
                                    float (&s)[BPL], int lane) {
    get(E, x, y, lane);
#pragma unroll
    for (int b = 0; b < BPL; ++b) s[b] = E.v[2][lane][b];
}

// LDS of one work-group: slot w holds what wave w reads.  near2: the two rows
// on the side the step reads two rows from, near1: the one on the other side.
// The outermost waves' slots without a writer are never stored outputs'
// operands (the tile's halo absorbs them).
template <int NW, int BPL, int SCH> struct Lds {
    EdgeRow<BPL, SCH> near2[NW][2];
    EdgeRow<BPL, SCH> near1[NW];
};

// T_P: x1 += P x0, x2 += P* x0, x3 += P P* x0 + P* x1 + P x2.
template <bool NEG, int NW, int BPL, int K>
__device__ __forceinline__ void predict(float (&a)[K][4 * BPL], Lds<NW, BPL, kSchemeFused>& L, int lane, int wv) {
    constexpr Taps t = predict_taps<NEG>();
    float H[K + 3][BPL];                           // sums of x0, rows -1 .. K + 1 at index row + 1
#pragma unroll
    for (int r = 0; r < K; ++r) row_sums<BPL, -1>(a[r], 0, t, H[r + 1]);
    if (wv > 0) {
        put<BPL>(L.near2[wv - 1][0], a[0], 0, H[1], lane);
        put<BPL>(L.near2[wv - 1][1], a[1], 0, H[2], lane);
    }
    if (wv < NW - 1) put<BPL>(L.near1[wv + 1], a[K - 1], 0, H[K], lane);
    __syncthreads();
    float u0[BPL], u1[BPL], d0[2][BPL], d1[2][BPL];
    get<BPL>(L.near1[wv], u0, u1, H[0], lane);
    get<BPL>(L.near2[wv][0], d0[0], d1[0], H[K + 1], lane);
    get<BPL>(L.near2[wv][1], d0[1], d1[1], H[K + 2], lane);
    // x1 of the row above, before its update
    float up1[BPL];
#pragma unroll
    for (int b = 0; b < BPL; ++b) up1[b] = u1[b];
#pragma unroll
    for (int r = 0; r < K; ++r) {
        float h2[BPL];
        row_sums<BPL, -1>(a[r], 2, t, h2);
#pragma unroll
        for (int b = 0; b < BPL; ++b) {
            const float x0u = r > 0 ? a[r > 0 ? r - 1 : 0][4 * b] : u0[b];
            const float x0d = r + 1 < K ? a[r + 1 < K ? r + 1 : 0][4 * b] : d0[0][b];
            const float x0e = r + 2 < K ? a[r + 2 < K ? r + 2 : 0][4 * b] : d0[r + 2 - K == 1 ? 1 : 0][b];
            const float x1d = r + 1 < K ? a[r + 1 < K ? r + 1 : 0][4 * b + 1] : d1[0][b];
            const float x1e = r + 2 < K ? a[r + 2 < K ? r + 2 : 0][4 * b + 1] : d1[r + 2 - K == 1 ? 1 : 0][b];
            const float x1 = a[r][4 * b + 1];
            const float pp = sum4z(t, H[r][b], H[r + 1][b], H[r + 2][b], H[r + 3][b]);
            a[r][4 * b + 3] = a[r][4 * b + 3] + pp + sum4(t, up1[b], x1, x1d, x1e) + h2[b];
            a[r][4 * b + 1] = x1 + H[r + 1][b];
            a[r][4 * b + 2] = a[r][4 * b + 2] + sum4(t, x0u, a[r][4 * b], x0d, x0e);
            up1[b] = x1;
        }
    }
}

// S_U: x0 += U x1 + U* x2 + U U* x3, x1 += U* x3, x2 += U x3.
template <bool NEG, int NW, int BPL, int K>
__device__ __forceinline__ void update(float (&a)[K][4 * BPL], Lds<NW, BPL, kSchemeFused>& L, int lane, int wv) {
    constexpr Taps t = update_taps<NEG>();
    float H[K + 3][BPL];                           // sums of x3, rows -2 .. K at index row + 2
#pragma unroll
    for (int r = 0; r < K; ++r) row_sums<BPL, -2>(a[r], 3, t, H[r + 2]);
    if (wv < NW - 1) {
        put<BPL>(L.near2[wv + 1][0], a[K - 2], 2, H[K], lane);
        put<BPL>(L.near2[wv + 1][1], a[K - 1], 2, H[K + 1], lane);
    }
    if (wv > 0) put<BPL>(L.near1[wv - 1], a[0], 2, H[2], lane);
    __syncthreads();
    float u2[2][BPL], u3[2][BPL], d2[BPL], d3[BPL];
    get<BPL>(L.near2[wv][0], u2[0], u3[0], H[0], lane);
    get<BPL>(L.near2[wv][1], u2[1], u3[1], H[1], lane);
    get<BPL>(L.near1[wv], d2, d3, H[K + 2], lane);
    // x2 of the row below, before its update
    float dn2[BPL];
#pragma unroll
    for (int b = 0; b < BPL; ++b) dn2[b] = d2[b];
#pragma unroll
    for (int r = K - 1; r >= 0; --r) {
        float h1[BPL];
        row_sums<BPL, -2>(a[r], 1, t, h1);
#pragma unroll
        for (int b = 0; b < BPL; ++b) {
            const float x3v = r > 1 ? a[r > 1 ? r - 2 : 0][4 * b + 3] : u3[r == 1 ? 1 : 0][b];
            const float x3u = r > 0 ? a[r > 0 ? r - 1 : 0][4 * b + 3] : u3[1][b];
            const float x3d = r + 1 < K ? a[r + 1 < K ? r + 1 : 0][4 * b + 3] : d3[b];
            const float x2v = r > 1 ? a[r > 1 ? r - 2 : 0][4 * b + 2] : u2[r == 1 ? 1 : 0][b];
            const float x2u = r > 0 ? a[r > 0 ? r - 1 : 0][4 * b + 2] : u2[1][b];
            const float x2 = a[r][4 * b + 2];
            const float uu = sum4z(t, H[r][b], H[r + 1][b], H[r + 2][b], H[r + 3][b]);
            a[r][4 * b] = a[r][4 * b] + h1[b] + sum4(t, x2v, x2u, x2, dn2[b]) + uu;
            a[r][4 * b + 1] = a[r][4 * b + 1] + sum4(t, x3v, x3u, a[r][4 * b + 3], x3d);
            a[r][4 * b + 2] = x2 + H[r + 2][b];
            dn2[b] = x2;
        }
    }
}

// The same steps as their two 1-D factors (16 operations per block and step, the
// fused form 25): the horizontal one stays inside the wave, the vertical one
// reads the edge rows.  FIRST: the first tap's offset, -1 or -2.
__device__ __forceinline__ float add4(Taps t, float a, float b, float c, float d, float x) {
    return fmaf(t.c3, d, fmaf(t.c2, c, fmaf(t.c1, b, fmaf(t.c0, a, x))));
}
template <int BPL, int FIRST>
__device__ __forceinline__ void add_row(float (&row)[4 * BPL], int from, int to, Taps t) {
    float x[BPL + 3];                              // blocks FIRST .. BPL + FIRST + 2 of the lane's window
#pragma unroll
    for (int i = 0; i < BPL + 3; ++i) x[i] = block_at<BPL>(row, i + FIRST, from);
#pragma unroll
    for (int b = 0; b < BPL; ++b) row[4 * b + to] = add4(t, x[b], x[b + 1], x[b + 2], x[b + 3], row[4 * b + to]);
}

// T_P^H: x1 += P x0, x3 += P x2; T_P^V: x2 += P* x0, x3 += P* x1.
template <bool NEG, int NW, int BPL, int K>
__device__ __forceinline__ void predict(float (&a)[K][4 * BPL], Lds<NW, BPL, kSchemeFactored>& L, int lane, int wv) {
    constexpr Taps t = predict_taps<NEG>();
#pragma unroll
    for (int r = 0; r < K; ++r) {
        add_row<BPL, -1>(a[r], 0, 1, t);
        add_row<BPL, -1>(a[r], 2, 3, t);
    }
    if (wv > 0) {
        put(L.near2[wv - 1][0], a[0], 0, lane);
        put(L.near2[wv - 1][1], a[1], 0, lane);
    }
    if (wv < NW - 1) put(L.near1[wv + 1], a[K - 1], 0, lane);
    __syncthreads();
    float u[2][BPL], d[2][2][BPL];                 // x0, x1 of row -1 and of rows K, K + 1
    get(L.near1[wv], u[0], u[1], lane);
    get(L.near2[wv][0], d[0][0], d[1][0], lane);
    get(L.near2[wv][1], d[0][1], d[1][1], lane);
#pragma unroll
    for (int r = 0; r < K; ++r)
#pragma unroll
        for (int b = 0; b < BPL; ++b)
#pragma unroll
            for (int k = 0; k < 2; ++k) {
                const float x0 = r > 0 ? a[r > 0 ? r - 1 : 0][4 * b + k] : u[k][b];
                const float x2 = r + 1 < K ? a[r + 1 < K ? r + 1 : 0][4 * b + k] : d[k][0][b];
                const float x3 = r + 2 < K ? a[r + 2 < K ? r + 2 : 0][4 * b + k] : d[k][r + 2 - K == 1 ? 1 : 0][b];
                a[r][4 * b + 2 + k] = add4(t, x0, a[r][4 * b + k], x2, x3, a[r][4 * b + 2 + k]);
            }
}

// S_U^H: x0 += U x1, x2 += U x3; S_U^V: x0 += U* x2, x1 += U* x3.
template <bool NEG, int NW, int BPL, int K>
__device__ __forceinline__ void update(float (&a)[K][4 * BPL], Lds<NW, BPL, kSchemeFactored>& L, int lane, int wv) {
    constexpr Taps t = update_taps<NEG>();
#pragma unroll
    for (int r = 0; r < K; ++r) {
        add_row<BPL, -2>(a[r], 1, 0, t);
        add_row<BPL, -2>(a[r], 3, 2, t);
    }
    if (wv < NW - 1) {
        put(L.near2[wv + 1][0], a[K - 2], 2, lane);
        put(L.near2[wv + 1][1], a[K - 1], 2, lane);
    }
    if (wv > 0) put(L.near1[wv - 1], a[0], 2, lane);
    __syncthreads();
    float u[2][2][BPL], d[2][BPL];                 // x2, x3 of rows -2, -1 and of row K
    get(L.near2[wv][0], u[0][0], u[1][0], lane);
    get(L.near2[wv][1], u[0][1], u[1][1], lane);
    get(L.near1[wv], d[0], d[1], lane);
#pragma unroll
    for (int r = K - 1; r >= 0; --r)
#pragma unroll
        for (int b = 0; b < BPL; ++b)
#pragma unroll
            for (int k = 0; k < 2; ++k) {
                const float x0 = r > 1 ? a[r > 1 ? r - 2 : 0][4 * b + 2 + k] : u[k][r == 1 ? 1 : 0][b];
                const float x1 = r > 0 ? a[r > 0 ? r - 1 : 0][4 * b + 2 + k] : u[k][1][b];
                const float x3 = r + 1 < K ? a[r + 1 < K ? r + 1 : 0][4 * b + 2 + k] : d[k][b];
                a[r][4 * b + k] = add4(t, x0, x1, a[r][4 * b + 2 + k], x3, a[r][4 * b + k]);
            }
}

// The tile into registers.  g.cb0: block column of lane 0's first block
// (negative for the first tile of a row).
template <int DIR, typename T, int BPL, int K>
__device__ __forceinline__ void load(float (&a)[K][4 * BPL], const LevelParams& P, const Geo& g, bool interior,
                                     int lane) {
    int rows[2 * K];
#pragma unroll
    for (int i = 0; i < 2 * K; ++i) rows[i] = 2 * g.gr0 + i;
    if (!interior) fold(rows, P.h);
    const int c0 = 2 * g.gcL;
    const bool full = interior || (c0 >= 0 && c0 + 2 * BPL <= P.w);
    int cols[2 * BPL];
#pragma unroll
    for (int i = 0; i < 2 * BPL; ++i) cols[i] = c0 + i;
    if constexpr (DIR == kForward) {
        const T* in = static_cast<const T*>(P.in);
        if (full) {
            const T* const base = in + 2 * g.cb0;
#pragma unroll
            for (int i = 0; i < 2 * K; ++i) {
                float v[2 * BPL];
                load_vec<T, 2 * BPL>(lane_at(base + (int64_t)rows[i] * P.in_pitch,
                                             (uint32_t)lane * (2 * BPL * sizeof(T))), v);
#pragma unroll
                for (int s = 0; s < 2 * BPL; ++s) a[i >> 1][4 * (s >> 1) + 2 * (i & 1) + (s & 1)] = v[s];
            }
        } else {
            pair::fold_both(cols, P.w);
#pragma unroll
            for (int i = 0; i < 2 * K; ++i)
#pragma unroll
                for (int s = 0; s < 2 * BPL; ++s)
                    a[i >> 1][4 * (s >> 1) + 2 * (i & 1) + (s & 1)] =
                        load_at(in + (int64_t)rows[i] * P.in_pitch, cols[s]);
        }
    } else {
        const T* ll = static_cast<const T*>(P.in_ll);
        const T* det = static_cast<const T*>(P.in);
        if (full) {
#pragma unroll
            for (int r = 0; r < K; ++r)
#pragma unroll
                for (int k = 0; k < 4; ++k) {
                    float v[BPL];
                    load_vec<T, BPL>(lane_at(subband_row(ll, P.in_ll_pitch, det, P.in_pitch, g, k,
                                                         rows[2 * r + (k >> 1)] >> 1) + g.cb0,
                                             (uint32_t)lane * (BPL * sizeof(T))), v);
#pragma unroll
                    for (int b = 0; b < BPL; ++b) a[r][4 * b + k] = v[b];
                }
        } else {
            pair::fold_both(cols, P.w);
#pragma unroll
            for (int r = 0; r < K; ++r)
#pragma unroll
                for (int k = 0; k < 4; ++k) {
                    const T* row = subband_row(ll, P.in_ll_pitch, det, P.in_pitch, g, k, rows[2 * r + (k >> 1)] >> 1);
#pragma unroll
                    for (int b = 0; b < BPL; ++b) a[r][4 * b + k] = load_at(row, cols[2 * b + (k & 1)] >> 1);
                }
        }
#pragma unroll
        for (int r = 0; r < K; ++r)
#pragma unroll
            for (int b = 0; b < BPL; ++b) {
                a[r][4 * b] *= kZ2Inv;
                a[r][4 * b + 3] *= kZ2;
            }
    }
}

// The core of the tile to memory.
template <int DIR, typename T, int NW, int BPL, int K, int EL, bool BORDER>
__device__ __forceinline__ void store(float (&a)[K][4 * BPL], const LevelParams& P, const Geo& g, int lane, int wv) {
    if (lane < EL || lane >= kLanes - EL) return;
    auto core_row = [&](int r) { return !(r < kHalo4 && wv == 0) && !(r >= K - kHalo4 && wv == NW - 1); };
    if constexpr (DIR == kForward) {
        T* ll = static_cast<T*>(P.out_ll);
        T* det = static_cast<T*>(P.out);
        T* row[4];
#pragma unroll
        for (int k = 0; k < 4; ++k) row[k] = subband_row(ll, P.out_ll_pitch, det, P.out_pitch, g, k, g.gr0) + g.cb0;
        constexpr bool kBySubband = !BORDER && sizeof(T) == 4;
#pragma unroll
        for (int k0 = 0; k0 < (kBySubband ? 4 : 1); ++k0)
#pragma unroll
            for (int r = 0; r < K; ++r)
#pragma unroll
                for (int k = (kBySubband ? k0 : 0); k < (kBySubband ? k0 + 1 : 4); ++k) {
                    T* const p = lane_at(row[k], (uint32_t)lane * (BPL * sizeof(T)));
                    row[k] += k == 0 ? P.out_ll_pitch : P.out_pitch;
                    if (!core_row(r)) continue;
                    if (BORDER && g.gr0 + r >= (k >= 2 ? g.nOr : g.nEr)) continue;
                    float v[BPL];
#pragma unroll
                    for (int b = 0; b < BPL; ++b)
                        v[b] = k == 0 ? a[r][4 * b] * kZ2 : k == 3 ? a[r][4 * b + 3] * kZ2Inv : a[r][4 * b + k];
                    const int left = BORDER ? ((k & 1) ? g.nOc : g.nEc) - g.gcL : BPL;   // samples to the row's end
                    if (!BORDER || left >= BPL) {
                        store_vec<T, BPL>(p, v);
                    } else {
#pragma unroll
                        for (int b = 0; b + 1 < BPL; ++b)
                            if (b < left) p[b] = St<T>::store(v[b]);
                    }
                }
    } else {
        T* row = static_cast<T*>(P.out) + (int64_t)(2 * g.gr0) * P.out_pitch + 2 * g.cb0;
        const int left = P.w - 2 * g.gcL;
#pragma unroll
        for (int i = 0; i < 2 * K; ++i) {
            T* const p = lane_at(row, (uint32_t)lane * (2 * BPL * sizeof(T)));
            row += P.out_pitch;
            if (!core_row(i >> 1)) continue;
            if (BORDER && 2 * g.gr0 + i >= P.h) continue;
            float v[2 * BPL];
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
}

template <int DIR, typename T, int SCH, int NW, int K, int BPL, int EL>
__global__ void __launch_bounds__(NW * kLanes) taps4_kernel(LevelParams P0) {
    static_assert(K >= kHalo4 && BPL * EL >= kHalo4, "halo within the first and last wave / lanes");
    __shared__ Lds<NW, BPL, SCH> lds;
    const int lane = threadIdx.x & (kLanes - 1);
    const int wv = __builtin_amdgcn_readfirstlane(threadIdx.x / kLanes);
    fetch_params(P0);
    // XCD remap of the tile list (all planes), as in the two-tap tile kernel
    const int nt = P0.tiles_x * P0.tiles_y;
    const int j = (int)(blockIdx.x >> 3);
    const int n = ((j / P0.chunk) * 8 + (int)(blockIdx.x & 7)) * P0.chunk + j % P0.chunk;
    if (n >= nt * P0.planes) return;              // uniform over the work-group
    const int pl = n / nt;
    const int t = n - pl * nt;
    const int ty = t / P0.tiles_x;
    const int tx = t - ty * P0.tiles_x;
    const LevelParams P = plane_params<T>(P0, pl);
    constexpr int CX = (kLanes - 2 * EL) * BPL, CY = NW * K - 2 * kHalo4;
    Geo g;
    g.nEr = (P.h + 1) >> 1; g.nOr = P.h >> 1;
    g.nEc = (P.w + 1) >> 1; g.nOc = P.w >> 1;
    g.cb0 = tx * CX - EL * BPL;
    g.gcL = g.cb0 + BPL * lane;
    g.gr0 = ty * CY - kHalo4 + wv * K;
    // every loaded block inside the image, all four components
    const bool interior = ty > 0 && tx > 0 && (ty + 1) * CY + kHalo4 <= g.nOr && g.cb0 + kLanes * BPL <= g.nOc;
    float a[K][4 * BPL];
    load<DIR, T, BPL, K>(a, P, g, interior, lane);
    if constexpr (DIR == kForward) {
        predict<false, NW, BPL, K>(a, lds, lane, wv);
        __syncthreads();                          // both steps use the same edge rows
        update<false, NW, BPL, K>(a, lds, lane, wv);
    } else {
        update<true, NW, BPL, K>(a, lds, lane, wv);
        __syncthreads();
        predict<true, NW, BPL, K>(a, lds, lane, wv);
    }
    if (interior) store<DIR, T, NW, BPL, K, EL, false>(a, P, g, lane, wv);
    else store<DIR, T, NW, BPL, K, EL, true>(a, P, g, lane, wv);
}

// Tile shapes, one level, us (FP32 forward and inverse 8192^2; BF16 8192^2;
// FP32 256^2), 2 blocks per lane:
//   4 waves x 4 rows: 102.3  98.2;  62.4  58.3;  5.6
//   4 waves x 5 rows: 103.8  97.7;  64.2  56.2;  6.1
//   8 waves x 4 rows: 107.4  95.5;  69.2  57.8;  6.7
//   4 waves x 8 rows: 109.0  96.4;  70.7  57.4;  7.7
// and 4 blocks per lane (4 x 4) 99.2 105.8; 70.9 69.3; 7.6.  Shorter tiles take
// less time from launch to end, taller ones recompute fewer halo rows.
constexpr int kWaves = 4, kBpl = 2, kEdge = 2;
constexpr int kCols = (kLanes - 2 * kEdge) * kBpl;
static_assert(kCols == kCols4 && kWaves == kWaves4 && kWaves * 5 - 2 * kHalo4 == kRows4, "taps4_fits");

template <int DIR, typename T, int SCH, int K>
hipError_t launch_rows(LevelParams p, int planes, hipStream_t s) {
    constexpr int CY = kWaves * K - 2 * kHalo4;
    p.tiles_x = ((p.w + 1) / 2 + kCols - 1) / kCols;
    p.tiles_y = ((p.h + 1) / 2 + CY - 1) / CY;
    return for_each_launch((int64_t)p.tiles_x * p.tiles_y, (int64_t)kRemapRows * p.tiles_x, kWaves, planes,
                           [&](int64_t p0, int32_t n, Deal deal) {
        LevelParams q = from_plane<T>(p, p0);
        q.planes = n;
        q.chunk = (int32_t)deal.chunk;
        hipLaunchKernelGGL((taps4_kernel<DIR, T, SCH, kWaves, K, kBpl, kEdge>), dim3((unsigned)deal.grid),
                           dim3(kWaves * kLanes), 0, s, q);
        return hipGetLastError();
    });
}

// A level whose tiles all run at once (four work-groups on each of 256 CUs)
// takes one tile's time: the shorter tile.  Otherwise the one that recomputes
// fewer halo rows.
template <int DIR, typename T, int SCH>
hipError_t launch_t(const LevelParams& p, int planes, hipStream_t s) {
    const int64_t tiles = (int64_t)(((p.w + 1) / 2 + kCols - 1) / kCols) * (((p.h + 1) / 2 + 9) / 10) * planes;
    return tiles <= 1024 ? launch_rows<DIR, T, SCH, 4>(p, planes, s) : launch_rows<DIR, T, SCH, 5>(p, planes, s);
}

template <int DIR, typename T>
hipError_t launch_scheme(Scheme sch, const LevelParams& p, int planes, hipStream_t s) {
    if (sch == kSchemeFused) return launch_t<DIR, T, kSchemeFused>(p, planes, s);
    if constexpr (sizeof(T) == 2)
        if (sch == kSchemeFactored) return launch_t<DIR, T, kSchemeFactored>(p, planes, s);
    return hipErrorInvalidValue;
}
template <int DIR>
hipError_t launch_dt(Dtype dt, Scheme sch, const LevelParams& p, int planes, hipStream_t s) {
    switch (dt) {
        case kF32: return launch_scheme<DIR, float>(sch, p, planes, s);
        case kBF16: return launch_scheme<DIR, __hip_bfloat16>(sch, p, planes, s);
        case kF16: return launch_scheme<DIR, __half>(sch, p, planes, s);
        default: return hipErrorInvalidValue;
    }
}

// ---- two levels in one launch -------------------------------------------------
// As the two-tap wavelets' (dwt2_pair.inl): a lane's LL samples of level 1 are its
// blocks of level 2.  The halo is 3 blocks of each level, 9 of level 1, rounded up to
// whole blocks of level 2: kHalo4x2 block rows, kEdge4x2 lanes.  The edge rows of
// both levels and the plane that carries a border tile's LL samples share LDS, a
// barrier apart.  For levels whose tiles all run at once (taps4_pair_rows): 512^2
// FP32, 2 levels, 13.4 us in two launches, 10.4 in one; 4096^2, 3 levels, 43.3 and 40.5.
template <int NW, int K, int SCH> union PairLds {
    Lds<NW, 2, SCH> l1;
    Lds<NW, 1, SCH> l2;
    pair::PairPlane<float, NW * K> ll;
};

template <int DIR, typename T, int SCH, int NW, int K>
__global__ void __launch_bounds__(NW * kLanes) pair_kernel(PairParams P0) {
    static_assert(K % 4 == 0 || K == 6, "a wave's rows are whole blocks of level 2, two at least");
    static_assert(2 * kEdge4x2 >= 3 * kHalo4 && kHalo4x2 >= 3 * kHalo4, "halo of both levels");
    constexpr int R = NW * K, K2 = K / 2;
    __shared__ PairLds<NW, K, SCH> L;
    const int lane = threadIdx.x & (kLanes - 1);
    const int wv = __builtin_amdgcn_readfirstlane(threadIdx.x / kLanes);
    PairParams P;
    int tx, ty;
    if (!pair::pick_tile<T>(P0, P, tx, ty)) return;
    Geo g, g2;
    const int h2 = (P.h + 1) >> 1, w2 = (P.w + 1) >> 1;
    g.nEr = h2; g.nOr = P.h >> 1;
    g.nEc = w2; g.nOc = P.w >> 1;
    g2.nEr = (h2 + 1) >> 1; g2.nOr = h2 >> 1;
    g2.nEc = (w2 + 1) >> 1; g2.nOc = w2 >> 1;
    const int r0 = ty * (R - 2 * kHalo4x2) - kHalo4x2;
    g.cb0 = tx * kCols4x2 - 2 * kEdge4x2;
    g.gcL = g.cb0 + 2 * lane;
    g.gr0 = r0 + wv * K;
    g2.cb0 = g.cb0 >> 1;
    g2.gcL = g2.cb0 + lane;
    g2.gr0 = g.gr0 >> 1;
    const bool interior = r0 >= 0 && g.cb0 >= 0 && r0 + R <= g.nOr && g.cb0 + 2 * kLanes <= g.nOc;
    const bool core_lane = lane >= kEdge4x2 && lane < kLanes - kEdge4x2;
    auto plane = [&](int row, int col) -> float& {
        return L.ll.p[pair::clamp_to(row - r0, R)][pair::clamp_to(col - g.cb0, 2 * kLanes)];
    };
    float a[K][8], b[K2][4];
    if constexpr (DIR == kForward) {
        pair::load_image<T, 2, K>(a, static_cast<const T*>(P.in), P.in_pitch, P.h, P.w, g, interior, lane);
        predict<false, NW, 2, K>(a, L.l1, lane, wv);
        __syncthreads();
        update<false, NW, 2, K>(a, L.l1, lane, wv);
        pair::scale_bands<2, K>(a, kZ2, kZ2Inv);
        T* const out = static_cast<T*>(P.out);
        if (core_lane) pair::store_bands<T, 1, kHalo4x2, NW, 2, K>(a, out, 0, out, P.out_pitch, g, lane, wv);
#pragma unroll
        for (int r = 0; r < K2; ++r)
#pragma unroll
            for (int k = 0; k < 4; ++k) b[r][k] = pair::stored<T>(a[2 * r + (k >> 1)][4 * (k & 1)]);
        __syncthreads();
        if (!interior) {
#pragma unroll
            for (int r = 0; r < K2; ++r)
#pragma unroll
                for (int k = 0; k < 4; ++k) L.ll.p[wv * K + 2 * r + (k >> 1)][2 * lane + (k & 1)] = b[r][k];
            __syncthreads();
            int rows[K], cols[2] = {2 * g2.gcL, 2 * g2.gcL + 1};
#pragma unroll
            for (int i = 0; i < K; ++i) rows[i] = 2 * g2.gr0 + i;
            pair::fold_both(rows, h2);
            pair::fold_both(cols, w2);
#pragma unroll
            for (int r = 0; r < K2; ++r)
#pragma unroll
                for (int k = 0; k < 4; ++k) b[r][k] = plane(rows[2 * r + (k >> 1)], cols[k & 1]);
            __syncthreads();
        }
        predict<false, NW, 1, K2>(b, L.l2, lane, wv);
        __syncthreads();
        update<false, NW, 1, K2>(b, L.l2, lane, wv);
        pair::scale_bands<1, K2>(b, kZ2, kZ2Inv);
        T* const ll = static_cast<T*>(P.ll);
        if (core_lane)
            pair::store_bands<T, 0, kHalo4x2 / 2, NW, 1, K2>(b, ll, P.ll_pitch, out, P.out_pitch, g2, lane, wv);
    } else {
        const T* const det = static_cast<const T*>(P.in);
        int rows[2 * K], cols[4], rows2[2 * K2], cols2[2];
        pair::load_bands<T, 0, 1, K2>(b, static_cast<const T*>(P.ll), P.ll_pitch, det, P.in_pitch, h2, w2, g2, interior,
                                      lane, rows2, cols2);
        pair::load_bands<T, 1, 2, K>(a, det, P.in_pitch, det, P.in_pitch, P.h, P.w, g, interior, lane, rows, cols);
        pair::scale_bands<1, K2>(b, kZ2Inv, kZ2);
        update<true, NW, 1, K2>(b, L.l2, lane, wv);
        __syncthreads();
        predict<true, NW, 1, K2>(b, L.l2, lane, wv);
#pragma unroll
        for (int r = 0; r < K2; ++r)
#pragma unroll
            for (int k = 0; k < 4; ++k) a[2 * r + (k >> 1)][4 * (k & 1)] = pair::stored<T>(b[r][k]);
        __syncthreads();
        if (!interior) {
#pragma unroll
            for (int r = 0; r < K; ++r)
#pragma unroll
                for (int c = 0; c < 2; ++c) L.ll.p[wv * K + r][2 * lane + c] = a[r][4 * c];
            __syncthreads();
            pair::reflect_ll<2, K, false>(a, g, P.h, P.w, 1.f, 1.f, plane);
            __syncthreads();
        }
        pair::scale_bands<2, K>(a, kZ2Inv, kZ2);
        update<true, NW, 2, K>(a, L.l1, lane, wv);
        __syncthreads();
        predict<true, NW, 2, K>(a, L.l1, lane, wv);
        if (core_lane) {
            T* const out = static_cast<T*>(P.out);
            if (interior) pair::store_image<T, false, kHalo4x2, NW, 2, K>(a, out, P.out_pitch, P.h, P.w, g, lane, wv);
            else pair::store_image<T, true, kHalo4x2, NW, 2, K>(a, out, P.out_pitch, P.h, P.w, g, lane, wv);
        }
    }
}

template <int DIR, typename T>
hipError_t launch_pair_t(const PairParams& p, int planes, hipStream_t s) {
    constexpr int SCH = sizeof(T) == 4 ? kSchemeFused : kSchemeFactored;
    if constexpr (DIR == kForward && sizeof(T) == 2)
        if (taps4_pair_rows(kForward, sizeof(T), p.h, p.w, planes) == 64)
            return pair::launch_tiles<T>(pair_kernel<DIR, T, SCH, 16, 4>, kCols4x2, 64 - 2 * kHalo4x2, 16, p, planes, s);
    return pair::launch_tiles<T>(pair_kernel<DIR, T, SCH, 8, 6>, kCols4x2, 48 - 2 * kHalo4x2, 8, p, planes, s);
}
template <int DIR>
hipError_t launch_pair_dt(Dtype dt, const PairParams& p, int planes, hipStream_t s) {
    switch (dt) {
        case kF32: return launch_pair_t<DIR, float>(p, planes, s);
        case kBF16: return launch_pair_t<DIR, __hip_bfloat16>(p, planes, s);
        case kF16: return launch_pair_t<DIR, __half>(p, planes, s);
        default: return hipErrorInvalidValue;
    }
}

}  // namespace taps4
}  // namespace kern

hipError_t launch_taps4_pair(Direction dir, Dtype dt, const PairParams& p, int planes, hipStream_t s) {
    if (planes <= 0) return hipSuccess;
    switch (dir) {
        case kForward: return kern::taps4::launch_pair_dt<kForward>(dt, p, planes, s);
        case kInverse: return kern::taps4::launch_pair_dt<kInverse>(dt, p, planes, s);
        default: return hipErrorInvalidValue;
    }
}

hipError_t launch_taps4(Direction dir, Dtype dt, Scheme sch, const LevelParams& p, int planes, hipStream_t s) {
    if (planes <= 0) return hipSuccess;
    switch (dir) {
        case kForward: return kern::taps4::launch_dt<kForward>(dt, sch, p, planes, s);
        case kInverse: return kern::taps4::launch_dt<kInverse>(dt, sch, p, planes, s);
        default: return hipErrorInvalidValue;
    }
}

}  // namespace dwt2
