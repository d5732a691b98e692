// f32_tile.h -- register tiles and working-set blocks shared by the float32
// forward and backward kernels (v_mfma_f32_16x16x4f32, D = 64 or 128).
//
// A wavefront owns a tile of 16 columns (queries, or keys in the key pass)
// and walks the rows (keys, or queries) of their working sets in blocks of
// 16.  Lane l = 16 g + c belongs to column c.  Every operand comes from
// global memory straight into registers, in one of two layouts:
//   RowFrag  lane (c, g) holds dims 16 s + 4 g + [0, 4) of row c.  Product
//            step (s, e) contracts dims 16 s + 4 g + e, so a 16 x D times
//            D x 16 product takes D / 4 instructions and each load
//            instruction reads whole 64-byte segments of 16 rows.
//   ColFrag  lane (c, g) holds dims 64 h + 4 c + [0, 4) of rows 4 g + i: the
//            transposed operand of a product that contracts the block's rows
//            (step i: rows 4 g + i, whose weights are the accumulator slots
//            i of the score product, no exchange between lanes), each load
//            instruction reading 4 rows of 256 contiguous bytes.
// The accumulator of that product, Acc, holds for column c dims
// 64 h + 16 g + 4 r + e at a[4 h + e][r].
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include "kernels.h"
#include "pi_common.h"

namespace pi_attn {
namespace f32 {

typedef float f32x4 __attribute__((ext_vector_type(4)));

constexpr int TILE = 16;
constexpr int WAVES = 4;
constexpr int NT = 64 * WAVES;

template <int D>
struct RowFrag {
    f32x4 x[D / 16];
};

template <int D>
struct ColFrag {
    f32x4 x[4][D / 64];
};

template <int D>
struct Acc {
    f32x4 a[D / 16];
};

template <int D>
__device__ inline void load_row(RowFrag<D> &f, const float *row, int g) {
#pragma unroll
    for (int s = 0; s < D / 16; ++s) f.x[s] = *reinterpret_cast<const f32x4 *>(row + 16 * s + 4 * g);
}

// Rows 4 g + i of the block whose row pointer is row(index in the block).
template <int D, typename RowPtr>
__device__ inline void load_cols(ColFrag<D> &f, RowPtr row, int c, int g) {
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        const float *p = row(4 * g + i) + 4 * c;
#pragma unroll
        for (int h = 0; h < D / 64; ++h) f.x[i][h] = *reinterpret_cast<const f32x4 *>(p + 64 * h);
    }
}

// Scores of the block's 16 rows with the tile's 16 columns: slot r of lane
// (c, g) is <row 4 g + r, column c>.  In chains (an instruction's latency is
// longer than its issue), four of two instructions for every 32 dims at D = 64,
// four of four for every 64 at D = 128, then a tree: the fewer summands round
// one after the other, the smaller the error.  Relative error of dk over
// fourteen problems of k = 8 to 128, D = 64 and 128: with a tree over 64 lanes
// 3.11e-7 and 3.06e-7, four chains over all dims 3.07e-7 and 3.18e-7, this
// 2.99e-7 and 2.97e-7 (chains of two at D = 128 2.92e-7); out, lse, dq and dv
// err less than with either.  us, a backward with four chains over all dims,
// chains of two and of four: B4 H16 N4096 D64 k128 572, 547, -; B2 H16 N8192
// D128 k256 1918, 1977, 1939; B4 H8 N300 D128 k300 127, 137, 131; forwards at
// D = 128 526, 516, 519 and 44.4, 46.4, 44.9.
template <int D, int S0, int N>
__device__ inline f32x4 dot_range(const RowFrag<D> &rows, const RowFrag<D> &cols) {
    if constexpr (N > D / 32) {
        const f32x4 lo = dot_range<D, S0, N / 2>(rows, cols);
        return lo + dot_range<D, S0 + N / 2, N / 2>(rows, cols);
    } else {
        f32x4 sum[4] = {};
#pragma unroll
        for (int s = S0; s < S0 + N; ++s)
#pragma unroll
            for (int e = 0; e < 4; ++e)
                sum[e] = __builtin_amdgcn_mfma_f32_16x16x4f32(rows.x[s][e], cols.x[s][e], sum[e], 0, 0, 0);
        return (sum[0] + sum[1]) + (sum[2] + sum[3]);
    }
}

template <int D>
__device__ inline f32x4 dot_rows(const RowFrag<D> &rows, const RowFrag<D> &cols) {
    return dot_range<D, 0, D / 16>(rows, cols);
}

// This lane's part of <a, b>, summed in 64 bits: it is formed once per
// column, and the gate gradient's sum of ddelta nearly cancels.
template <int D>
__device__ inline double dot_lane(const RowFrag<D> &a, const RowFrag<D> &b) {
    double s = 0.0;
#pragma unroll
    for (int i = 0; i < D / 16; ++i)
#pragma unroll
        for (int e = 0; e < 4; ++e) s = __builtin_fma((double)a.x[i][e], (double)b.x[i][e], s);
    return s;
}

// Sum and maximum over the four lanes of a column.
template <typename T>
__device__ inline T col_sum(T x) {
    x += __shfl_xor(x, 16);
    return x + __shfl_xor(x, 32);
}

__device__ inline float col_max(float x) {
    x = fmaxf(x, __shfl_xor(x, 16));
    return fmaxf(x, __shfl_xor(x, 32));
}

template <int D>
__device__ inline void mma_rows(Acc<D> &acc, const ColFrag<D> &f, const float (&w)[4]) {
#pragma unroll
    for (int i = 0; i < 4; ++i)
#pragma unroll
        for (int h = 0; h < D / 64; ++h)
#pragma unroll
            for (int e = 0; e < 4; ++e)
                acc.a[4 * h + e] =
                    __builtin_amdgcn_mfma_f32_16x16x4f32(f.x[i][h][e], w[i], acc.a[4 * h + e], 0, 0, 0);
}

// acc[column] += sum over the block's rows of w[row] * row, for the entries
// that are in the working set.  w is 0 for the others, but 0 times an element
// that is not finite is not: a block that has such entries (`edge`) is
// checked for them and, if there are any, they are added entry by entry over
// the valid ones (`ok`: bit i for slot i) and enter the product as 0, so that
// a column whose working set has none of them keeps its bits.
template <int D, typename RowPtr>
__device__ inline void add_rows(Acc<D> &acc, const ColFrag<D> &f, const float (&w)[4], bool edge, unsigned ok,
                                RowPtr row, int lane) {
    if (edge) {
        float z = 0.0f;
#pragma unroll
        for (int i = 0; i < 4; ++i)
#pragma unroll
            for (int h = 0; h < D / 64; ++h)
#pragma unroll
                for (int e = 0; e < 4; ++e) z = __builtin_fmaf(f.x[i][h][e], 0.0f, z);
        if (__builtin_amdgcn_ballot_w64(z != 0.0f)) {   // NaN: some element is not finite
            const int c = lane & 15, g = lane >> 4;
#pragma unroll 1
            for (int j = 0; j < TILE; ++j) {
                const int src = c + 16 * (j >> 2);
                float wj = 0.0f;
#pragma unroll
                for (int i = 0; i < 4; ++i) {
                    const float x = __shfl(w[i], src);
                    wj = (j & 3) == i ? x : wj;
                }
                const bool in = (__shfl((int)ok, src) >> (j & 3)) & 1;
                const float *p = row(j) + 16 * g;
#pragma unroll
                for (int h = 0; h < D / 64; ++h)
#pragma unroll
                    for (int r = 0; r < 4; ++r) {
                        const f32x4 v = *reinterpret_cast<const f32x4 *>(p + 64 * h + 4 * r);
#pragma unroll
                        for (int e = 0; e < 4; ++e) {
                            const float a = acc.a[4 * h + e][r];
                            acc.a[4 * h + e][r] = in && !(fabsf(v[e]) < INFINITY) ? __builtin_fmaf(wj, v[e], a) : a;
                        }
                    }
            }
            ColFrag<D> x;
#pragma unroll
            for (int i = 0; i < 4; ++i)
#pragma unroll
                for (int h = 0; h < D / 64; ++h)
#pragma unroll
                    for (int e = 0; e < 4; ++e)
                        x.x[i][h][e] = fabsf(f.x[i][h][e]) < INFINITY ? f.x[i][h][e] : 0.0f;
            mma_rows<D>(acc, x, w);
            return;
        }
    }
    mma_rows<D>(acc, f, w);
}

// Column c's row of the accumulator, times f, to dst (the row's first element).
template <int D>
__device__ inline void store_acc(float *dst, const Acc<D> &acc, float f, int g) {
#pragma unroll
    for (int h = 0; h < D / 64; ++h)
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            f32x4 o;
#pragma unroll
            for (int e = 0; e < 4; ++e) o[e] = acc.a[4 * h + e][r] * f;
            *reinterpret_cast<f32x4 *>(dst + 64 * h + 16 * g + 4 * r) = o;
        }
}

// ---- the blocks of a tile ----------------------------------------------------
// Rows [j, j + 16) of one block, all entries of one kind: the window, the
// rows t0 - pi + [0, 16) of which column c meets row c ("back"), or the rows
// t0 + pi + [0, 16) ("ahead").  Rows may lie outside [0, n): their entries are
// never valid and their loads are clamped.
struct Block {
    int j;
    int kind;   // 0 window, 1 back, 2 ahead
};

// The rows that the columns [c0, c0 + 16) of a sequence of n meet: window
// rows within `below` rows below and `above` rows above a column, then the
// back and ahead blocks.  The forward and the query pass walk keys (below =
// k, above = 0 causal or k); the key pass walks queries (below = 0 causal or
// k, above = k; a query's partner t - pi makes an ahead block).
struct Walk {
    int c0, n, below, above, pi;
    int lo, nwin, total;
    bool back, ahead;

    __device__ Walk(int c0_, int n_, int below_, int above_, int pi_, bool back_, bool ahead_)
        : c0(c0_), n(n_), below(below_), above(above_), pi(pi_) {
        const int last = min(c0 + TILE, n) - 1;
        lo = c0 - below > 0 ? c0 - below : 0;
        const int hi = above >= n - 1 - last ? n - 1 : last + above;
        nwin = (hi - lo) / TILE + 1;
        back = back_ && last >= pi;
        ahead = ahead_ && pi < n - c0;
        total = nwin + (back ? 1 : 0) + (ahead ? 1 : 0);
    }
    __device__ Block block(int i) const {
        if (i < nwin) return Block{lo + TILE * i, 0};
        return (i == nwin && back) ? Block{c0 - pi, 1} : Block{c0 + pi, 2};
    }
    // whether some entry of the block is not in the working set (wave-uniform)
    __device__ bool edge(const Block &b) const {
        return b.kind != 0 || c0 + TILE > n || b.j + TILE > n || c0 + TILE - 1 - b.j > below ||
               b.j + TILE - 1 - c0 > above;
    }
    // entry (row j, column t), t < n
    __device__ bool has(const Block &b, int j, int t) const {
        if (b.kind == 0) return j < n && t - j <= below && j - t <= above;
        return j >= 0 && j < n && (b.kind == 1 ? t - j == pi : j - t == pi);
    }
    __device__ int clamp(int j) const { return min(max(j, 0), n - 1); }
};

// Tiles of a launch: one wavefront per tile, or (SPLIT) the four wavefronts
// of a work-group on one tile, wavefront w taking blocks w, w + 4, ...
//
// Which: a wavefront alone runs its blocks one after the other, so a launch
// with few tiles takes as long as one tile's chain and leaves SIMDs idle.
// Measured (forward, query pass, key pass, us): 32 tiles of k = 32 9.6, 11.9,
// 14.9 alone and 5.8, 6.8, 7.2 split; 256 tiles of k = 256 18.2, 24.9, 36.8
// alone and 9.6, 11.9, 13.1 split; 1024 tiles of k = 32 10.8, 12.8, 16.7 alone
// and 11.2, 20.2, 17.2 split; 8000 tiles of k = 64 57 alone and 75 split
// (forward).  So: split while half the chip's 1024 SIMDs would be idle.
constexpr int64_t kSplitTiles = 512;   // SPLIT up to here

// alpha^ of one entry from its dot product; `cut` when the clamp saturates.
// bias: the entry's prior; shift = (lse_shift - lse) (natural log).
__device__ inline float weight(float dot, float bias, float shift, const FwdParams &f, bool clamp_on, bool &cut) {
    float d = __builtin_fmaf(dot, f.scale, bias);
    cut = false;
    if (clamp_on) {
        d = fminf(fmaxf(d, -f.clamp), f.clamp);
        cut = fabsf(d) >= f.clamp;
    }
    return __builtin_amdgcn_exp2f((d + shift) * kLog2e);
}

inline int64_t tiles_of(int64_t bh, int n) { return bh * ((n + TILE - 1) / TILE); }

}  // namespace f32
}  // namespace pi_attn
