// bwd_tile.h -- what the bf16 backward passes share: the LDS layout of a
// 64-row tile that is read both as rows and by transpose reads, its direct
// fetch, and the per-lane products of the partner rows.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include "pi_common.h"

namespace pi_attn {
namespace bwd {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef __bf16 bf16x4 __attribute__((ext_vector_type(4)));
typedef short s16x4 __attribute__((ext_vector_type(4)));
typedef float f32x16 __attribute__((ext_vector_type(16)));
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef __attribute__((address_space(3))) s16x4 lds_s16x4;

constexpr int WAVES = 4;
constexpr int TK = 64;   // rows per tile

// Rows are padded by 64 bytes and the low two bits of a row's 16-byte chunk
// index are XORed with bits 2-3 of the row, which keeps both the row reads
// (16 rows, one chunk each) and the transpose reads (4 rows, 4 chunks each)
// free of bank conflicts; offsets stay affine in the k-step and in the
// dimension block.
template <int D>
struct Tile {
    static constexpr int CPR = D / 8;         // 16-byte chunks per row
    static constexpr int ROW = 2 * D + 64;    // LDS row stride (bytes)
    static constexpr int BYTES = TK * ROW;
    static constexpr int KS = D / 16;         // k-steps of the score products
    static constexpr int DB = D / 32;         // 32-dim output blocks
};

// Chunk pc of row r sits at chunk pc ^ chunk_x(r).
__device__ inline int chunk_x(int row) { return (row >> 2) & 3; }

// Fetch rows [row0, row0 + TK) (counted from the descriptor's base; negative
// rows and rows past its range read as zeros) into the tile at `lds`:
// instruction u fills bytes [1024u, 1024u + 1024), 16 bytes per lane, each
// lane's source chosen so that the bytes land in the tile's layout (pad
// chunks take an out-of-range offset and are written as zeros); wavefront w
// issues u = w, w + WAVES, ...
template <int D, bool NEG>
__device__ inline void fetch_tile(unsigned char *lds, u32x4 rsrc, int rowb, int row0, int w, int lane) {
    using T = Tile<D>;
    constexpr int U = T::ROW / 16, I = TK * U / 64;   // LDS chunks per row, instructions per tile
    static_assert(TK * U % 64 == 0, "tile fetch shape");
#pragma unroll
    for (int u0 = 0; u0 < I; u0 += WAVES) {
        const int u = u0 + w;
        if (u < I) {   // wave-uniform
            const int pidx = 64 * u + lane, row = pidx / U, pc = pidx % U;
            const bool in = pc < T::CPR && (!NEG || row0 + row >= 0);
            const int off = in ? (row0 + row) * rowb + (pc ^ chunk_x(row)) * 16 : kOutOfRange;
            lds_fetch16(rsrc, off, lds + 1024 * u);
        }
    }
}

__device__ inline float other_half(float x) {
    const auto p = __builtin_amdgcn_permlane32_swap(__float_as_uint(x), __float_as_uint(x), false, false);
    return __uint_as_float(__lane_id() < 32 ? p[1] : p[0]);
}

// acc + <a, b> over eight bf16 pairs (packed products, fp32 sums).
__device__ inline float dot_bf16x8(const bf16x8 &a, const bf16x8 &b, float acc) {
    acc = __builtin_amdgcn_fdot2_f32_bf16(__builtin_shufflevector(a, a, 0, 1), __builtin_shufflevector(b, b, 0, 1),
                                          acc, false);
    acc = __builtin_amdgcn_fdot2_f32_bf16(__builtin_shufflevector(a, a, 2, 3), __builtin_shufflevector(b, b, 2, 3),
                                          acc, false);
    acc = __builtin_amdgcn_fdot2_f32_bf16(__builtin_shufflevector(a, a, 4, 5), __builtin_shufflevector(b, b, 4, 5),
                                          acc, false);
    return __builtin_amdgcn_fdot2_f32_bf16(__builtin_shufflevector(a, a, 6, 7), __builtin_shufflevector(b, b, 6, 7),
                                           acc, false);
}

// Row fragments (A operand: row l%32, dims 16s + 8(l/32)) of 32-row block
// `blk`: chunk (2s + g) ^ x = 2(s ^ (x >> 1)) + (g ^ (x & 1)), x =
// chunk_x(row), so even and odd k-steps have one base each.
template <int D>
__device__ inline void read_rows(bf16x8 f[Tile<D>::KS], const unsigned char *tile, int blk, int c, int g) {
    const int row = 32 * blk + c, x = chunk_x(row);
    const int rb = row * Tile<D>::ROW + 16 * (g ^ (x & 1));
    const int rbo[2] = {rb + 32 * (x >> 1), rb - 32 * (x >> 1)};
#pragma unroll
    for (int s = 0; s < Tile<D>::KS; ++s) f[s] = *reinterpret_cast<const bf16x8 *>(tile + rbo[s & 1] + 32 * s);
}

// Transposed fragments (A operand: dim 32db + l%32, rows 16cc + {4g..4g+3,
// 8+4g..8+4g+3}) of 32-row block `blk` by LDS transpose reads: rows 32 blk +
// 4g + r + 8hh + 16cc, whose chunk_x is g + 2hh.
template <int D>
__device__ inline void read_cols(bf16x8 f[2][Tile<D>::DB], const unsigned char *tile, int blk, int lane) {
    const int g = lane >> 5, G = lane >> 4, r = (lane >> 2) & 3, qd = lane & 3;
    const int jq = 2 * (G & 1) + (qd >> 1);
    const int toff[2] = {(32 * blk + 4 * g + r) * Tile<D>::ROW + 16 * (jq ^ g) + (qd & 1) * 8,
                         (32 * blk + 4 * g + r + 8) * Tile<D>::ROW + 16 * (jq ^ (g + 2)) + (qd & 1) * 8};
#pragma unroll
    for (int cc = 0; cc < 2; ++cc) {
#pragma unroll
        for (int db = 0; db < Tile<D>::DB; ++db) {
#pragma unroll
            for (int hh = 0; hh < 2; ++hh) {
                const unsigned char *src = tile + toff[hh] + 16 * cc * Tile<D>::ROW + 64 * db;
                const bf16x4 y = __builtin_bit_cast(bf16x4, __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s16x4 *)src));
                f[cc][db][4 * hh + 0] = y[0];
                f[cc][db][4 * hh + 1] = y[1];
                f[cc][db][4 * hh + 2] = y[2];
                f[cc][db][4 * hh + 3] = y[3];
            }
        }
    }
}

// A row held as fragments (lane (c, g): dims 16s + 8g + [0, 8)) in the
// accumulator layout: calls add(db, i, raw) with dims 32db + 8i + 4g + [0, 4)
// of the lane's row.  The 8-dim group m = 4db + i, whose half 4g..4g+3 this
// lane needs, is held whole by lane (c, m & 1) in f[m >> 1]; each lane keeps
// its own half of its groups and takes the other half from the other half of
// the wavefront.
template <int D, typename Add>
__device__ inline void regroup_row(const bf16x8 (&f)[Tile<D>::KS], int g, Add add) {
#pragma unroll
    for (int s2 = 0; s2 < Tile<D>::KS; ++s2) {
        const uint4 own = __builtin_bit_cast(uint4, f[s2]);
        // lane g = 0 sends dims 4..7 of its group, lane g = 1 dims 0..3
        const uint2 send = g == 0 ? make_uint2(own.z, own.w) : make_uint2(own.x, own.y);
        const uint2 recv = make_uint2(__float_as_uint(other_half(__uint_as_float(send.x))),
                                      __float_as_uint(other_half(__uint_as_float(send.y))));
        // groups 2 s2 (held by g = 0) and 2 s2 + 1 (held by g = 1)
        const uint2 lo = g == 0 ? make_uint2(own.x, own.y) : recv;   // group 2 s2, dims 4g..4g+3
        const uint2 hi = g == 0 ? recv : make_uint2(own.z, own.w);   // group 2 s2 + 1
#pragma unroll
        for (int half = 0; half < 2; ++half) {
            const int m = 2 * s2 + half;
            add(m >> 2, m & 3, half ? hi : lo);
        }
    }
}

// acc[dims] += w * those dims of the row
template <int D>
__device__ inline void add_row(f32x16 (&acc)[Tile<D>::DB], const bf16x8 (&f)[Tile<D>::KS], float w, int g) {
    regroup_row<D>(f, g, [&](int db, int i, uint2 raw) __attribute__((always_inline)) {
        acc[db][4 * i + 0] += w * __uint_as_float(raw.x << 16);
        acc[db][4 * i + 1] += w * __uint_as_float(raw.x & 0xffff0000u);
        acc[db][4 * i + 2] += w * __uint_as_float(raw.y << 16);
        acc[db][4 * i + 3] += w * __uint_as_float(raw.y & 0xffff0000u);
    });
}

}  // namespace bwd
}  // namespace pi_attn
