// bwd_tile.h -- what the bf16 backward passes share: the LDS layout of a
// 64-row tile that is read both as rows and by transpose reads, its direct
// fetch, and the sums over partner rows.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include "bf16_rows.h"
#include "pi_common.h"

namespace pi_attn {
namespace bwd {

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

// acc[dims] += w * those dims of the row
template <int D>
__device__ inline void add_row(f32x16 (&acc)[Tile<D>::DB], const bf16x8 (&f)[Tile<D>::KS], float w, int g) {
    regroup_row(f, g, [&](int db, int i, uint2 raw) __attribute__((always_inline)) {
        acc[db][4 * i + 0] += w * __uint_as_float(raw.x << 16);
        acc[db][4 * i + 1] += w * __uint_as_float(raw.x & 0xffff0000u);
        acc[db][4 * i + 2] += w * __uint_as_float(raw.y << 16);
        acc[db][4 * i + 3] += w * __uint_as_float(raw.y & 0xffff0000u);
    });
}

}  // namespace bwd
}  // namespace pi_attn
