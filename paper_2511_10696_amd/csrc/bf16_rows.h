// bf16_rows.h -- what the banded bf16 kernels share: vector types, products of
// a lane's own row, and the exchange between the halves of a wavefront.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

namespace pi_attn {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef __bf16 bf16x4 __attribute__((ext_vector_type(4)));
typedef short s16x4 __attribute__((ext_vector_type(4)));
typedef float f32x16 __attribute__((ext_vector_type(16)));
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef __attribute__((address_space(3))) s16x4 lds_s16x4;

// The value held by the other half of the wavefront (lane l ^ 32).
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

// A row held as fragments (lane (c, g): dims 16s + 8g + [0, 8)) in the
// accumulator layout: calls add(db, i, raw) with dims 32db + 8i + 4g + [0, 4)
// of the lane's row.  The 8-dim group m = 4db + i, whose half 4g..4g+3 this
// lane needs, is held whole by lane (c, m & 1) in f[m >> 1]; each lane keeps
// its own half of its groups and takes the other half from the other half of
// the wavefront.
template <int KS, typename Add>
__device__ inline void regroup_row(const bf16x8 (&f)[KS], int g, Add add) {
#pragma unroll
    for (int s2 = 0; s2 < KS; ++s2) {
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

}  // namespace pi_attn
