// decode.hip -- one KV-cached decode step of causal pi-Attention, bf16 or
// float32 caches, fp32 arithmetic, D = 64 or 128.
//
// One work-group of one to eight wavefronts per (sequence s, head h); t =
// len_in[s].  The working set W_t (Sec. 3.5, eq. online_ws) is the cache
// window rows max(0,t-k)..t-1, the partner row t-pi (when pi > k and t >= pi)
// and the new row t itself, which is taken from k_new/v_new and also appended
// to the caches.
//
// The window rows are split across the work-group's wavefronts in chunks of
// CH load instructions: a row is covered by LPR lanes with 16-byte loads, so
// one instruction reads 64 / LPR whole rows (coalesced).  Each lane keeps a
// 16-byte slice of q and of the output accumulator; a row's score is the sum
// of its lanes' partial dot products.  Every chunk issues all of its key and
// value loads before using any, to keep many bytes in flight.  The partner
// and the new row form one more load slot of the wavefront whose turn comes
// after the last chunk, issued with its first chunk, so that they cost no
// round trip of their own.  Each wavefront runs its own online softmax; the
// wavefronts are merged in LDS at the end (max, rescaled sums).
//
// What bounds it: HBM reads at large launches, one round trip (lengths, then
// rows) plus the merge at small ones, the wavefronts' own instructions at
// windows of a few rows (a chunk's slots are worked on whether they hold a row
// or not, so short windows take short chunks).  The wavefront rule, the extra
// slot and the loads below together, against four wavefronts of eight slots
// (bf16) and one wavefront, row after row (float32): bf16 12.4 -> 6.5 us at one
// sequence of 32 heads (D = 128, k = 512), 98.9 -> 81.8 us at 64; float32
// 379 -> 167 us at 64.
#include <algorithm>

#include "kernels.h"
#include "pi_common.h"

namespace pi_attn {

namespace {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float f32x4 __attribute__((ext_vector_type(4)));

template <typename T, int D>
struct Row {
    static constexpr int EPL = 16 / (int)sizeof(T);   // elements per lane
    static constexpr int LPR = D / EPL;               // lanes per row
    static constexpr int RPI = 64 / LPR;              // rows per load instruction
};

typedef unsigned raw16 __attribute__((ext_vector_type(4)));

__device__ inline uint4 ld16(const void *p) { return *reinterpret_cast<const uint4 *>(p); }

// A window row's load that does not keep the row in the caches.
__device__ inline uint4 ld16_once(const void *p) {
    return __builtin_bit_cast(uint4, __builtin_nontemporal_load(reinterpret_cast<const raw16 *>(p)));
}

template <typename T>
__device__ inline void to_f32(uint4 u, float (&f)[16 / sizeof(T)]) {
    if constexpr (sizeof(T) == 2) {
        const bf16x8 b = __builtin_bit_cast(bf16x8, u);
#pragma unroll
        for (int i = 0; i < 8; ++i) f[i] = (float)b[i];
    } else {
        const f32x4 b = __builtin_bit_cast(f32x4, u);
#pragma unroll
        for (int i = 0; i < 4; ++i) f[i] = b[i];
    }
}

// Sum over the LPR lanes of a row, left in each of them: xor 1 and 2 inside
// quads, the mirrored half-row (8 lanes), the mirrored row (16), then the
// neighbouring row (32).
template <int LPR>
__device__ inline float row_sum(float x) {
    x += __int_as_float(__builtin_amdgcn_mov_dpp(__float_as_int(x), 0xB1, 0xF, 0xF, false));
    x += __int_as_float(__builtin_amdgcn_mov_dpp(__float_as_int(x), 0x4E, 0xF, 0xF, false));
    x += __int_as_float(__builtin_amdgcn_mov_dpp(__float_as_int(x), 0x141, 0xF, 0xF, false));
    if constexpr (LPR >= 16) x += __int_as_float(__builtin_amdgcn_mov_dpp(__float_as_int(x), 0x140, 0xF, 0xF, false));
    if constexpr (LPR >= 32) x += __shfl_xor(x, 16);
    return x;
}

// CH: load instructions per chunk; ONCE: window rows are not kept in the caches;
// PACED: with few of a wavefront's loads in flight at a time.
template <typename T, int D, bool CLAMP, int WAVES, int CH, bool ONCE, bool PACED>
__global__ __launch_bounds__(64 * WAVES) void decode_kernel(DecodeParams p) {
    using R = Row<T, D>;
    constexpr int LPR = R::LPR, RPI = R::RPI, EPL = R::EPL;
    constexpr int RPC = RPI * CH;   // rows per chunk

    __shared__ float s_m[WAVES], s_l[WAVES];
    __shared__ float s_acc[WAVES][D];

    const int64_t sh = blockIdx.x;
    const DivMod head_of = divmod(blockIdx.x, p.H);
    const int s = (int)head_of.quot, h = (int)head_of.rem;
    const int tid = threadIdx.x, lane = __lane_id();
    const int w = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int sub = lane % LPR, rg = lane / LPR;
    const int t = p.len_in[s];
    T *out = (T *)p.out + sh * D;

    if (t < 0 || t >= p.cap) {
        for (int d = tid; d < D; d += 64 * WAVES) out[d] = (T)NAN;
        if (tid == 0) {
            if (p.lse) p.lse[sh] = NAN;
            if (p.len_out && h == 0) p.len_out[s] = t;
        }
        return;
    }

    T *kc = (T *)p.k_cache + sh * (int64_t)p.cap * D + sub * EPL;
    T *vc = (T *)p.v_cache + sh * (int64_t)p.cap * D + sub * EPL;

    float qf[EPL];
    to_f32<T>(ld16((const T *)p.q_new + sh * D + sub * EPL), qf);

    const FusionBias fb = fusion_bias(p.gate[s * p.gss + h * p.gsh], CLAMP);
    const float c2 = p.scale * kLog2e;

    const int lo = window_lo(t, p.k);
    const int nwin = t - lo;   // cache rows lo + [0, nwin)
    const int nchunks = (nwin + RPC - 1) / RPC;
    const int jp = partner_of(t, p.k, p.pi);

    uint4 kr[CH], vr[CH];
    // Slots past the window read its last row again (and count as zeros below):
    // behind a branch each, every load is waited for before the next few, which
    // is what PACED is for.
    auto load = [&](int ch) __attribute__((always_inline)) {
#pragma unroll
        for (int c = 0; c < CH; ++c) {
            const int i = ch * RPC + c * RPI + rg;
            if constexpr (PACED) {
                const bool in = i < nwin;
                const int64_t off = (int64_t)(lo + i) * D;
                kr[c] = in ? ld16_once(kc + off) : make_uint4(0, 0, 0, 0);
                vr[c] = in ? ld16_once(vc + off) : make_uint4(0, 0, 0, 0);
            } else {
                const int64_t off = (int64_t)(lo + min(i, nwin - 1)) * D;
                kr[c] = ONCE ? ld16_once(kc + off) : ld16(kc + off);
                vr[c] = ONCE ? ld16_once(vc + off) : ld16(vc + off);
            }
        }
    };
    // logit (log2 units) of a row from this lane's part of it
    auto logit = [&](uint4 k, float bias) __attribute__((always_inline)) {
        float kf[EPL];
        to_f32<T>(k, kf);
        float part = 0.0f;
#pragma unroll
        for (int e = 0; e < EPL; ++e) part += qf[e] * kf[e];
        part = row_sum<LPR>(part);
        if constexpr (CLAMP) return fminf(fmaxf(part * p.scale + bias, -p.clamp), p.clamp) * kLog2e;
        return part * c2 + bias * kLog2e;
    };

    float m = -INFINITY, l = 0.0f;
    float acc[EPL];
#pragma unroll
    for (int e = 0; e < EPL; ++e) acc[e] = 0.0f;

    // The slot of the new row (row group 0) and the partner (row group 1).
    const bool extra = w == nchunks % WAVES;   // wave-uniform
    uint4 kx, vx;
    if (extra) {
        const bool par = rg == 1 && jp >= 0;
        kx = ld16(par ? kc + (int64_t)jp * D : (const T *)p.k_new + sh * D + sub * EPL);
        vx = ld16(par ? vc + (int64_t)jp * D : (const T *)p.v_new + sh * D + sub * EPL);
    }
    if (w < nchunks) load(w);
    if (extra) {
        const float v = logit(kx, rg == 1 ? fb.partner : fb.local);
        const bool entry = rg == 0 || (rg == 1 && jp >= 0);
        const float sc = entry ? v : -INFINITY;
        m = sc;
#pragma unroll
        for (int o = LPR; o < 64; o <<= 1) m = fmaxf(m, __shfl_xor(m, o));
        const float pr = __builtin_amdgcn_exp2f(sc - (m == -INFINITY ? 0.0f : m));
        l = pr;
        float vf[EPL];
        to_f32<T>(vx, vf);
        if (entry) {
#pragma unroll
            for (int e = 0; e < EPL; ++e) acc[e] = pr * vf[e];
        }
        // append the new key/value as cache row t (no row read here is row t)
        if (rg == 0) {
            *reinterpret_cast<uint4 *>(kc + (int64_t)t * D) = kx;
            *reinterpret_cast<uint4 *>(vc + (int64_t)t * D) = vx;
        }
    }
    for (int ch = w; ch < nchunks; ch += WAVES) {
        if (ch != w) load(ch);
        float sc[CH];
        float cmax = -INFINITY;
#pragma unroll
        for (int c = 0; c < CH; ++c) {
            const float v = logit(kr[c], fb.local);
            sc[c] = ch * RPC + c * RPI + rg < nwin ? v : -INFINITY;
            cmax = fmaxf(cmax, sc[c]);
        }
#pragma unroll
        for (int o = LPR; o < 64; o <<= 1) cmax = fmaxf(cmax, __shfl_xor(cmax, o));
        const float m_new = fmaxf(m, cmax);
        const float m_use = m_new == -INFINITY ? 0.0f : m_new;
        const float alpha = __builtin_amdgcn_exp2f(m - m_use);
        m = m_new;
        l *= alpha;
#pragma unroll
        for (int e = 0; e < EPL; ++e) acc[e] *= alpha;
        if (!PACED && (ch + 1) * RPC > nwin) {
#pragma unroll
            for (int c = 0; c < CH; ++c)
                if (ch * RPC + c * RPI + rg >= nwin) vr[c] = make_uint4(0, 0, 0, 0);
        }
#pragma unroll
        for (int c = 0; c < CH; ++c) {
            const float pr = __builtin_amdgcn_exp2f(sc[c] - m_use);
            l += pr;
            float vf[EPL];
            to_f32<T>(vr[c], vf);
#pragma unroll
            for (int e = 0; e < EPL; ++e) acc[e] += pr * vf[e];
        }
    }

    // Merge the row groups of the wavefront (lanes with the same sub).
#pragma unroll
    for (int o = LPR; o < 64; o <<= 1) {
        l += __shfl_xor(l, o);
#pragma unroll
        for (int e = 0; e < EPL; ++e) acc[e] += __shfl_xor(acc[e], o);
    }
    if (rg == 0) {
#pragma unroll
        for (int e = 0; e < EPL; ++e) s_acc[w][sub * EPL + e] = acc[e];
        if (sub == 0) {
            s_m[w] = m;
            s_l[w] = l;
        }
    }
    __syncthreads();

    for (int d = tid; d < D; d += 64 * WAVES) {
        float M = -INFINITY;
#pragma unroll
        for (int i = 0; i < WAVES; ++i) M = fmaxf(M, s_m[i]);
        float L = 0.0f, o = 0.0f;
#pragma unroll
        for (int i = 0; i < WAVES; ++i) {
            const float f = s_m[i] == -INFINITY ? 0.0f : __builtin_amdgcn_exp2f(s_m[i] - M);
            L += s_l[i] * f;
            o += s_acc[i][d] * f;
        }
        out[d] = (T)(o / L);
        if (d == 0) {
            if (p.lse) p.lse[sh] = (M + __log2f(L)) * kLn2 + fb.lse_shift;
            if (p.len_out && h == 0) p.len_out[s] = t + 1;
        }
    }
}

// ONCE, by the bytes of a step's window rows: they are read once, and kept in
// the caches they only push out what is there.  With the caches of several
// layers in turn (more than the last-level cache together), bf16, D = 128, k =
// 512: 26.6 -> 23.5 us at 16 x 32 (s, h) (134 MB a step), 47.8 -> 42.6 us at
// 32 x 32, 91.0 -> 82.6 us at 64 x 32 (5.9 -> 6.5 TB/s).  The rows of a small
// step lie in the L2s at the next one, if nothing else ran, and cost no more
// when kept even if they do not: 5.3 us kept and 5.8 us not at 32 (s, h) (D =
// 64, k = 384, 3 MB), and from 17 MB on the other way round.
constexpr int64_t kKeepBytes = 12 << 20;

template <typename T, int D, bool CLAMP, int WAVES, int CH, bool PACED = false>
hipError_t launch_n(const DecodeParams &p, hipStream_t stream) {
    const int64_t n = (int64_t)p.S * p.H;
    const bool once = 2 * n * std::min(p.k, p.cap) * D * (int64_t)sizeof(T) > kKeepBytes;
    return launch_kernel(once ? decode_kernel<T, D, CLAMP, WAVES, CH, true, PACED>
                              : decode_kernel<T, D, CLAMP, WAVES, CH, false, false>,
                         dim3((unsigned)n), dim3(64 * WAVES), stream, p);
}

// Wavefronts and chunk size, by the window's load instructions (of keys) and
// the launch; each within 8% of the best of one to eight wavefronts of two,
// four and eight slots, caches in turn and the same ones again, from 32 to
// 32768 (s, h), both dtypes, D = 64 and 128.  Against four wavefronts of eight
// slots: a chip full of short windows is bound by its wavefronts (loads <= 2:
// 2.1 to 3 times as fast from 4096 (s, h) on, float32 D = 64, k = 4 at 8192:
// 22 -> 9.4 us; 3 to 8: 1.2 to 1.8 times), a few (s, h) by one wavefront's
// chain (9 to 32 loads at 32 and 256 (s, h): equal to 12% faster), and eight
// wavefronts stream long windows best from 33 loads on (1 to 3% at 4096 (s, h),
// 12% at 32 and 128 loads; below, up to 1.7 times as long).  Of four slots:
// bf16 D = 128 k = 512 at 2048 (s, h) 80.3 to 84 us by the caches' capacity, of
// eight 82.0 to 85, D = 64 k = 300 26.0 and 27.9, 32 (s, h) 6.3 and 6.5;
// float32 D = 128 k = 512 at 2048 the other way round, 164.7 and 163.3.  Where
// long windows are 400 MB and more together (a load instruction is 1 KiB), the
// memory is a little faster when each wavefront has few loads in flight: D =
// 128, k = 512 at 2048 (s, h) 80.5 and 82.2 us, k = 1024 161.6 and 164.3,
// float32 D = 64, k = 512 81.0 and 83.5.  With 268 MB it is the other way round
// (42.9 and 41.2 us, D = 64 42.7 and 41.1), and so with 68 loads, little more
// than a chunk for each wavefront (99.5 and 90.6 us at 4096 (s, h), k = 270).
// A launch has fewer than 2^32 threads: from 2^24 (s, h) on, one wavefront.
template <typename T, int D, bool CLAMP>
hipError_t launch_w(const DecodeParams &p, hipStream_t stream) {
    const int64_t n = (int64_t)p.S * p.H;
    const int loads = (std::min(p.k, p.cap) + Row<T, D>::RPI - 1) / Row<T, D>::RPI;
    if (n >= (1 << 24)) return launch_n<T, D, CLAMP, 1, 2>(p, stream);
    if (loads >= 128 && 2 * n * loads > (400 << 10)) return launch_n<T, D, CLAMP, 8, 8, true>(p, stream);
    if (loads > 32) return launch_n<T, D, CLAMP, 8, 4>(p, stream);
    if (loads > 8 || (loads > 4 && n <= 1024)) return launch_n<T, D, CLAMP, 4, 4>(p, stream);
    if (loads > 2 || n < 2048) return launch_n<T, D, CLAMP, 2, 2>(p, stream);
    return launch_n<T, D, CLAMP, 1, 2>(p, stream);
}

template <typename T>
hipError_t launch_t(const DecodeParams &p, hipStream_t stream) {
    const bool clamp = p.clamp > 0.0f;
    if (p.D == 64) return clamp ? launch_w<T, 64, true>(p, stream) : launch_w<T, 64, false>(p, stream);
    return clamp ? launch_w<T, 128, true>(p, stream) : launch_w<T, 128, false>(p, stream);
}

}  // namespace

hipError_t launch_decode(const DecodeParams &p, bool bf16, hipStream_t stream) {
    if ((int64_t)p.S * p.H == 0) return hipSuccess;
    return bf16 ? launch_t<__bf16>(p, stream) : launch_t<float>(p, stream);
}

}  // namespace pi_attn
