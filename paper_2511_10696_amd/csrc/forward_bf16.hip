// forward_bf16.hip -- banded MFMA forward of pi-Attention, bf16 in, fp32
// accumulate, for head dimension D = 64 or 128, causal or bidirectional.
//
// Work decomposition.  One work-group (4 wavefronts) owns a query tile of
// BM = 128 consecutive positions [t0, t0+128) of one (b, h); wavefront w owns
// the 32 queries q0 = t0 + 32w + [0, 32).  The window keys of the tile,
// [max(0, t0-k), t0+127] (bidirectional: up to t0+127+k), form a band that is
// streamed through LDS in 64-row tiles (two 32-key blocks, aligned to
// multiples of 32); each wavefront works on the blocks that meet its own band
// [q0 - k, q0 + 31] (bidirectional: [q0 - k, q0 + 31 + k]).  Two work-groups
// share a CU, so each SIMD interleaves two wavefronts.
//
// MFMA layout (v_mfma_f32_32x32x16_bf16).  Scores are computed transposed,
// S^T = K Q^T: A = 32 key rows x 16 dims read from LDS, B = Q^T kept in
// registers for the whole tile, C = 32 keys x 32 queries, so lane l holds the
// scores of query l%32 for keys 8i + 4(l/32) + j in accumulator slot 4i+j;
// the softmax row reductions are in-lane plus one exchange between the two
// halves of the wavefront.  The output is O^T = V^T P^T on the same
// instruction: B = P^T is taken straight from the score registers (slots
// 8c..8c+7 feed key chunk c, with the key order permuted inside the chunk)
// and A = V^T comes from the LDS transpose read (ds_read_b64_tr_b16) of the
// row-major value tile, with the same permutation.
//
// Tiles go from global memory straight into LDS (buffer loads with the LDS
// destination, no staging registers), the next tile while the two blocks
// of the current one are consumed, row-major.  K rows have their
// 16-byte chunks XOR-swizzled (chunk ^ (r mod chunks-per-row)): the
// fragment reads (16 lanes, 16 rows, one chunk each) hit 16 distinct groups
// of 4 banks.  V rows are padded by 64 bytes at D = 128: the transpose reads
// (4 rows, 64 bytes each per 32 lanes) then hit 64 distinct banks, whereas a
// chunk swizzle (chunk ^ 2(r mod 4), kept at D = 64, whose LDS budget has no
// room for padding) leaves them two-way conflicted when the LDS serves
// 8-byte reads 32 lanes at a time (23.9% conflict cycles by the counters at
// fwd32k, none with the padding, same time; what the counters show now, 7.6%,
// is the store staging at the end).  The global side uses buffer loads whose
// descriptor range ends at the tile's last usable row: the hardware range
// check zero-fills rows past it, and offsets are 32-bit with no per-load
// clamping or 64-bit address arithmetic.
//
// The long-range partner (Sec. 3.4, eq. Npi; Sec. 3.5, eq. online_ws): the
// partner rows of a wavefront's 32 queries are 32 consecutive rows shifted by
// pi, read straight from global memory in the layout of the query fragments.
// Its score (a per-lane dot product of the two) seeds the online softmax:
// running max = partner logit, running sum = 1, accumulator = partner value.
// The bidirectional mode scores the second partner t + pi the same way and
// seeds the state with both.
//
// Online softmax with a lazily updated maximum: a lane raises its reference
// maximum m only when a block's maximum exceeds it by more than 2^8 (exp2
// units); otherwise probabilities exp2(s - m) <= 256 are accumulated against
// the stale m, which changes nothing in exact arithmetic (numerator and
// denominator share the reference) and keeps the rescale of the accumulators
// out of the common path.
//
// Normalisation.  The value product takes the probabilities rounded to bf16,
// so the output is divided by the sum of those rounded values (accumulated
// with v_dot2c_f32_bf16, two per instruction): the weights actually applied
// to V sum to one, and a query whose attention sits on one key returns that
// key's value row exactly, whatever the rounding of its stale-maximum
// probability.  The lse, when requested, is taken from a second, fp32 sum of
// the unrounded values (a separate instantiation keeps it off the common
// path).
#include <algorithm>

#include "bf16_rows.h"
#include "kernels.h"
#include "pi_common.h"

namespace pi_attn {

namespace {

typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));

constexpr int WAVES = 4;
constexpr int NT = 64 * WAVES;   // threads per work-group
constexpr int BM = 32 * WAVES;   // queries per work-group
constexpr int TK = 64;           // key rows per LDS tile (two 32-key blocks)
constexpr float kTau = 8.0f;     // lazy-max threshold, log2 units

template <int D>
struct Tile {
    static constexpr int CPR = D / 8;   // 16-byte chunks per row
    static constexpr int ROW_BYTES = 2 * D;
    static constexpr int BYTES = TK * ROW_BYTES;
    // V rows: padded by 64 bytes at D = 128 (not swizzled), XOR-swizzled at D = 64
    static constexpr bool VPAD = D == 128;
    static constexpr int VROW = VPAD ? 2 * D + 64 : 2 * D;
    static constexpr int VBYTES = TK * VROW;
};

// One LDS tile buffer: 64 key rows and 64 value rows.  The kernel declares
// two of them (double buffering) as separate objects.
template <int D>
struct TileBuf {
    alignas(16) unsigned char k[Tile<D>::BYTES];
    alignas(16) unsigned char v[Tile<D>::VBYTES];
};

__device__ inline int k_swz(int row, int chunk, int cpr) { return chunk ^ (row & (cpr - 1)); }
__device__ inline int v_swz(int row, int chunk) { return chunk ^ ((row & 3) << 1); }


// Fetch tile rows [row0, row0 + TK) (counted from the window start) into
// LDS buffer tb with buffer loads that write LDS directly: 16 bytes per
// lane, the 64 lanes of one instruction filling 1 KB of consecutive LDS,
// each lane's source offset chosen so that the bytes land in the tile's
// layout.  Instruction u fills bytes [1024u, 1024u + 1024) of the K or the V
// buffer; wavefront w issues u = w, w + WAVES, ...  K: LDS chunk pc of row r
// holds global chunk k_swz(r, pc).  V: D = 128 rows are padded to VROW and
// the pad chunks take an out-of-range offset (written as zeros); D = 64 rows
// hold global chunk v_swz(r, pc) at chunk pc.  Offsets past the rows the
// descriptor covers read as zeros.
template <int D>
struct Fetch {
    static constexpr int KI = TK * Tile<D>::CPR / 64;   // instructions per K tile
    static constexpr int VU = Tile<D>::VROW / 16;       // LDS chunks per V row
    static constexpr int VI = TK * VU / 64;             // instructions per V tile
};

template <int D>
__device__ inline void tile_fetch(TileBuf<D> &tb, u32x4 rk, u32x4 rv, int rowb, int row0, int w, int lane) {
    using T = Tile<D>;
    using F = Fetch<D>;
    static_assert(F::KI % WAVES == 0 && TK * T::CPR % 64 == 0 && TK * F::VU % 64 == 0, "tile fetch shape");
#pragma unroll
    for (int u0 = 0; u0 < F::KI; u0 += WAVES) {
        const int u = u0 + w, pidx = 64 * u + lane;
        const int row = pidx / T::CPR, pc = pidx % T::CPR;
        const int off = (row0 + row) * rowb + k_swz(row, pc, T::CPR) * 16;
        lds_fetch16(rk, off, tb.k + 1024 * u);
    }
#pragma unroll
    for (int u0 = 0; u0 < F::VI; u0 += WAVES) {
        const int u = u0 + w;
        if (u < F::VI) {   // wave-uniform
            const int pidx = 64 * u + lane;
            const int row = pidx / F::VU, pc = pidx % F::VU;
            const int off = T::VPAD ? (pc < T::CPR ? (row0 + row) * rowb + pc * 16 : kOutOfRange)
                                    : (row0 + row) * rowb + v_swz(row, pc) * 16;
            lds_fetch16(rv, off, tb.v + 1024 * u);
        }
    }
}

__device__ inline float max16(const f32x16 &a) {
    float m0 = fmaxf(fmaxf(a[0], a[1]), a[2]), m1 = fmaxf(fmaxf(a[3], a[4]), a[5]);
    float m2 = fmaxf(fmaxf(a[6], a[7]), a[8]), m3 = fmaxf(fmaxf(a[9], a[10]), a[11]);
    float m4 = fmaxf(fmaxf(a[12], a[13]), a[14]);
    return fmaxf(fmaxf(fmaxf(m0, m1), fmaxf(m2, m3)), fmaxf(m4, a[15]));
}

// Per-wavefront state: lane (c, g) = (l % 32, l / 32) belongs to query q0 + c.
template <int D>
struct Wave {
    static constexpr int DB = D / 32;   // 32-dim output blocks
    static constexpr int KS = D / 16;   // 16-dim k-steps of the score MFMA
    bf16x8 qf[KS];                      // B operand: Q[t][16s + 8g .. +8]
    f32x16 o[DB];                       // O^T accumulators: dims 32db + 8i + 4g + j
    float m;                            // reference (lazy) maximum, log2 units
    float l;                            // this lane's part of the running sum (kept for the lse)
    float lb;                           // the same sum over the bf16-rounded probabilities
};

// s + the sum of the eight bf16 values of p.
__device__ inline float sum_bf16x8(const bf16x8 &p, float s) {
    const bf16x2 one = {(__bf16)1.0f, (__bf16)1.0f};
    s = __builtin_amdgcn_fdot2_f32_bf16(__builtin_shufflevector(p, p, 0, 1), one, s, false);
    s = __builtin_amdgcn_fdot2_f32_bf16(__builtin_shufflevector(p, p, 2, 3), one, s, false);
    s = __builtin_amdgcn_fdot2_f32_bf16(__builtin_shufflevector(p, p, 4, 5), one, s, false);
    s = __builtin_amdgcn_fdot2_f32_bf16(__builtin_shufflevector(p, p, 6, 7), one, s, false);
    return s;
}

// Scores of one 32-key block -> log2-unit logits (masked to -inf on edge
// blocks), running state update, and bf16 probabilities for the value product.
template <int D, bool CLAMP, bool BIDIR, bool LSE>
__device__ inline void softmax_block(Wave<D> &ws, f32x16 &s, bool edge, int j0, int t, int kw, int N, bool t_ok,
                                     float c2, float scale, float bias, float clampv, int g, bf16x8 pb[2]) {
    if constexpr (CLAMP) {
#pragma unroll
        for (int e = 0; e < 16; ++e) s[e] = fminf(fmaxf(s[e] * scale + bias, -clampv), clampv) * kLog2e;
    }
    if (edge) {
#pragma unroll
        for (int e = 0; e < 16; ++e) {
            const int j = j0 + 8 * (e >> 2) + 4 * g + (e & 3);
            bool ok;
            if constexpr (BIDIR) {
                ok = t_ok && j < N && j - t <= kw && t - j <= kw;
            } else {
                ok = t_ok && j <= t && j >= t - kw;
            }
            s[e] = ok ? s[e] : -INFINITY;
        }
    }
    float mx = max16(s);
    mx = fmaxf(mx, other_half(mx));
    if constexpr (!CLAMP) mx *= c2;
    // Only lanes whose own maximum moved update their reference (the others
    // scale by exactly 1), so a query's result never depends on the data of
    // the other queries sharing the wavefront.
    const bool need = mx > ws.m + kTau;
    if (__builtin_amdgcn_ballot_w64(need)) {
        const float m_new = need ? mx : ws.m;
        const float alpha = need ? __builtin_amdgcn_exp2f(ws.m - m_new) : 1.0f;
        ws.m = m_new;
        if constexpr (LSE) ws.l *= alpha;
        ws.lb *= alpha;
#pragma unroll
        for (int db = 0; db < Wave<D>::DB; ++db) ws.o[db] *= alpha;
    }
    const float mu = ws.m == -INFINITY ? 0.0f : ws.m;
    float lsum = 0.0f;
#pragma unroll
    for (int c = 0; c < 2; ++c) {
#pragma unroll
        for (int e = 0; e < 8; ++e) {
            float v;
            if constexpr (CLAMP) {
                v = s[8 * c + e] - mu;
            } else {
                v = __builtin_fmaf(s[8 * c + e], c2, -mu);
            }
            const float p = __builtin_amdgcn_exp2f(v);
            if constexpr (LSE) lsum += p;
            pb[c][e] = (__bf16)p;
        }
    }
    if constexpr (LSE) ws.l += lsum;
    ws.lb = sum_bf16x8(pb[1], sum_bf16x8(pb[0], ws.lb));
}

template <int D, bool CLAMP, bool BIDIR, bool LSE, bool FULL, bool HEADS>
__global__ __launch_bounds__(NT, D == 64 ? 4 : 2) void forward_bf16_kernel(FwdParams p, int n_qt, uint32_t n_logical) {
    using T = Tile<D>;
    using W = Wave<D>;
    __shared__ TileBuf<D> tA, tB;
    const uint32_t logical = xcd_remap(blockIdx.x, n_logical);
    if (logical >= n_logical) return;
    const Order o = tile_order<HEADS>(logical, n_qt, p.H);
    const int qt = o.tile, h = o.h, b = o.b;
    const int64_t bh = o.bh;

    const int tid = threadIdx.x;
    const int lane = __lane_id();
    const int w = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int g = lane >> 5, c = lane & 31;
    const int kw = p.k, pi = p.pi;
    // absolute positions: queries [qpos0, NQ), keys and partners below NS
    const int NQ = p.qpos0 + p.N, NS = p.nseq;
    const int t0 = p.qpos0 + qt * BM;
    const int q0 = t0 + 32 * w;   // first query of this wavefront
    const int t = q0 + c;         // this lane's query
    const bool t_ok = t < NQ;

    const int64_t sn = p.sn, ksn = p.ksn;
    // row pointers indexed by absolute position (only rows held are read)
    const __bf16 *qp = (const __bf16 *)p.q + b * p.sb + h * p.sh - (int64_t)p.qpos0 * sn;
    const int64_t kvbase = b * p.ksb + h * p.ksh - (int64_t)p.kvpos0 * ksn;
    const __bf16 *kp = (const __bf16 *)p.k_ptr + kvbase;
    const __bf16 *vp = (const __bf16 *)p.v + kvbase;

    // Window tiles: rows [kb0, kend) in 64-row steps, blocks aligned to 32.
    const int kb0 = window_lo(t0, kw) & ~31;
    const int kend = min(BIDIR ? (int)min((int64_t)t0 + BM + kw, (int64_t)NS) : min(t0 + BM, NQ), p.kvend);
    const int ntiles = (kend - kb0 + TK - 1) / TK;
    // ---- prologue: every load is issued before any is waited for ----------
    // (the query fragments, the gate logit, the partner key/value rows, then
    // the first tile), so the prologue costs one memory round trip.  Causal at
    // D = 128 the compiler moves one of the partners' registers as soon as it is
    // loaded, and the tile's fetch behind them waits a round trip for that.
    // Where a sequence is one query tile, the tile goes before them (45.9 ->
    // 40.6 us at B256 H16 N20 k17, 30.2 -> 29.4 at B64 H16 N128 k32).  Where
    // other tiles' work-groups read the same rows, it stays behind: the partner
    // rows then come from the L2 more often (68.5 and 71.2 us at B4 H16 N4096
    // k128 in [B][N][H][D] storage; bidirectionally, B1 H32 N32768 k512, 763
    // and 773).
    const bool tile_first = D == 128 && !BIDIR && n_qt == 1;
    // Buffer descriptors over rows [kb0, kend) of this head's keys and values,
    // up to the last row's end (row strides may be below D, or 0).
    const int rowb = (int)(2 * ksn);
    const int band = (kend - kb0 - 1) * rowb + T::ROW_BYTES;
    const u32x4 rk = raw_rsrc(kp + (int64_t)kb0 * ksn, band), rv = raw_rsrc(vp + (int64_t)kb0 * ksn, band);

    // Loads use a clamped, always-readable row; lanes without a query or a
    // partner zero the data afterwards.
    W ws;
    const int tq = t_ok ? t : p.qpos0;
    // The query rows.  D = 64: fetched whole into this wavefront's part of the
    // second tile buffer (free until the first barrier) in the key tile's
    // layout, rows past the last query as zeros: eight 128-byte lines an
    // instruction instead of 32 bytes of each of 32 rows (36.5 -> 35.9 us at
    // B4 H16 N4096 k128, 39.2 -> 38.3 us bidirectionally at B8 H12 N2000, 8.3
    // -> 8.1 us at B1 H16 N1000; no gain at D = 128).
    constexpr bool QLDS = D == 64;
    bf16x8 qraw[W::KS];
    unsigned char *qreg = reinterpret_cast<unsigned char *>(&tB) + w * 32 * T::ROW_BYTES;
    if constexpr (QLDS) {
        static_assert(WAVES * 32 * T::ROW_BYTES <= (int)sizeof(TileBuf<D>), "the query rows fit a tile buffer");
        const int rowbq = (int)(2 * sn);
        const u32x4 rq = raw_rsrc(qp + (int64_t)min(q0, NQ - 1) * sn,
                                  q0 < NQ ? (min(32, NQ - q0) - 1) * rowbq + T::ROW_BYTES : 0);
#pragma unroll
        for (int u = 0; u < 32 * T::CPR / 64; ++u) {
            const int pidx = 64 * u + lane, row = pidx / T::CPR, pc = pidx % T::CPR;
            lds_fetch16(rq, row * rowbq + k_swz(row, pc, T::CPR) * 16, qreg + 1024 * u);
        }
    } else {
#pragma unroll
        for (int s = 0; s < W::KS; ++s) qraw[s] = *reinterpret_cast<const bf16x8 *>(qp + tq * sn + 16 * s + 8 * g);
    }
    const float gl = p.gate[b * p.gsb + h * p.gsh + (tq - p.qpos0) * p.gsn];

    if (tile_first && ntiles > 0) tile_fetch<D>(tA, rk, rv, rowb, 0, w, lane);

    // Partner rows: A-operand row c of the wavefront is row q0 + c - pi, the
    // partner of query q0 + c; the accumulator seed is that row's value, of
    // which lane (c, g) holds dims 32db + 8i + 4g + [0, 4).  Both rows are
    // read in the layout of the query fragments (dims 16s + 8g + [0, 8));
    // the value row is then regrouped by an exchange between the two halves
    // of the wavefront (seed_layout).
    const int prow = t - pi;
    const bool has_p = partner_enabled(kw, pi) && prow >= 0 && t_ok;   // depends on c only
    const bool any_p = __builtin_amdgcn_ballot_w64(has_p) != 0;       // wave-uniform
    const int prc = has_p ? prow : p.kvpos0;
    bf16x8 kpf[W::KS], vpf[W::KS];
    if (any_p) {
#pragma unroll
        for (int s = 0; s < W::KS; ++s) {
            kpf[s] = *reinterpret_cast<const bf16x8 *>(kp + prc * ksn + 16 * s + 8 * g);
            vpf[s] = *reinterpret_cast<const bf16x8 *>(vp + prc * ksn + 16 * s + 8 * g);
        }
    }
    // Bidirectional: the second partner t + pi, loaded the same way.
    const bool has_f = BIDIR && t_ok && partner_fwd_of(t, kw, pi, NS) >= 0;
    const bool any_f = BIDIR && __builtin_amdgcn_ballot_w64(has_f) != 0;
    const int frc = has_f ? t + pi : p.kvpos0;
    bf16x8 kff[W::KS], vff[W::KS];
    if (any_f) {
#pragma unroll
        for (int s = 0; s < W::KS; ++s) {
            kff[s] = *reinterpret_cast<const bf16x8 *>(kp + frc * ksn + 16 * s + 8 * g);
            vff[s] = *reinterpret_cast<const bf16x8 *>(vp + frc * ksn + 16 * s + 8 * g);
        }
    }
    if (!tile_first && ntiles > 0) tile_fetch<D>(tA, rk, rv, rowb, 0, w, lane);
    if constexpr (QLDS) {
        __builtin_amdgcn_s_waitcnt(0xF70);   // vmcnt(0): this wavefront's own fetches, read by itself alone
        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup", "local");
#pragma unroll
        for (int s = 0; s < W::KS; ++s)
            ws.qf[s] = *reinterpret_cast<const bf16x8 *>(qreg + c * T::ROW_BYTES + k_swz(c, 2 * s + g, T::CPR) * 16);
    } else {
#pragma unroll
        for (int s = 0; s < W::KS; ++s) ws.qf[s] = t_ok ? qraw[s] : bf16x8{};
    }

    const FusionBias fb = fusion_bias(gl, CLAMP);
    const float c2 = p.scale * kLog2e;
    // Partner logit (log2 units) of this lane's query from the partner rows
    // kf: lane (c, g) holds dims 16s + 8g + [0, 8) of query c and of its
    // partner row, so the score is a per-lane dot product (packed bf16
    // pairs, fp32 sums) plus the other half's.
    auto partner_logit = [&](const bf16x8 (&kf)[W::KS], bool has) {
        float part = 0.0f;
#pragma unroll
        for (int s = 0; s < W::KS; ++s) part = dot_bf16x8(ws.qf[s], has ? kf[s] : bf16x8{}, part);
        const float diag = part + other_half(part);
        float sp;
        if constexpr (CLAMP) {
            sp = fminf(fmaxf(diag * p.scale + fb.partner, -p.clamp), p.clamp) * kLog2e;
        } else {
            sp = diag * c2 + fb.partner * kLog2e;
        }
        return has ? sp : -INFINITY;
    };
    // Seed: running max = the larger partner logit, running sum and
    // accumulator = the partners' weights and weighted values.
    const float sp = any_p ? partner_logit(kpf, has_p) : -INFINITY;
    const float sf = any_f ? partner_logit(kff, has_f) : -INFINITY;
    ws.m = fmaxf(sp, sf);
    const float wp = has_p ? (BIDIR ? __builtin_amdgcn_exp2f(sp - ws.m) : 1.0f) : 0.0f;
    const float wf = has_f ? __builtin_amdgcn_exp2f(sf - ws.m) : 0.0f;
    ws.l = g == 0 ? wp + wf : 0.0f;
    ws.lb = ws.l;   // the partner weights enter the accumulator unrounded
    // Lanes without that partner contribute exactly 0 (their loads read a
    // clamped row whose data is not used, not even multiplied by 0).
    auto seed_layout = [&](const bf16x8 (&vf)[W::KS], uint2 (&vr)[W::DB][4]) {
        regroup_row(vf, g, [&](int db, int i, uint2 raw) __attribute__((always_inline)) { vr[db][i] = raw; });
    };
    auto seed = [&](uint2 (&vr)[W::DB][4], float wt, bool has, bool add) {
#pragma unroll
        for (int db = 0; db < W::DB; ++db) {
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                if (!has) vr[db][i] = make_uint2(0, 0);
                const float e[4] = {__uint_as_float(vr[db][i].x << 16), __uint_as_float(vr[db][i].x & 0xffff0000u),
                                    __uint_as_float(vr[db][i].y << 16), __uint_as_float(vr[db][i].y & 0xffff0000u)};
#pragma unroll
                for (int j = 0; j < 4; ++j) {
                    const float x = BIDIR ? wt * e[j] : e[j];   // causal: the one partner has weight 1
                    ws.o[db][4 * i + j] = add ? ws.o[db][4 * i + j] + x : x;
                }
            }
        }
    };
    uint2 vraw[W::DB][4];
    if (any_p) {
        seed_layout(vpf, vraw);
    } else {
#pragma unroll
        for (int db = 0; db < W::DB; ++db)
#pragma unroll
            for (int i = 0; i < 4; ++i) vraw[db][i] = make_uint2(0, 0);
    }
    seed(vraw, wp, has_p, false);
    if constexpr (BIDIR) {
        uint2 vfraw[W::DB][4];
        if (any_f) {
            seed_layout(vff, vfraw);
        } else {
#pragma unroll
            for (int db = 0; db < W::DB; ++db)
#pragma unroll
                for (int i = 0; i < 4; ++i) vfraw[db][i] = make_uint2(0, 0);
        }
        seed(vfraw, wf, has_f, true);
    }

    // ---- window band -------------------------------------------------------
    // One 32-key block: rows [32 blk, 32 blk + 32) of the tile at kt / vt,
    // keys [j0, j0 + 32).
    auto block = [&](const unsigned char *kt, const unsigned char *vt, int j0, int blk) {
        // Wave-uniform: does the block meet the band, is it wholly inside it?
        const bool act = BIDIR ? j0 < kend && q0 < NQ && j0 - (q0 + 31) <= kw && j0 + 31 >= q0 - kw
                               : j0 < kend && q0 < NQ && j0 <= q0 + 31 && j0 + 31 >= q0 - kw;
        if (!act) return;
        const bool edge = BIDIR ? !(j0 + 31 - q0 <= kw && q0 + 31 - j0 <= kw) || q0 + 31 >= NQ || j0 + 31 >= NS
                                : !(j0 + 31 <= q0 && j0 >= q0 + 31 - kw) || q0 + 31 >= NQ;

        // Fragment reads: the K rows (A operand of the scores) are issued
        // together ahead of the score MFMAs; the V^T reads (A operand of
        // O^T, by transpose reads) go out behind the score MFMAs and land
        // during the softmax.
        const int krow = 32 * blk + c;
        bf16x8 kf[W::KS];
#pragma unroll
        for (int s = 0; s < W::KS; ++s)
            kf[s] = *reinterpret_cast<const bf16x8 *>(kt + krow * T::ROW_BYTES + k_swz(krow, 2 * s + g, T::CPR) * 16);
        __builtin_amdgcn_sched_barrier(0);

        f32x16 sc = {};
#pragma unroll
        for (int s = 0; s < W::KS; ++s) sc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(kf[s], ws.qf[s], sc, 0, 0, 0);
        const int G = lane >> 4, r = (lane >> 2) & 3, qd = lane & 3;
        bf16x8 vf[2][W::DB];
#pragma unroll
        for (int cc = 0; cc < 2; ++cc) {
#pragma unroll
            for (int db = 0; db < W::DB; ++db) {
#pragma unroll
                for (int hh = 0; hh < 2; ++hh) {
                    const int vrow = 32 * blk + 16 * cc + 8 * hh + 4 * g + r;
                    const int chunk = 4 * db + 2 * (G & 1) + (qd >> 1);
                    const unsigned char *src =
                        T::VPAD ? vt + vrow * T::VROW + chunk * 16 + (qd & 1) * 8
                                : vt + vrow * T::ROW_BYTES + v_swz(vrow, chunk) * 16 + (qd & 1) * 8;
                    const bf16x4 y =
                        __builtin_bit_cast(bf16x4, __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s16x4 *)src));
                    vf[cc][db][4 * hh + 0] = y[0];
                    vf[cc][db][4 * hh + 1] = y[1];
                    vf[cc][db][4 * hh + 2] = y[2];
                    vf[cc][db][4 * hh + 3] = y[3];
                }
            }
        }
        bf16x8 pb[2];
        softmax_block<D, CLAMP, BIDIR, LSE>(ws, sc, edge, j0, t, kw, NS, t_ok, c2, p.scale, fb.local, p.clamp, g, pb);
#pragma unroll
        for (int cc = 0; cc < 2; ++cc) {
#pragma unroll
            for (int db = 0; db < W::DB; ++db)
                ws.o[db] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(vf[cc][db], pb[cc], ws.o[db], 0, 0, 0);
        }
    };
    // Tile m (keys kb0 + 64m ..) is in buffer m mod 2.  Before its blocks a
    // wavefront waits for its own fetches of it (the only ones in flight)
    // and the barrier makes every wavefront's share visible; then tile m + 1
    // is fetched into the other buffer, which every wavefront finished
    // reading (tile m - 1) before that barrier, and lands while tile m's two
    // blocks are computed.  The fences around the barrier are LDS-scoped: a
    // work-group fence would also wait for the fetch of the next tile.
    auto tile = [&](const TileBuf<D> &cur, TileBuf<D> &ahead, int m) {
        __builtin_amdgcn_s_waitcnt(0xF70);   // vmcnt(0): this wavefront's fetches of tile m
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup", "local");
        __builtin_amdgcn_s_barrier();
        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup", "local");
        if (m + 1 < ntiles) tile_fetch<D>(ahead, rk, rv, rowb, TK * (m + 1), w, lane);
        block(cur.k, cur.v, kb0 + TK * m, 0);
        block(cur.k, cur.v, kb0 + TK * m + 32, 1);
    };
    // unrolled by two so that every fetch and every read names its buffer
    // statically
    for (int m = 0; m < ntiles; m += 2) {
        tile(tA, tB, m);
        if (m + 1 >= ntiles) break;
        tile(tB, tA, m + 1);
    }

    // ---- normalise and store -----------------------------------------------
    // Lane (c, g) holds dims 32db + 8i + 4g + [0, 4) of query c: stored as they
    // lie, an instruction writes 16 bytes of each of 32 rows.  Launches that
    // fill the chip (FULL) pass each wavefront's rows through a private
    // LDS region and store whole rows, 16 bytes per lane, not kept in the
    // caches: 43.1 -> 37.5 us at B4 H16 N4096 D64 k128 and 43.4 -> 39.5 us
    // bidirectionally at B8 H12 N2000, equal at D = 128; stores as they lie
    // are 2% faster where the latency of one work-group counts (8.3 against
    // 8.5 us at B1 H16 N1000).  Kept in the caches, whole rows take 38.7 and
    // 41.8 us.
    const float lb_tot = ws.lb + other_half(ws.lb);
    const float inv = 1.0f / lb_tot;
    __bf16 *op = (__bf16 *)p.out + b * p.osb + h * p.osh - (int64_t)p.qpos0 * p.osn;
    auto out4 = [&](int db, int i) __attribute__((always_inline)) {
        bf16x4 o4;
#pragma unroll
        for (int j = 0; j < 4; ++j) o4[j] = (__bf16)(ws.o[db][4 * i + j] * inv);
        return o4;
    };
    if constexpr (FULL) {
        // LDS row pitch (bytes): rows shifted by 4 of the 64 banks, so the writes
        // (8 bytes of 32 rows) meet in pairs, where unpadded rows would all meet;
        // the reads run along the rows.  7.6% of the kernel's LDS cycles (D = 128).
        constexpr int P = 2 * D + 16;
        constexpr int LPR = D / 8, RPI = 64 / LPR;        // lanes per row, rows per instruction
        static_assert(2 * 32 * P <= (int)sizeof(TileBuf<D>), "store staging fits a tile buffer");
        __syncthreads();   // every wavefront is done with the tile buffers
        unsigned char *reg = reinterpret_cast<unsigned char *>(w < 2 ? &tA : &tB) + (w & 1) * 32 * P;
#pragma unroll
        for (int db = 0; db < W::DB; ++db)
#pragma unroll
            for (int i = 0; i < 4; ++i)
                *reinterpret_cast<bf16x4 *>(reg + c * P + (32 * db + 8 * i + 4 * g) * 2) = out4(db, i);
#pragma unroll
        for (int v = 0; v < 32 / RPI; ++v) {
            const int r = RPI * v + lane / LPR, ch = lane % LPR;
            const bf16x8 o8 = *reinterpret_cast<const bf16x8 *>(reg + r * P + ch * 16);
            if (q0 + r < NQ)
                __builtin_nontemporal_store(o8, reinterpret_cast<bf16x8 *>(op + (int64_t)(q0 + r) * p.osn + 8 * ch));
        }
    } else if (t_ok) {
#pragma unroll
        for (int db = 0; db < W::DB; ++db)
#pragma unroll
            for (int i = 0; i < 4; ++i)
                *reinterpret_cast<bf16x4 *>(op + (int64_t)t * p.osn + 32 * db + 8 * i + 4 * g) = out4(db, i);
    }
    if constexpr (LSE) {
        const float l_tot = ws.l + other_half(ws.l);
        if (t_ok && g == 0) p.lse[bh * p.N + (t - p.qpos0)] = (ws.m + __log2f(l_tot)) * kLn2 + fb.lse_shift;
    }
}

// Order of the work-groups: the tiles of a head one after the other (they
// share most of their keys), or, at D = 64 in launches that fill the chip, the
// heads of a tile: 36.2 -> 34.4 us at B4 H16 N4096 k128, 39.5 -> 34.7 us
// bidirectionally at B8 H12 N2000 ([B][N][H][D] storage).  The 128 work-groups
// resident on an XCD then hold the band of every head, H times the window's
// rows (256 bytes of K and V each) more than those of one head, beside the 4
// MB of their own rows; past 1 MB more they are read from memory again:
// B2 H16 N8192 k256 (4096 rows) 41.2 us tiles first and 41.3 us heads first,
// k512 58.8 and 60.6; B1 H64 N4096 k64 29.4 and 30.3, k128 33.2 and 37.9, k512
// 58.8 and 75.8; bidirectionally B2 H32 N4096 k64 39.1 and 41.2, k512 99.6 and
// 109.3.  At D = 128 a band is twice the bytes (B1 H32 N32768 k512 487 -> 547
// us), and small launches lose (8.1 -> 8.3 us at B1 H16 N1000).  With the lse a
// backward follows, which starts on the tiles of a head: a training pass at
// the first shape takes 166.6 us in that order and 167.6 us in the other.
constexpr int64_t kHeadsFirstRows = 4096;

template <int D, bool LSE>
constexpr bool heads_first() {
    return D == 64 && !LSE;
}

template <int D, bool CLAMP, bool BIDIR, bool LSE>
hipError_t launch(const FwdParams &p, hipStream_t stream) {
    const int n_qt = (p.N + BM - 1) / BM;
    const int64_t n_logical = (int64_t)p.B * p.H * n_qt;
    if (n_logical == 0) return hipSuccess;
    const int64_t grid = xcd_grid(n_logical);
    // FULL: four work-groups per CU at D = 64; at D = 128, with a tile of at
    // most 40 queries (two wavefronts or one of the four), the barrier and the
    // way through LDS cost more than whole lines save (2 to 6% of a launch at
    // N = 20 and 32, 1 to 5% at 40, equal at 48, 5% gained at 64).
    const bool full = n_logical >= 1024 && (D == 64 || p.N > 40);
    auto kernel = full ? forward_bf16_kernel<D, CLAMP, BIDIR, LSE, true, false>
                       : forward_bf16_kernel<D, CLAMP, BIDIR, LSE, false, false>;
    if constexpr (heads_first<D, LSE>())
        if (full && p.H * (int64_t)std::min(p.k, p.nseq) * (BIDIR ? 2 : 1) <= kHeadsFirstRows)
            kernel = forward_bf16_kernel<D, CLAMP, BIDIR, LSE, true, true>;
    return launch_kernel(kernel, dim3((unsigned)grid), dim3(NT), stream, p, n_qt, (uint32_t)n_logical);
}

template <int D, bool BIDIR, bool LSE>
hipError_t launch_l(const FwdParams &p, hipStream_t stream) {
    return p.clamp > 0.0f ? launch<D, true, BIDIR, LSE>(p, stream) : launch<D, false, BIDIR, LSE>(p, stream);
}

template <int D, bool BIDIR>
hipError_t launch_d(const FwdParams &p, hipStream_t stream) {
    return p.lse ? launch_l<D, BIDIR, true>(p, stream) : launch_l<D, BIDIR, false>(p, stream);
}

}  // namespace

hipError_t launch_forward_bf16(const FwdParams &p, hipStream_t stream) {
    if (p.D == 64) return p.causal ? launch_d<64, false>(p, stream) : launch_d<64, true>(p, stream);
    return p.causal ? launch_d<128, false>(p, stream) : launch_d<128, true>(p, stream);
}

}  // namespace pi_attn
