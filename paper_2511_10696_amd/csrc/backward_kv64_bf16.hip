// backward_kv64_bf16.hip -- MFMA key pass of the backward for bf16 inputs at
// D = 64: dk and dv, fp32 accumulation.
//
// The mirror of the query pass (backward_bf16.hip): a work-group of 4
// wavefronts owns 128 keys [j0, j0 + 128) of one (b, h), wavefront w the 32
// keys kq0 = j0 + 32w + [0, 32); the queries that hold these keys in their
// window, the band [j0, j0 + 127 + k] (key j is in W_t iff j <= t <= j + k,
// Sec. 3.2 eq. Nr; bidirectionally [j0 - k, j0 + 127 + k], |t - j| <= k),
// stream through LDS in 64-row tiles of Q and dL/dy.  Per 32-query block, on
// v_mfma_f32_32x32x16_bf16, lane l holding key l%32 and queries 8i + 4(l/32)
// + j at slot 4i + j:
//   S  = Q K^T        A = Q rows (LDS), B = K^T (registers)
//   dP = dO V^T       A = dO rows (LDS), B = V^T (registers)
//   alpha^ = exp(delta - lse_t),  dS = alpha^ (dP - r_t)   (Sec. 3.5 eq. jac;
//                     0 where the clamp saturates)
//   dV^T += dO^T alpha^,  dK^T += Q^T dS    A by LDS transpose reads
// The query whose partner is key j, t = j + pi (bidirectionally also t =
// j - pi; Sec. 3.4 eq. Npi, pi > k), is read straight from global memory in
// the layout of the key fragments, and its score and dP are per-lane dot
// products (then the other half's).
//
// Why not the wavefront pairs of backward_kv_bf16.hip: at D = 64 one
// wavefront holds both accumulators (64 registers) and both operand blocks
// (32), two wavefronts to a SIMD, so nothing is handed over through LDS, one
// barrier per tile is left of two and 51 KB of LDS instead of 83 let two
// work-groups share a CU.  The arithmetic and its order are the pairs', so
// gradients are the same to the bit whichever kernel forms them.
// Measured against the pairs (causal, bidirectional): 101 -> 73 and 135 -> 93
// us at B4 H16 N4096 k128, 250 -> 173 and 372 -> 260 us at B2 H16 N16384
// k256.  It moves at least 268 MB at the first shape (56 us at the copy rate
// of 4.8 TB/s).  Partner rows read before the band instead of after it: 75
// us.
#include "bwd_tile.h"
#include "kernels.h"
#include "pi_common.h"

namespace pi_attn {

namespace {

using namespace bwd;

constexpr int D = 64;
constexpr int NT = 64 * WAVES;
constexpr int BK = 32 * WAVES;
using T = Tile<D>;
constexpr int KS = T::KS, DB = T::DB;

struct TileBuf {
    alignas(16) unsigned char q[T::BYTES];
    alignas(16) unsigned char o[T::BYTES];
    alignas(16) float lse2[TK];   // (lse_t - lse_shift_t) * log2 e (with the clamp)
    alignas(16) float r[TK];      // row term
    alignas(16) float bias[TK];   // with the clamp: local prior (natural log);
                                  // without: that prior * log2 e - lse2, the exponent offset
};

template <bool CLAMP, bool BIDIR>
__global__ __launch_bounds__(NT, 2) void backward_kv64_bf16_kernel(BwdParams bp, int n_kt, uint32_t n_logical) {
    const FwdParams &p = bp.f;
    __shared__ TileBuf tA, tB;
    const uint32_t logical = xcd_remap(blockIdx.x, n_logical);
    if (logical >= n_logical) return;
    const DivMod tile_of = divmod(logical, n_kt), head_of = divmod(tile_of.quot, p.H);
    const int kt = (int)tile_of.rem, h = (int)head_of.rem, b = (int)head_of.quot;
    const int64_t bh = tile_of.quot;

    const int tid = threadIdx.x;
    const int lane = __lane_id();
    const int w = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int g = lane >> 5, c = lane & 31;
    const int N = p.N, kw = p.k, pi = p.pi;
    // absolute positions: keys [kvpos0, NK) (this pass's keys), query rows
    // held [QS, QE) (their q, dL/dy, lse, row terms and gate)
    const int NK = p.kvpos0 + N, QS = p.qpos0, QE = min(p.qend, p.nseq);
    const int j0 = p.kvpos0 + kt * BK;
    const int kq0 = j0 + 32 * w;
    const int j = kq0 + c;   // this lane's key
    const bool j_ok = j < NK;
    const int jq = j_ok ? j : p.kvpos0;

    // row pointers and per-row arrays indexed by absolute position
    const int64_t sn = p.sn, ksn = p.ksn, osn = bp.osn;
    const __bf16 *qp = (const __bf16 *)p.q + b * p.sb + h * p.sh - (int64_t)QS * sn;
    const __bf16 *op = (const __bf16 *)bp.dout + b * bp.osb + h * bp.osh - (int64_t)QS * osn;
    const int64_t kvbase = b * p.ksb + h * p.ksh - (int64_t)p.kvpos0 * ksn;
    const float *gp = p.gate + b * p.gsb + h * p.gsh - (int64_t)QS * p.gsn;
    const int64_t rbase = bh * (int64_t)(p.qend - QS) - QS;   // lse, row terms [B][H][qend - qpos0]
    const float c2 = p.scale * kLog2e;

    // The band's query rows [band_lo, band_hi); rows before QS (the band of a
    // shard is aligned down) are zero and masked.
    const int band_lo = BIDIR ? window_lo(j0, kw) & ~31 : j0;
    const int band_hi = BIDIR ? (int)min((int64_t)j0 + BK + kw, (int64_t)QE) : (int)min((int64_t)QE, (int64_t)j0 + BK + kw);
    const int ntiles = band_hi > band_lo ? (band_hi - band_lo + TK - 1) / TK : 0;
    const int b0 = max(band_lo, QS);
    const int rowq = (int)(2 * sn), rowo = (int)(2 * osn);
    // up to the last row's end (row strides may be 0)
    const u32x4 rq = raw_rsrc(qp + (int64_t)b0 * sn, (band_hi - b0 - 1) * rowq + 2 * D);
    const u32x4 ro = raw_rsrc(op + (int64_t)b0 * osn, (band_hi - b0 - 1) * rowo + 2 * D);
    auto fetch = [&](TileBuf &tb, int m) __attribute__((always_inline)) {
        const int row0 = band_lo + TK * m - b0;
        fetch_tile<D, BIDIR>(tb.q, rq, rowq, row0, w, lane);
        fetch_tile<D, BIDIR>(tb.o, ro, rowo, row0, w, lane);
    };
    // per-row values of a tile: loaded by the first wavefront a tile ahead,
    // stored once the tile is current
    float st_gl = 0.0f, st_lse = 0.0f, st_r = 0.0f;
    auto load_values = [&](int m) __attribute__((always_inline)) {
        const int t = min(max(band_lo + TK * m + lane, QS), QE - 1);
        st_gl = gp[t * p.gsn];
        st_lse = bp.lse[rbase + t];
        st_r = bp.rowterm[rbase + t];
    };
    auto store_values = [&](TileBuf &tb) __attribute__((always_inline)) {
        const FusionBias fb = fusion_bias(st_gl, CLAMP);
        const float l2 = (st_lse - fb.lse_shift) * kLog2e;
        if constexpr (CLAMP) tb.lse2[lane] = l2;
        tb.r[lane] = st_r;
        tb.bias[lane] = CLAMP ? fb.local : __builtin_fmaf(fb.local, kLog2e, -l2);
    };
    if (ntiles > 0) {
        fetch(tA, 0);
        if (w == 0) load_values(0);
    }

    // K^T and V^T of this wavefront's keys, zero past the last one
    bf16x8 kf[KS], vf[KS];
#pragma unroll
    for (int s = 0; s < KS; ++s) {
        const bf16x8 kx = *reinterpret_cast<const bf16x8 *>((const __bf16 *)p.k_ptr + kvbase + jq * ksn + 16 * s + 8 * g);
        const bf16x8 vx = *reinterpret_cast<const bf16x8 *>((const __bf16 *)p.v + kvbase + jq * ksn + 16 * s + 8 * g);
        kf[s] = j_ok ? kx : bf16x8{};
        vf[s] = j_ok ? vx : bf16x8{};
    }
    f32x16 dk[DB], dv[DB];
#pragma unroll
    for (int db = 0; db < DB; ++db) dk[db] = dv[db] = f32x16{};

    // ---- window band ---------------------------------------------------------
    auto block = [&](const TileBuf &tb, int t0b, int blk) __attribute__((always_inline)) {
        // Wave-uniform: does the block meet these keys' queries, is it wholly
        // inside them?
        const bool act = BIDIR ? t0b < band_hi && kq0 < NK && t0b - (kq0 + 31) <= kw && t0b + 31 >= kq0 - kw
                               : t0b < band_hi && kq0 < NK && t0b - (kq0 + 31) <= kw && t0b + 31 >= kq0;
        if (!act) return;
        const bool edge = BIDIR ? !(t0b + 31 - kq0 <= kw && kq0 + 31 - t0b <= kw) || t0b + 31 >= QE || kq0 + 31 >= NK ||
                                      t0b < QS
                                : !(t0b >= kq0 + 31 && t0b + 31 - kq0 <= kw) || t0b + 31 >= QE || kq0 + 31 >= NK;
        bf16x8 f[KS];
        read_rows<D>(f, tb.q, blk, c, g);
        f32x16 sc = {};
#pragma unroll
        for (int s = 0; s < KS; ++s) sc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(f[s], kf[s], sc, 0, 0, 0);
        read_rows<D>(f, tb.o, blk, c, g);
        f32x16 dp = {};
#pragma unroll
        for (int s = 0; s < KS; ++s) dp = __builtin_amdgcn_mfma_f32_32x32x16_bf16(f[s], vf[s], dp, 0, 0, 0);
        float pr[16];
        bool cut[16];
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            const f32x4 b4 = *reinterpret_cast<const f32x4 *>(tb.bias + 32 * blk + 8 * i + 4 * g);
            if constexpr (CLAMP) {
                const f32x4 l4 = *reinterpret_cast<const f32x4 *>(tb.lse2 + 32 * blk + 8 * i + 4 * g);
#pragma unroll
                for (int x = 0; x < 4; ++x) {
                    const float dl = fminf(fmaxf(sc[4 * i + x] * p.scale + b4[x], -p.clamp), p.clamp);
                    cut[4 * i + x] = fabsf(dl) >= p.clamp;
                    pr[4 * i + x] = __builtin_amdgcn_exp2f(dl * kLog2e - l4[x]);
                }
            } else {
#pragma unroll
                for (int x = 0; x < 4; ++x) {
                    cut[4 * i + x] = false;
                    pr[4 * i + x] = __builtin_amdgcn_exp2f(__builtin_fmaf(sc[4 * i + x], c2, b4[x]));
                }
            }
        }
        float ds[16];
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            const f32x4 r4 = *reinterpret_cast<const f32x4 *>(tb.r + 32 * blk + 8 * i + 4 * g);
#pragma unroll
            for (int x = 0; x < 4; ++x) {
                const float d = pr[4 * i + x] * (dp[4 * i + x] - r4[x]);
                ds[4 * i + x] = cut[4 * i + x] ? 0.0f : d;
            }
        }
        // Edge blocks: the working-set entries of this lane's key j among the
        // block's queries are one run of rows, the window [j, j + k] (|t - j|
        // <= k bidirectionally), cut to the held rows [QS, QE) and to the
        // block; bit r of keep marks row 4g + r of the block (this lane's
        // rows 4g + 8i + x at bit 8i + x), and the other entries are cleared.
        // The empty asm keeps this a branch that interior blocks skip.
        if (edge) {
            asm volatile("" ::: "memory");
            const int lo = max(BIDIR ? j - kw : j, max(QS, t0b));
            const int hi = (int)min((int64_t)j + kw, (int64_t)min(QE - 1, t0b + 31));
            const int n = hi - lo + 1;
            uint32_t keep = !j_ok || n <= 0 ? 0u : n >= 32 ? ~0u : ((1u << n) - 1u) << (lo - t0b);
            keep >>= 4 * g;
#pragma unroll
            for (int e = 0; e < 16; ++e) {   // all bits, or none
                const int bit = __builtin_amdgcn_sbfe((int)keep, 8 * (e >> 2) + (e & 3), 1);
                pr[e] = __int_as_float(__float_as_int(pr[e]) & bit);
                ds[e] = __int_as_float(__float_as_int(ds[e]) & bit);
            }
        }
        bf16x8 pb[2], sb[2];
#pragma unroll
        for (int cc = 0; cc < 2; ++cc)
#pragma unroll
            for (int e = 0; e < 8; ++e) {
                pb[cc][e] = (__bf16)pr[8 * cc + e];
                sb[cc][e] = (__bf16)ds[8 * cc + e];
            }
        bf16x8 ft[2][DB];
        read_cols<D>(ft, tb.o, blk, lane);
#pragma unroll
        for (int cc = 0; cc < 2; ++cc)
#pragma unroll
            for (int db = 0; db < DB; ++db)
                dv[db] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(ft[cc][db], pb[cc], dv[db], 0, 0, 0);
        read_cols<D>(ft, tb.q, blk, lane);
#pragma unroll
        for (int cc = 0; cc < 2; ++cc)
#pragma unroll
            for (int db = 0; db < DB; ++db)
                dk[db] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(ft[cc][db], sb[cc], dk[db], 0, 0, 0);
    };
    // Tile m (queries band_lo + 64m ..) is in buffer m mod 2.  A wavefront
    // waits for its own fetches of it and its row values (the only
    // vector-memory operations in flight here), the barrier makes every
    // wavefront's share visible, and tile m + 1 then goes into the other
    // buffer (last read for tile m - 1, before that barrier).  LDS-scoped
    // fences: a work-group fence would also wait for the fetch of the next
    // tile.
    auto tile = [&](TileBuf &cur, TileBuf &ahead, int m) __attribute__((always_inline)) {
        __builtin_amdgcn_s_waitcnt(0xF70);   // vmcnt(0)
        if (w == 0) store_values(cur);
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup", "local");
        __builtin_amdgcn_s_barrier();
        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup", "local");
        if (m + 1 < ntiles) {
            fetch(ahead, m + 1);
            if (w == 0) load_values(m + 1);
        }
        block(cur, band_lo + TK * m, 0);
        block(cur, band_lo + TK * m + 32, 1);
    };
    // unrolled by two so that every fetch and every read names its buffer
    // statically
    for (int m = 0; m < ntiles; m += 2) {
        tile(tA, tB, m);
        if (m + 1 >= ntiles) break;
        tile(tB, tA, m + 1);
    }

    // ---- partner queries -----------------------------------------------------
    // The query t whose partner is this lane's key (has: it exists and is held).
    auto partner = [&](int t, bool has) __attribute__((always_inline)) {
        if (__builtin_amdgcn_ballot_w64(has) == 0) return;
        const int tc = has ? t : QS;
        bf16x8 qf[KS], of[KS];
#pragma unroll
        for (int s = 0; s < KS; ++s) {
            qf[s] = *reinterpret_cast<const bf16x8 *>(qp + tc * sn + 16 * s + 8 * g);
            of[s] = *reinterpret_cast<const bf16x8 *>(op + tc * osn + 16 * s + 8 * g);
        }
        const FusionBias fb = fusion_bias(gp[tc * p.gsn], CLAMP);
        const float l2 = (bp.lse[rbase + tc] - fb.lse_shift) * kLog2e, rt = bp.rowterm[rbase + tc];
        float sa = 0.0f, da = 0.0f;
#pragma unroll
        for (int s = 0; s < KS; ++s) {
            qf[s] = has ? qf[s] : bf16x8{};
            of[s] = has ? of[s] : bf16x8{};
            sa = dot_bf16x8(qf[s], kf[s], sa);
            da = dot_bf16x8(of[s], vf[s], da);
        }
        const float sd = sa + other_half(sa), dpd = da + other_half(da);
        float pr;
        bool cut = false;
        if constexpr (CLAMP) {
            const float dl = fminf(fmaxf(sd * p.scale + fb.partner, -p.clamp), p.clamp);
            cut = fabsf(dl) >= p.clamp;
            pr = __builtin_amdgcn_exp2f(dl * kLog2e - l2);
        } else {
            pr = __builtin_amdgcn_exp2f(__builtin_fmaf(sd, c2, __builtin_fmaf(fb.partner, kLog2e, -l2)));
        }
        pr = has ? pr : 0.0f;
        add_row<D>(dv, of, pr, g);
        add_row<D>(dk, qf, has && !cut ? pr * (dpd - rt) : 0.0f, g);
    };
    if (partner_enabled(kw, pi)) {
        partner(j + pi, j_ok && pi < QE - j);
        if constexpr (BIDIR) partner(j - pi, j_ok && j - pi >= QS && j - pi < QE);
    }

    // ---- store: lane (c, g) holds dims 32db + 8i + 4g + [0, 4) of key c ----
    // Whole rows: each wavefront passes its 32 rows through a private LDS
    // region (the tile buffers, free once every wavefront has left the loop)
    // and stores 256 contiguous bytes per row, 16 bytes per lane, not kept in
    // the caches (a training pass at B4 H16 N4096 k128: 173 -> 167 us).
    constexpr int P = 4 * D + 16;   // LDS row pitch (bytes): rows shifted by 4 of the 64 banks, as unpadded ones all meet
    static_assert(2 * 32 * P <= (int)sizeof(TileBuf), "store staging fits a tile buffer");
    __syncthreads();
    unsigned char *reg = reinterpret_cast<unsigned char *>(w < 2 ? &tA : &tB) + (w & 1) * 32 * P;
    const int64_t obase = bh * (int64_t)N - p.kvpos0;   // dk, dv [B][H][N]
    auto store = [&](float *dst, const f32x16 (&acc)[DB], float f) __attribute__((always_inline)) {
#pragma unroll
        for (int db = 0; db < DB; ++db)
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                f32x4 a;
#pragma unroll
                for (int x = 0; x < 4; ++x) a[x] = acc[db][4 * i + x] * f;
                *reinterpret_cast<f32x4 *>(reg + c * P + (32 * db + 8 * i + 4 * g) * 4) = a;
            }
#pragma unroll
        for (int v = 0; v < 8; ++v) {
            const int r = 4 * v + (lane >> 4), ch = lane & 15;
            const f32x4 a = *reinterpret_cast<const f32x4 *>(reg + r * P + ch * 16);
            if (kq0 + r < NK) __builtin_nontemporal_store(a, reinterpret_cast<f32x4 *>(dst + (obase + kq0 + r) * D + 4 * ch));
        }
    };
    store(bp.dv, dv, 1.0f);
    store(bp.dk, dk, p.scale);
}

template <bool CLAMP>
hipError_t launch(const BwdParams &p, hipStream_t stream) {
    const int n_kt = (p.f.N + BK - 1) / BK;
    const int64_t n_logical = (int64_t)p.f.B * p.f.H * n_kt;
    return launch_kernel(p.f.causal ? backward_kv64_bf16_kernel<CLAMP, false> : backward_kv64_bf16_kernel<CLAMP, true>,
                         dim3((unsigned)xcd_grid(n_logical)), dim3(NT), stream, p, n_kt,
                         (uint32_t)n_logical);
}

}  // namespace

hipError_t launch_backward_kv64_bf16(const BwdParams &p, hipStream_t stream) {
    return p.f.clamp > 0.0f ? launch<true>(p, stream) : launch<false>(p, stream);
}

}  // namespace pi_attn
