// backward_bf16.hip -- MFMA query pass of the backward for bf16 inputs:
// dq and the per-query gate gradient (D = 64 or 128), fp32 accumulation.
//
// Same decomposition and operand layouts as the bf16 forward: a work-group
// of 4 wavefronts owns 128 queries of one (b, h), wavefront w the 32 queries
// q0 = t0 + 32w + [0, 32); the window keys stream through LDS in 64-row
// tiles.  Per 32-key block, on v_mfma_f32_32x32x16_bf16:
//   S^T  = K Q^T        A = K rows (LDS), B = Q^T (registers)
//   dP^T = V dO^T       A = V rows (LDS), B = dO^T (registers)
// which land in the same accumulator layout (lane l: query l%32, keys
// 8i + 4(l/32) + j at slot 4i + j).  The weights come back from the
// forward's lse, alpha^ = exp(delta - lse), and
//   dS^T = alpha^ (dP^T - r_t)     (softmax Jacobian, Sec. 3.5 eq. jac)
// with r_t = <dL/dy_t, y_t> from the forward output (two lanes per query,
// each with half the dims of dL/dy_t and y_t); dS^T, rounded to bf16, is
// the B operand of
//   dQ^T += K^T dS^T    A = K^T by LDS transpose reads of the key tile
// with the key order permuted inside each 16-key chunk exactly as the
// forward permutes V^T against P^T.  The gate gradient
// sum_j dS_tj d(log omega_tj)/dg (eqs. ddelta_da, dalpha_da) nearly cancels
// between window and partner, so it is formed at the end from the exact
// row term r* = sum_j alpha^_tj dP_tj accumulated along the way (the r_t
// used for dS comes from the bf16-rounded forward output): with
// A = sum alpha^ dP and B = sum alpha^ over the unclamped entries of each
// prior, dg = sum_prior d(log omega)/dg (A - r* B).  r* is also written out
// as the row term of the key pass.  The partner
// row (Sec. 3.4, eq. Npi) is read straight from global memory in the layout
// of the query fragments, and its score and dP are per-lane dot products
// (then the other half's), as in the forward; the bidirectional mode
// (window |j - t| <= k, band up to t0 + 127 + k) adds the second partner
// t + pi the same way.
//
// Tiles go from global memory straight into LDS (buffer loads with the LDS
// destination, range-checked so that rows past the query tile's last usable
// row read as zeros), the next tile while the two blocks of the current one
// are consumed.  The key tile is read both as rows and by transpose reads:
// its rows are padded by 64 bytes and the low two bits of a row's 16-byte
// chunk index are XORed with bits 2-3 of the row, which keeps both patterns
// free of bank conflicts; the value tile, read as rows only, has rows padded
// by 16 bytes.
#include "bwd_tile.h"
#include "kernels.h"
#include "pi_common.h"

namespace pi_attn {

namespace {

using namespace bwd;

constexpr int NT = 64 * WAVES;
constexpr int BM = 32 * WAVES;

template <int D>
struct VTile {
    static constexpr int ROW = 2 * D + 16;   // value-tile LDS row stride (bytes)
};

template <int D>
struct TileBuf {
    alignas(16) unsigned char k[Tile<D>::BYTES];
    alignas(16) unsigned char v[TK * VTile<D>::ROW];
};

// Fetch tile rows [row0, row0 + TK) (counted from the window start) into LDS
// buffer tb, the value tile's rows padded by 16 bytes and not swizzled.
template <int D>
__device__ inline void tile_fetch(TileBuf<D> &tb, u32x4 rk, u32x4 rv, int rowb, int row0, int w, int lane) {
    using T = Tile<D>;
    constexpr int VU = VTile<D>::ROW / 16;   // LDS chunks per row
    constexpr int VI = TK * VU / 64;         // instructions per tile
    static_assert(TK * VU % 64 == 0, "tile fetch shape");
    fetch_tile<D, false>(tb.k, rk, rowb, row0, w, lane);
#pragma unroll
    for (int u0 = 0; u0 < VI; u0 += WAVES) {
        const int u = u0 + w;
        if (u < VI) {
            const int pidx = 64 * u + lane, row = pidx / VU, pc = pidx % VU;
            const int off = pc < T::CPR ? (row0 + row) * rowb + pc * 16 : kOutOfRange;
            lds_fetch16(rv, off, tb.v + 1024 * u);
        }
    }
}

// Row fragments (A operand, row l%32, dims 16s + 8(l/32)) of 32-row block
// `blk` of the value tile.
template <int D>
__device__ inline void read_vrows(bf16x8 f[Tile<D>::KS], const unsigned char *tile, int blk, int c, int g) {
    const unsigned char *base = tile + (32 * blk + c) * VTile<D>::ROW + 16 * g;
#pragma unroll
    for (int s = 0; s < Tile<D>::KS; ++s) f[s] = *reinterpret_cast<const bf16x8 *>(base + 32 * s);
}

template <int D, bool CLAMP, bool BIDIR, bool FULL>
__global__ __launch_bounds__(NT, 2) void backward_q_bf16_kernel(BwdParams bp, int n_qt, uint32_t n_logical) {
    using T = Tile<D>;
    constexpr int KS = T::KS, DB = T::DB;
    const FwdParams &p = bp.f;
    __shared__ TileBuf<D> tA, tB;
    const uint32_t logical = xcd_remap(blockIdx.x, n_logical);
    if (logical >= n_logical) return;
    const DivMod tile_of = divmod(logical, n_qt), head_of = divmod(tile_of.quot, p.H);
    const int qt = (int)tile_of.rem, h = (int)head_of.rem, b = (int)head_of.quot;
    const int64_t bh = tile_of.quot;

    const int tid = threadIdx.x;
    const int lane = __lane_id();
    const int w = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int g = lane >> 5, c = lane & 31;
    const int N = p.N, kw = p.k, pi = p.pi;
    // absolute positions: queries [qpos0, NQ), keys and partners below NS
    const int NQ = p.qpos0 + N, NS = p.nseq;
    const int t0 = p.qpos0 + qt * BM;
    const int q0 = t0 + 32 * w;
    const int t = q0 + c;
    const bool t_ok = t < NQ;
    const int tq = t_ok ? t : p.qpos0;
    const int64_t row = bh * N + (tq - p.qpos0);

    // row pointers indexed by absolute position (only rows held are read)
    const int64_t sn = p.sn, ksn = p.ksn;
    const __bf16 *qp = (const __bf16 *)p.q + b * p.sb + h * p.sh - (int64_t)p.qpos0 * sn;
    const int64_t kvbase = b * p.ksb + h * p.ksh - (int64_t)p.kvpos0 * ksn;
    const __bf16 *kp = (const __bf16 *)p.k_ptr + kvbase;
    const __bf16 *vp = (const __bf16 *)p.v + kvbase;
    const __bf16 *op = (const __bf16 *)bp.dout + b * bp.osb + h * bp.osh - (int64_t)p.qpos0 * bp.osn;

    const int kb0 = window_lo(t0, kw) & ~31;
    const int kend = min(BIDIR ? (int)min((int64_t)t0 + BM + kw, (int64_t)NS) : min(t0 + BM, NQ), p.kvend);
    const int ntiles = (kend - kb0 + TK - 1) / TK;
    const int rowb = (int)(2 * ksn);
    // up to the last row's end (row strides may be below D, or 0)
    const int band = (kend - kb0 - 1) * rowb + 2 * D;
    const u32x4 rk = raw_rsrc(kp + (int64_t)kb0 * ksn, band), rv = raw_rsrc(vp + (int64_t)kb0 * ksn, band);
    if (ntiles > 0) tile_fetch<D>(tA, rk, rv, rowb, 0, w, lane);

    // Query and dL/dy rows as B operands (lanes without a query hold zeros).
    bf16x8 qf[KS], of[KS];
#pragma unroll
    for (int s = 0; s < KS; ++s) {
        const bf16x8 qv = *reinterpret_cast<const bf16x8 *>(qp + tq * sn + 16 * s + 8 * g);
        const bf16x8 ov = *reinterpret_cast<const bf16x8 *>(op + tq * bp.osn + 16 * s + 8 * g);
        qf[s] = t_ok ? qv : bf16x8{};
        of[s] = t_ok ? ov : bf16x8{};
    }
    const float gl = p.gate[b * p.gsb + h * p.gsh + (tq - p.qpos0) * p.gsn];
    const FusionBias fb = fusion_bias(gl, CLAMP);
    // r_t = <dL/dy_t, y_t>: this lane's dims 16s + 8g + [0, 8), then the pair
    const __bf16 *yp = (const __bf16 *)bp.out + b * bp.osb + h * bp.osh - (int64_t)p.qpos0 * bp.osn;
    float rpart = 0.0f;
#pragma unroll
    for (int s = 0; s < KS; ++s) {
        const bf16x8 yv = *reinterpret_cast<const bf16x8 *>(yp + tq * bp.osn + 16 * s + 8 * g);
#pragma unroll
        for (int e = 0; e < 8; ++e) rpart += (float)of[s][e] * (float)yv[e];
    }
    const float r = rpart + other_half(rpart);
    const float lse = bp.lse[row];
    // alpha^ = exp2(delta * log2e - lse2), delta with the biases of fb
    const float lse2 = (lse - fb.lse_shift) * kLog2e;
    const float c2 = p.scale * kLog2e;
    const float ga = 1.0f / (1.0f + __expf(-gl));
    const float gat = kGateEps + (1.0f - 2.0f * kGateEps) * ga;
    const float gcoef = (1.0f - 2.0f * kGateEps) * ga * (1.0f - ga);
    const float dlog_local = gcoef / gat, dlog_partner = -gcoef / (1.0f - gat);

    f32x16 dq[DB];
#pragma unroll
    for (int db = 0; db < DB; ++db) dq[db] = f32x16{};
    // exact row term and per-prior sums for the gate gradient
    float r_all = 0.0f, a_loc = 0.0f, b_loc = 0.0f, a_par = 0.0f, b_par = 0.0f;

    // ---- partners: scores and dP of the partner rows ------------------------
    // Partner row prow of this lane's query (has_p: it exists).
    auto partner = [&](int prow, bool has_p) __attribute__((always_inline)) {
        if (__builtin_amdgcn_ballot_w64(has_p) == 0) return;
        const int prc = has_p ? prow : p.kvpos0;
        bf16x8 kpf[KS], vpf[KS];
#pragma unroll
        for (int s = 0; s < KS; ++s) {
            kpf[s] = *reinterpret_cast<const bf16x8 *>(kp + prc * ksn + 16 * s + 8 * g);
            vpf[s] = *reinterpret_cast<const bf16x8 *>(vp + prc * ksn + 16 * s + 8 * g);
        }
        // score and dP of the partner: per-lane dot products of the query and
        // dL/dy fragments with the partner rows (same layout), then the pair
        float sa = 0.0f, da = 0.0f;
#pragma unroll
        for (int s = 0; s < KS; ++s) {
            sa = dot_bf16x8(qf[s], has_p ? kpf[s] : bf16x8{}, sa);
            da = dot_bf16x8(of[s], has_p ? vpf[s] : bf16x8{}, da);
        }
        const float sd = sa + other_half(sa), dpd = da + other_half(da);
        float delta2;
        bool cut = false;
        if constexpr (CLAMP) {
            const float dl = fminf(fmaxf(sd * p.scale + fb.partner, -p.clamp), p.clamp);
            cut = fabsf(dl) >= p.clamp;
            delta2 = dl * kLog2e;
        } else {
            delta2 = sd * c2 + fb.partner * kLog2e;
        }
        const float wgt = has_p ? __builtin_amdgcn_exp2f(delta2 - lse2) : 0.0f;
        const float dd = cut ? 0.0f : wgt * (dpd - r);
        if (g == 0) {   // one lane of the pair counts the partner
            r_all += wgt * dpd;
            a_par += cut ? 0.0f : wgt * dpd;
            b_par += cut ? 0.0f : wgt;
        }
        // dq += dd * k_p (no key where there is no partner: zeros)
#pragma unroll
        for (int s = 0; s < KS; ++s) kpf[s] = has_p ? kpf[s] : bf16x8{};
        add_row<D>(dq, kpf, dd, g);
    };
    partner(t - pi, partner_enabled(kw, pi) && t - pi >= 0 && t_ok);
    if constexpr (BIDIR) partner(t + pi, t_ok && partner_fwd_of(t, kw, pi, NS) >= 0);

    // ---- window band ---------------------------------------------------------
    auto block = [&](const TileBuf<D> &tb, int j0, int blk) __attribute__((always_inline)) {
        const bool act = BIDIR ? j0 < kend && q0 < NQ && j0 - (q0 + 31) <= kw && j0 + 31 >= q0 - kw
                               : j0 < kend && q0 < NQ && j0 <= q0 + 31 && j0 + 31 >= q0 - kw;
        if (!act) return;
        const bool edge = BIDIR ? !(j0 + 31 - q0 <= kw && q0 + 31 - j0 <= kw) || q0 + 31 >= NQ || j0 + 31 >= NS
                                : !(j0 + 31 <= q0 && j0 >= q0 + 31 - kw) || q0 + 31 >= NQ;
        bf16x8 f[KS];
        read_rows<D>(f, tb.k, blk, c, g);
        f32x16 sc = {};
#pragma unroll
        for (int s = 0; s < KS; ++s) sc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(f[s], qf[s], sc, 0, 0, 0);
        read_vrows<D>(f, tb.v, blk, c, g);
        f32x16 dp = {};
#pragma unroll
        for (int s = 0; s < KS; ++s) dp = __builtin_amdgcn_mfma_f32_32x32x16_bf16(f[s], of[s], dp, 0, 0, 0);
        bf16x8 kt[2][DB];
        float ds[16];
#pragma unroll
        for (int e = 0; e < 16; ++e) {
            float delta2;
            bool cut = false;
            if constexpr (CLAMP) {
                const float dl = fminf(fmaxf(sc[e] * p.scale + fb.local, -p.clamp), p.clamp);
                cut = fabsf(dl) >= p.clamp;
                delta2 = dl * kLog2e;
            } else {
                delta2 = sc[e] * c2;
            }
            if (edge) {
                const int j = j0 + 8 * (e >> 2) + 4 * g + (e & 3);
                const bool ok = BIDIR ? t_ok & (j < NS) & (j - t <= kw) & (t - j <= kw) : t_ok & (j <= t) & (j >= t - kw);
                delta2 = ok ? delta2 : -INFINITY;
            }
            const float wgt = __builtin_amdgcn_exp2f(delta2 - lse2);
            const float pd = wgt * dp[e];
            ds[e] = cut ? 0.0f : pd - wgt * r;
            r_all += pd;
            a_loc += cut ? 0.0f : pd;
            b_loc += cut ? 0.0f : wgt;
        }
        read_cols<D>(kt, tb.k, blk, lane);
        bf16x8 dsb[2];
#pragma unroll
        for (int cc = 0; cc < 2; ++cc)
#pragma unroll
            for (int e = 0; e < 8; ++e) dsb[cc][e] = (__bf16)ds[8 * cc + e];
#pragma unroll
        for (int cc = 0; cc < 2; ++cc)
#pragma unroll
            for (int db = 0; db < DB; ++db)
                dq[db] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(kt[cc][db], dsb[cc], dq[db], 0, 0, 0);
    };
    // Tile m (keys kb0 + 64m ..) is in buffer m mod 2.  A wavefront waits
    // for its own fetches of it (the only vector-memory operations in flight
    // here), the barrier makes every wavefront's share visible, and tile
    // m + 1 then goes into the other buffer (last read for tile m - 1,
    // before that barrier).  LDS-scoped fences: a work-group fence would
    // also wait for the fetch of the next tile.
    auto tile = [&](const TileBuf<D> &cur, TileBuf<D> &ahead, int m) __attribute__((always_inline)) {
        __builtin_amdgcn_s_waitcnt(0xF70);   // vmcnt(0)
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup", "local");
        __builtin_amdgcn_s_barrier();
        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup", "local");
        if (m + 1 < ntiles) tile_fetch<D>(ahead, rk, rv, rowb, TK * (m + 1), w, lane);
        block(cur, kb0 + TK * m, 0);
        block(cur, kb0 + TK * m + 32, 1);
    };
    // unrolled by two so that every fetch and every read names its buffer
    // statically
    for (int m = 0; m < ntiles; m += 2) {
        tile(tA, tB, m);
        if (m + 1 >= ntiles) break;
        tile(tB, tA, m + 1);
    }

    // ---- store ---------------------------------------------------------------
    const float rs = r_all + other_half(r_all);
    const float al = a_loc + other_half(a_loc), bl = b_loc + other_half(b_loc);
    const float ap = a_par + other_half(a_par), bpar = b_par + other_half(b_par);
    const float dg_tot = dlog_local * (al - rs * bl) + dlog_partner * (ap - rs * bpar);
    // dims 32db + 8i + 4g + [0, 4) of dq
    auto dq4 = [&](int db, int i) __attribute__((always_inline)) {
        f32x4 o;
#pragma unroll
        for (int jj = 0; jj < 4; ++jj) o[jj] = dq[db][4 * i + jj] * p.scale;
        return o;
    };
    if constexpr (FULL) {
        // Whole rows: each wavefront passes its 32 rows through a private LDS
        // region and stores them 16 bytes per lane along the rows, not kept in
        // the caches.
        constexpr int P = 4 * D + 16;
        constexpr int LPR = D / 4, RPI = 64 / LPR;
        static_assert(2 * 32 * P <= (int)sizeof(TileBuf<D>), "store staging fits a tile buffer");
        __syncthreads();
        unsigned char *reg = reinterpret_cast<unsigned char *>(w < 2 ? &tA : &tB) + (w & 1) * 32 * P;
#pragma unroll
        for (int db = 0; db < DB; ++db)
#pragma unroll
            for (int i = 0; i < 4; ++i)
                *reinterpret_cast<f32x4 *>(reg + c * P + (32 * db + 8 * i + 4 * g) * 4) = dq4(db, i);
        float *dqp = bp.dq + (bh * N + (q0 - p.qpos0)) * D;
#pragma unroll
        for (int v = 0; v < 32 / RPI; ++v) {
            const int r = RPI * v + lane / LPR, ch = lane % LPR;
            const f32x4 o = *reinterpret_cast<const f32x4 *>(reg + r * P + ch * 16);
            if (q0 + r < NQ) __builtin_nontemporal_store(o, reinterpret_cast<f32x4 *>(dqp + (int64_t)r * D + 4 * ch));
        }
    } else if (t_ok) {   // as it lies
#pragma unroll
        for (int db = 0; db < DB; ++db)
#pragma unroll
            for (int i = 0; i < 4; ++i)
                *reinterpret_cast<f32x4 *>(bp.dq + row * D + 32 * db + 8 * i + 4 * g) = dq4(db, i);
    }
    if (t_ok) {
        if (g == 0) {
            bp.dgate[row] = dg_tot;
            bp.rowterm[row] = rs;
        }
    }
}

template <int D, bool CLAMP, bool BIDIR>
hipError_t launch_q(const BwdParams &p, hipStream_t stream) {
    const int n_qt = (p.f.N + BM - 1) / BM;
    const int64_t n_logical = (int64_t)p.f.B * p.f.H * n_qt;
    const int64_t grid = xcd_grid(n_logical);
    // dq stored as whole rows once every CU has a work-group (pass at 512 tiles,
    // N1000 k64: D = 64 18.7 -> 17.5 us, D = 128 28.4 -> 26.9; at B4 H16 N4096
    // k128 59.7 -> 56.7 and 131 -> 122).  Below, one work-group's time counts
    // and the way through LDS adds to it (64 tiles: 11.2 against 11.6 us, D =
    // 128 15.8 against 16.5; a long band, B1 H4 N3000 k1000 bidirectionally at
    // D = 128, 79 against 87), and with tiles of one wavefront's rows most of it
    // is the barrier (B256 H16 N20: 30.8 against 32.8, 55 against 63).
    const bool full = n_logical >= 256 && p.f.N > 32;
    return launch_kernel(full ? backward_q_bf16_kernel<D, CLAMP, BIDIR, true> : backward_q_bf16_kernel<D, CLAMP, BIDIR, false>,
                         dim3((unsigned)grid), dim3(NT), stream, p, n_qt, (uint32_t)n_logical);
}

template <int D, bool BIDIR>
hipError_t launch_qc(const BwdParams &p, hipStream_t stream) {
    return p.f.clamp > 0.0f ? launch_q<D, true, BIDIR>(p, stream) : launch_q<D, false, BIDIR>(p, stream);
}

}  // namespace

hipError_t launch_backward_q_bf16(const BwdParams &p, hipStream_t stream) {
    if (p.f.D == 64) return p.f.causal ? launch_qc<64, false>(p, stream) : launch_qc<64, true>(p, stream);
    return p.f.causal ? launch_qc<128, false>(p, stream) : launch_qc<128, true>(p, stream);
}

}  // namespace pi_attn
