// backward_f32.hip -- gradients of the full-sequence operator for float32
// data on v_mfma_f32_16x16x4f32 (float32 products and sums), tiles and
// layouts as in f32_tile.h.
//
// For a loss L with dL/dy given, the weights are recomputed from the
// forward's lse as alpha^_tj = exp(delta_tj - lse_t), and
//   dp_tj    = <dL/dy_t, v_j>                    (eq. attn_adapt)
//   r_t      = sum_j alpha^_tj dp_tj = <dL/dy_t, y_t>
//   ddelta_tj = alpha^_tj (dp_tj - r_t)          (softmax Jacobian, eq. jac)
// with ddelta cut to 0 where the optional clamp saturates.  Then
//   dq_t = scale sum_j ddelta_tj k_j,  dk_j = scale sum_t ddelta_tj q_t,
//   dv_j = sum_t alpha^_tj dL/dy_t,
//   dg_t = sum_j ddelta_tj d(log omega_tj)/dg    (eqs. ddelta_da, dalpha_da)
// where d log alpha~/dg = (1 - 2 eps) a (1 - a) / alpha~ on the window and
// d log(1 - alpha~)/dg = -(1 - 2 eps) a (1 - a) / (1 - alpha~) on the partner,
// a = sigmoid(g).
//
// Query pass (dq, gate gradient, row terms): a wavefront owns 16 queries; per
// block of 16 keys S^T = K Q^T and dP^T = V dO^T land in one layout, and
// dQ^T += K^T dS^T takes dS^T from the registers.  r_t is formed from the
// forward output y and written as the key pass's row term.
// Key pass (dk, dv): a wavefront owns 16 keys and walks the queries whose
// working set holds them: t in [j, j + k] and, when pi > k, t = j + pi
// (causal); t in [j - k, j + k] and t = j -/+ pi (bidirectional).  S = Q K^T
// and dP = dO V^T, then dV^T += dO^T P and dK^T += Q^T dS.
//
// What bounds it: as the forward, the float32 matrix rate at large sizes and
// the chain of a tile's blocks at small ones.  Measured against one wavefront
// per row with a cross-lane reduction per entry: 299 -> 40 us a backward at
// B2 H8 N1000 D64 k64 (the launches' 35 us of host time included), 8350 -> 570
// us at B4 H16 N4096 D64 k128, 16.8 -> 2.2 ms at B2 H16 N8192 D128 k256.
#include "f32_tile.h"
#include "kernels.h"
#include "pi_common.h"

namespace pi_attn {

namespace {

using namespace f32;

// ---- query pass -----------------------------------------------------------------
template <int D, bool SPLIT>
__global__ __launch_bounds__(NT, D == 64 && !SPLIT ? 4 : 2) void backward_q_f32_kernel(BwdParams bp, int n_qt, uint32_t n_tiles,
                                                            uint32_t n_logical) {
    const FwdParams &p = bp.f;
    const uint32_t logical = xcd_remap(blockIdx.x, n_logical);
    if (logical >= n_logical) return;
    const int lane = __lane_id(), c = lane & 15, g = lane >> 4;
    const int w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const uint32_t tile = SPLIT ? logical : logical * WAVES + w;
    if (tile >= n_tiles) return;   // never with SPLIT
    const DivMod tile_of = divmod(tile, n_qt), head_of = divmod(tile_of.quot, p.H);
    const int q0 = (int)tile_of.rem * TILE, h = (int)head_of.rem, b = (int)head_of.quot;
    const int64_t bh = tile_of.quot;
    const int t = q0 + c, N = p.N;
    const bool t_ok = t < N;
    const int tq = t_ok ? t : N - 1;
    const int64_t base = b * p.sb + h * p.sh, obase = b * bp.osb + h * bp.osh;
    const float *kp = (const float *)p.k_ptr + base, *vp = (const float *)p.v + base;

    const bool par = partner_enabled(p.k, p.pi);
    const Walk walk(q0, N, p.k, p.causal ? 0 : p.k, p.pi, par, par && !p.causal);

    const int first = SPLIT ? w : 0;
    constexpr int STEP = SPLIT ? WAVES : 1;
    RowFrag<D> q, o;
    load_row<D>(q, (const float *)p.q + base + tq * p.sn, g);
    load_row<D>(o, (const float *)bp.dout + obase + tq * bp.osn, g);
    const bool clamp_on = p.clamp > 0.0f;
    const float gl = p.gate[b * p.gsb + h * p.gsh + tq * p.gsn];
    const FusionBias fb = fusion_bias(gl, clamp_on);
    const float shift = fb.lse_shift - bp.lse[bh * N + tq];
    float r_t;
    {
        RowFrag<D> y;
        load_row<D>(y, (const float *)bp.out + obase + tq * bp.osn, g);
        r_t = (float)col_sum(dot_lane<D>(o, y));
    }
    Acc<D> dq;
#pragma unroll
    for (int d = 0; d < D / 16; ++d) dq.a[d] = f32x4{};
    float d_win = 0.0f, d_par = 0.0f;   // sums of ddelta over the window and the partners

    for (int i = first; i < walk.total; i += STEP) {
        const Block bl = walk.block(i);
        const bool edge = walk.edge(bl);
        RowFrag<D> kr, vr;
        const int64_t row = walk.clamp(bl.j + c) * p.sn;
        load_row<D>(kr, kp + row, g);
        load_row<D>(vr, vp + row, g);
        const f32x4 dot = dot_rows<D>(kr, q), dp = dot_rows<D>(vr, o);
        __builtin_amdgcn_sched_barrier(0);   // the row registers are free for the transposed rows
        ColFrag<D> kt;
        load_cols<D>(kt, [&](int r) { return kp + walk.clamp(bl.j + r) * p.sn; }, c, g);
        const float bias = bl.kind ? fb.partner : fb.local;
        float ds[4];
        unsigned ok = 0xf;
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            bool cut;
            const float a = weight(dot[r], bias, shift, p, clamp_on, cut);
            ds[r] = cut ? 0.0f : a * (dp[r] - r_t);
        }
        if (edge) {
            ok = 0;
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                const bool in = t_ok && walk.has(bl, bl.j + 4 * g + r, t);
                ds[r] = in ? ds[r] : 0.0f;
                ok |= (in ? 1u : 0u) << r;
            }
        }
        const float sum = (ds[0] + ds[1]) + (ds[2] + ds[3]);
        d_par += bl.kind ? sum : 0.0f;
        d_win += bl.kind ? 0.0f : sum;
        add_rows<D>(dq, kt, ds, edge, ok, [&](int r) { return kp + walk.clamp(bl.j + r) * p.sn; }, lane);
    }


    const GateDeriv gg = gate_deriv(gl);
    d_win = col_sum(d_win);
    d_par = col_sum(d_par);
    float *dqp = bp.dq + (bh * N + q0) * D;
    if constexpr (!SPLIT) {
        if (t_ok) {
            store_acc<D>(dqp + c * D, dq, p.scale, g);
            if (g == 0) {
                bp.dgate[bh * N + t] = d_win * gg.local + d_par * gg.partner;
                bp.rowterm[bh * N + t] = r_t;
            }
        }
    } else {
        __shared__ float s_d[WAVES][2][TILE];
        __shared__ alignas(16) float s_q[WAVES][TILE][D + 4];
        store_acc<D>(&s_q[w][c][0], dq, 1.0f, g);
        if (g == 0) {
            s_d[w][0][c] = d_win;
            s_d[w][1][c] = d_par;
        }
        __syncthreads();
        const int cc = threadIdx.x >> 4, x = threadIdx.x & 15;
        if (q0 + cc < N) {
#pragma unroll
            for (int hh = 0; hh < D / 64; ++hh) {
                f32x4 s = {};
#pragma unroll
                for (int i = 0; i < WAVES; ++i) s += *reinterpret_cast<const f32x4 *>(&s_q[i][cc][64 * hh + 4 * x]);
                *reinterpret_cast<f32x4 *>(dqp + cc * D + 64 * hh + 4 * x) = s * p.scale;
            }
        }
        if (w == 0 && g == 0 && t_ok) {
            const float dw = (s_d[0][0][c] + s_d[1][0][c]) + (s_d[2][0][c] + s_d[3][0][c]);
            const float dr = (s_d[0][1][c] + s_d[1][1][c]) + (s_d[2][1][c] + s_d[3][1][c]);
            bp.dgate[bh * N + t] = dw * gg.local + dr * gg.partner;
            bp.rowterm[bh * N + t] = r_t;
        }
    }
}

// ---- key pass -------------------------------------------------------------------
template <int D, bool SPLIT>
__global__ __launch_bounds__(NT) void backward_kv_f32_kernel(BwdParams bp, int n_kt, uint32_t n_tiles,
                                                             uint32_t n_logical) {
    const FwdParams &p = bp.f;
    const uint32_t logical = xcd_remap(blockIdx.x, n_logical);
    if (logical >= n_logical) return;
    const int lane = __lane_id(), c = lane & 15, g = lane >> 4;
    const int w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const uint32_t tile = SPLIT ? logical : logical * WAVES + w;
    if (tile >= n_tiles) return;   // never with SPLIT
    const DivMod tile_of = divmod(tile, n_kt), head_of = divmod(tile_of.quot, p.H);
    const int j0 = (int)tile_of.rem * TILE, h = (int)head_of.rem, b = (int)head_of.quot;
    const int64_t bh = tile_of.quot;
    const int j = j0 + c, N = p.N;
    const bool j_ok = j < N;
    const int jq = j_ok ? j : N - 1;
    const int64_t base = b * p.sb + h * p.sh, obase = b * bp.osb + h * bp.osh;
    const float *qp = (const float *)p.q + base, *op = (const float *)bp.dout + obase;
    const float *gp = p.gate + b * p.gsb + h * p.gsh;
    const float *lsep = bp.lse + bh * N, *rtp = bp.rowterm + bh * N;

    // rows are queries: the partner t - pi of query j + pi is key j (an ahead
    // block), the partner t + pi of query j - pi (a back block)
    const bool par = partner_enabled(p.k, p.pi);
    const Walk walk(j0, N, p.causal ? 0 : p.k, p.k, p.pi, par && !p.causal, par);

    const int first = SPLIT ? w : 0;
    constexpr int STEP = SPLIT ? WAVES : 1;
    RowFrag<D> kk, vv;
    load_row<D>(kk, (const float *)p.k_ptr + base + jq * p.sn, g);
    load_row<D>(vv, (const float *)p.v + base + jq * p.sn, g);
    const bool clamp_on = p.clamp > 0.0f;
    Acc<D> dk, dv;
#pragma unroll
    for (int d = 0; d < D / 16; ++d) {
        dk.a[d] = f32x4{};
        dv.a[d] = f32x4{};
    }
    // The rows of the next block are loaded once the current ones are used
    // (train-size launches have one or two wavefronts per SIMD: 31 against
    // 37 us at B2 H8 N1000 D128 k64, 20 against 22 us at D = 64).
    RowFrag<D> qr, dr;
    auto load = [&](int i) __attribute__((always_inline)) {
        const int64_t t = walk.clamp(walk.block(i).j + c);
        load_row<D>(qr, qp + t * p.sn, g);
        load_row<D>(dr, op + t * bp.osn, g);
    };
    if (first < walk.total) load(first);
    for (int i = first; i < walk.total; i += STEP) {
        const Block bl = walk.block(i);
        const bool edge = walk.edge(bl);
        auto qrow = [&](int r) { return qp + walk.clamp(bl.j + r) * p.sn; };
        auto orow = [&](int r) { return op + walk.clamp(bl.j + r) * bp.osn; };
        float gl[4], lse[4], rt[4];   // of rows 4 g + r
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            const int64_t tr = walk.clamp(bl.j + 4 * g + r);
            gl[r] = gp[tr * p.gsn];
            lse[r] = lsep[tr];
            rt[r] = rtp[tr];
        }
        const f32x4 dot = dot_rows<D>(qr, kk), dp = dot_rows<D>(dr, vv);
        __builtin_amdgcn_sched_barrier(0);   // the row registers are free for the transposed rows
        ColFrag<D> qt, dt;
        load_cols<D>(dt, orow, c, g);
        if constexpr (D == 64) {
            load_cols<D>(qt, qrow, c, g);
            if (i + STEP < walk.total) load(i + STEP);
        }
        float a[4], ds[4];
        unsigned ok = 0xf;
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            const FusionBias fb = fusion_bias(gl[r], clamp_on);
            bool cut;
            a[r] = weight(dot[r], bl.kind ? fb.partner : fb.local, fb.lse_shift - lse[r], p, clamp_on, cut);
            ds[r] = cut ? 0.0f : a[r] * (dp[r] - rt[r]);
        }
        if (edge) {
            ok = 0;
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                const bool in = j_ok && walk.has(bl, bl.j + 4 * g + r, j);
                a[r] = in ? a[r] : 0.0f;
                ds[r] = in ? ds[r] : 0.0f;
                ok |= (in ? 1u : 0u) << r;
            }
        }
        add_rows<D>(dv, dt, a, edge, ok, orow, lane);
        if constexpr (D == 128) {   // both at once would leave one wavefront per SIMD
            __builtin_amdgcn_sched_barrier(0);
            load_cols<D>(qt, qrow, c, g);
        }
        add_rows<D>(dk, qt, ds, edge, ok, qrow, lane);
        if constexpr (D == 128) {
            if (i + STEP < walk.total) load(i + STEP);
        }
    }

    const int64_t grow = bh * N + j0;
    if constexpr (!SPLIT) {
        if (j_ok) {
            store_acc<D>(bp.dk + (grow + c) * D, dk, p.scale, g);
            store_acc<D>(bp.dv + (grow + c) * D, dv, 1.0f, g);
        }
    } else {
        __shared__ alignas(16) float s_a[WAVES][TILE][D + 4];
        const int cc = threadIdx.x >> 4, x = threadIdx.x & 15;
#pragma unroll
        for (int which = 0; which < 2; ++which) {
            if (which) __syncthreads();   // the first tensor's partial sums are read
            store_acc<D>(&s_a[w][c][0], which ? dv : dk, 1.0f, g);
            __syncthreads();
            float *dst = which ? bp.dv : bp.dk;
            const float f = which ? 1.0f : p.scale;
            if (j0 + cc < N) {
#pragma unroll
                for (int hh = 0; hh < D / 64; ++hh) {
                    f32x4 s = {};
#pragma unroll
                    for (int i2 = 0; i2 < WAVES; ++i2)
                        s += *reinterpret_cast<const f32x4 *>(&s_a[i2][cc][64 * hh + 4 * x]);
                    *reinterpret_cast<f32x4 *>(dst + (grow + cc) * D + 64 * hh + 4 * x) = s * f;
                }
            }
        }
    }
}

template <int D, bool SPLIT>
hipError_t launch(const BwdParams &p, hipStream_t stream) {
    const int n_t = (p.f.N + TILE - 1) / TILE;
    const int64_t n_tiles = tiles_of((int64_t)p.f.B * p.f.H, p.f.N);
    const int64_t n_logical = SPLIT ? n_tiles : (n_tiles + WAVES - 1) / WAVES;
    const dim3 grid((unsigned)xcd_grid(n_logical)), block(NT);
    const hipError_t e =
        launch_kernel(backward_q_f32_kernel<D, SPLIT>, grid, block, stream, p, n_t, (uint32_t)n_tiles, (uint32_t)n_logical);
    if (e != hipSuccess) return e;
    return launch_kernel(backward_kv_f32_kernel<D, SPLIT>, grid, block, stream, p, n_t, (uint32_t)n_tiles, (uint32_t)n_logical);
}

template <int D>
hipError_t launch_d(const BwdParams &p, hipStream_t stream) {
    const bool split = tiles_of((int64_t)p.f.B * p.f.H, p.f.N) <= kSplitTiles;
    return split ? launch<D, true>(p, stream) : launch<D, false>(p, stream);
}

}  // namespace

hipError_t launch_backward_f32(const BwdParams &p, hipStream_t stream) {
    if (one_per_row(p.f)) return launch_backward_rows_f32(p, stream);
    return p.f.D == 64 ? launch_d<64>(p, stream) : launch_d<128>(p, stream);
}

}  // namespace pi_attn
