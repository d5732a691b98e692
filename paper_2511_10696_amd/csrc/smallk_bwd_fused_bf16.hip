// smallk_bwd_fused_bf16.hip -- backward of pi-Attention for a small window
// radius in one pass over the sequence: bf16 inputs, fp32 arithmetic and fp32
// gradients, D = 64, causal or bidirectional, every entry of a working set
// within `reach` = max(k, pi) rows of its query (k when pi <= k).
//
// The two passes of smallk_bwd_bf16.hip each read q, k, v and dL/dy, and the
// key pass forms every weight and dP again; both run at the rate of a copy.
// Here a work-group owns a run of rows [c0, c1) of one (b, h) and walks it in
// steps of 32 rows, the rows of all four tensors in a ring in LDS (the next 32
// are loaded into registers meanwhile).  A step has two parts, each with a row
// on 8 lanes of 8 dimensions:
//   queries [s, s + 32): alpha^_tj and dP_tj of every entry, the exact row
//     term r_t = sum_j alpha^_tj dP_tj, ddelta_tj = alpha^_tj (dP_tj - r_t)
//     (Sec. 3.5 eq. jac; 0 where the clamp saturates), dq and the gate
//     gradient (eqs. ddelta_da, dalpha_da); alpha^ and ddelta go to a ring of
//     their own in LDS;
//   keys [s - reach, s - reach + 32), whose queries have all been seen:
//       dk_j = scale sum_t ddelta_tj q_t,  dv_j = sum_t alpha^_tj dL/dy_t.
// Each run also goes over the queries within reach of its keys that it does
// not own, for their weights only (reach of every run.len rows).
//
// What bounds it: at k <= 4, HBM (20 bytes a dimension and row, each input
// read about once: 1.35 GB at B8 H16 N8192); at k = 8 and bidirectionally the
// VALU, 84 instructions an entry and 8 rows.  Against the two passes: 400 ->
// 266 us at B8 H16 N8192 k4 pi16, 457 -> 320 us at k8, bidirectional 503 ->
// 357 us and 706 -> 549 us; B4 H8 N2000 38 -> 31 us.  With the sums of the two
// passes (dq = sum w dP k - r sum w k) in place of kept alpha^ and dP, a ring
// of three and four steps and two barriers a step: 309 and 153 us where this
// takes 300 and 100 (causal B8 H16 N8192, bidirectional B32 H8 N1000).
#include <algorithm>

#include "kernels.h"
#include "pi_common.h"
#include "smallk.h"
#include "smallk_common.h"

namespace pi_attn {

namespace {

using namespace sk;

typedef float f32x4 __attribute__((ext_vector_type(4)));

constexpr int D = 64;
constexpr int STEP = 32;        // rows per step
constexpr int ROWB = 2 * D;     // bytes of a row of one tensor
constexpr int BACK = 32;        // rows before s that a step reads at most

template <bool BIDIR>
struct Ring {
    static constexpr int REACH = BIDIR ? 16 : 32;   // largest reach
    // rows of a step: [s - BACK, s + 32), bidirectionally up to s + 32 + reach
    static constexpr int ROWS = BIDIR ? 80 : 64;
    static constexpr int BYTES = ROWS * ROWB;
};

struct Runs {
    int len, n;          // rows per run, runs per (b, h)
    uint32_t n_logical;
};

// x or x - n, for x in [0, 2 n)
__device__ inline int wrap(int x, int n) { return (int)min((unsigned)x, (unsigned)(x - n)); }

template <bool BIDIR, int KMAX>
__global__ __launch_bounds__(NT, BIDIR ? 3 : 4) void smallk_bwd_fused_kernel(BwdParams bp, Runs runs) {
    using R = Ring<BIDIR>;
    constexpr int NP = BIDIR ? 2 : 1;                        // partner slots
    constexpr int NW = BIDIR ? 2 * KMAX + 1 : KMAX + 1;      // window slots at most
    constexpr int NE = NP + NW;                              // entries of a query at most
    constexpr int WROW = 8 * NE, WBYTES = 64 * WROW;         // bytes of a query's weights, of the ring
    static_assert((BIDIR ? 2 : 1) * R::REACH <= BACK && BACK + STEP + (BIDIR ? R::REACH : 0) <= R::ROWS, "rows in use");
    const FwdParams &p = bp.f;
    __shared__ alignas(16) unsigned char ring[4][R::BYTES];   // q, k, v, dL/dy
    __shared__ float2 rs[R::ROWS];                            // lse, gate logit
    // Whole rows of gradients, half a row at a time (see store_row).
    constexpr bool WHOLE = BIDIR && KMAX == 4;
    __shared__ alignas(16) float stage[WHOLE ? NT / 64 : 1][8][32];
    __shared__ alignas(8) unsigned char we[WBYTES];           // (alpha^, ddelta) of queries [s - BACK, s + 32)

    const uint32_t logical = xcd_remap(blockIdx.x, runs.n_logical);
    if (logical >= runs.n_logical) return;
    const DivMod run_of = divmod(logical, runs.n), head_of = divmod(run_of.quot, p.H);
    const int64_t bh = run_of.quot;
    const int h = (int)head_of.rem, b = (int)head_of.quot;
    const int N = p.N, kw = p.k, pi = p.pi;
    const bool par = partner_enabled(kw, pi);
    const int reach = par ? pi : kw;
    const int c0 = (int)run_of.rem * runs.len, c1 = min(N, c0 + runs.len);
    const int tid = threadIdx.x;
    const int i = tid >> 3, sl = tid & 7;   // row of the step, lane within its row
    const int nw = BIDIR ? 2 * kw + 1 : kw + 1;
    const bool clamp_on = p.clamp > 0.0f;

    const int64_t base = b * p.sb + h * p.sh + 8 * sl;
    const __bf16 *qp = (const __bf16 *)p.q + base, *kp = (const __bf16 *)p.k_ptr + base, *vp = (const __bf16 *)p.v + base;
    const __bf16 *op = (const __bf16 *)bp.dout + b * bp.osb + h * bp.osh + 8 * sl;
    const float *gp = p.gate + b * p.gsb + h * p.gsh;
    const int64_t rbase = bh * N;

    // Step n: queries [s, s + 32), s = s0 + 32 n; keys [s - reach, ..); the
    // rows loaded last are [s + ahead, s + ahead + 32).
    const int ahead = BIDIR ? reach : 0;
    const int s0 = BIDIR ? c0 - reach : c0;
    const int steps = (c1 + reach - s0 + STEP - 1) / STEP;

    struct Rows {
        u32x4 q, k, v, o;
        float lse, gl;
    };
    // this thread's part of row x; zeros outside the sequence
    auto load = [&](Rows &r, int x) __attribute__((always_inline)) {
        r.q = r.k = r.v = r.o = u32x4{0, 0, 0, 0};
        r.lse = r.gl = 0.0f;
        if (x >= 0 && x < N) {
            r.k = *reinterpret_cast<const u32x4 *>(kp + x * p.sn);
            r.v = *reinterpret_cast<const u32x4 *>(vp + x * p.sn);
            r.q = *reinterpret_cast<const u32x4 *>(qp + x * p.sn);
            r.o = *reinterpret_cast<const u32x4 *>(op + x * bp.osn);
            r.lse = bp.lse[rbase + x];
            r.gl = gp[x * p.gsn];
        }
    };
    auto keep = [&](const Rows &r, int slot) __attribute__((always_inline)) {
        const int off = slot * ROWB + 16 * sl;
        *reinterpret_cast<u32x4 *>(ring[0] + off) = r.q;
        *reinterpret_cast<u32x4 *>(ring[1] + off) = r.k;
        *reinterpret_cast<u32x4 *>(ring[2] + off) = r.v;
        *reinterpret_cast<u32x4 *>(ring[3] + off) = r.o;
        if (sl == 0) rs[slot] = make_float2(r.lse, r.gl);
    };
    auto chunk = [&](int tensor, int off) { return *reinterpret_cast<const uint4 *>(ring[tensor] + off); };

    // A row of a gradient, times f, where `ok`.  As it lies a lane stores 32
    // bytes in two pieces.  WHOLE: the wavefront's 8 rows go through LDS, half
    // a row at a time, and out as whole 128-byte lines that are not kept in
    // the caches: 152.8 -> 145.7 us a training pass at B32 H8 N1000
    // bidirectionally; causal k = 4, at the copy rate either way, 425 -> 428
    // us; at k = 8 the LDS it takes costs a work-group per CU.
    auto store_row = [&](float *dst, const float (&v)[8], float f, bool ok) __attribute__((always_inline)) {
        const f32x4 lo = {v[0] * f, v[1] * f, v[2] * f, v[3] * f}, hi = {v[4] * f, v[5] * f, v[6] * f, v[7] * f};
        if constexpr (WHOLE) {
            float *reg = &stage[tid >> 6][i & 7][0];
#pragma unroll
            for (int half = 0; half < 2; ++half) {
                __builtin_amdgcn_wave_barrier();
                if ((sl >> 2) == half) {
                    *reinterpret_cast<f32x4 *>(reg + 8 * (sl & 3)) = lo;
                    *reinterpret_cast<f32x4 *>(reg + 8 * (sl & 3) + 4) = hi;
                }
                __builtin_amdgcn_wave_barrier();
                const f32x4 x = *reinterpret_cast<const f32x4 *>(reg + 4 * sl);
                if (ok) __builtin_nontemporal_store(x, reinterpret_cast<f32x4 *>(dst + 32 * half + 4 * sl));
            }
        } else if (ok) {
            *reinterpret_cast<f32x4 *>(dst + 8 * sl) = lo;
            *reinterpret_cast<f32x4 *>(dst + 8 * sl + 4) = hi;
        }
    };

    // ring slot of row s - BACK, and the weights' of query s - BACK (bytes)
    int os = 0, ws = 0;
    Rows nx;
    // the rows before step 0's own: [s0 - BACK, s0 + ahead), 32 at a time
    // (bidirectionally the last of them again, where they do not fill 32)
    for (int g = 0; g < BACK + ahead; g += STEP) {
        const int rel = min(g, BACK + ahead - STEP) + i;
        load(nx, s0 - BACK + rel);
        keep(nx, rel);
    }
    load(nx, s0 + ahead + i);
    keep(nx, BACK + ahead + i);
    __syncthreads();
    for (int n = 0; n < steps; ++n) {
        const int s = s0 + STEP * n;
        if (n + 1 < steps) load(nx, s + STEP + ahead + i);

        // ---- queries -----------------------------------------------------------
        const int t = s + i;
        // ring byte offsets, before wrapping, of this thread's chunk of row t
        const int tb = (os + BACK + i) * ROWB + 16 * sl;
        const bool t_ok = t >= 0 && t < N;
        {
            const int own = wrap(tb, R::BYTES);
            const uint4 qc = chunk(0, own), oc = chunk(3, own);
            const float2 sv = rs[wrap(os + BACK + i, R::ROWS)];
            const FusionBias fb = fusion_bias(sv.y, clamp_on);
            const GateDeriv gdv = gate_deriv(sv.y);
            const float lse2 = (sv.x - fb.lse_shift) * kLog2e;
            float al[NE], ds[NE], r = 0.0f;   // alpha^, dP
            // A query outside the sequence has no entries: alpha^ and ddelta
            // are 0 whatever the rows around it hold (0 times a row that is
            // not finite would reach keys that no query of that row's has).
            unsigned cuts = t_ok ? 0u : ~0u;
            const unsigned rows = t_ok ? N : 0;
            auto score = [&](int e, int off, bool ok, float bias) __attribute__((always_inline)) {
                bool cut;
                const float s2 = logit2(sum8(dot8(qc, chunk(1, off), 0.0f)), bias, p, clamp_on, cut);
                ds[e] = sum8(dot8(oc, chunk(2, off), 0.0f));
                al[e] = ok ? __builtin_amdgcn_exp2f(s2 - lse2) : 0.0f;
                cuts |= cut ? 1u << e : 0u;
                r += al[e] * ds[e];
            };
            // offset of row t + d (a row outside the sequence is zeros)
            auto at = [&](int d) { return wrap(tb + d * ROWB, R::BYTES); };
            if (par) {
                score(0, at(-pi), (unsigned)t - pi < rows, fb.partner);
                if constexpr (BIDIR) score(1, at(pi), (unsigned)t + pi < rows, fb.partner);
            }
#pragma unroll
            for (int x = 0; x < NW; ++x) {
                if (x < nw) score(NP + x, at(x - kw), (unsigned)t - kw + x < rows, fb.local);
            }
            float dq[8], d_par = 0.0f, d_loc = 0.0f;
#pragma unroll
            for (int e = 0; e < 8; ++e) dq[e] = 0.0f;
            auto add = [&](int e, int off, float &sum) __attribute__((always_inline)) {
                const float d = (cuts >> e) & 1 ? 0.0f : al[e] * (ds[e] - r);
                sum += d;
                axpy8(dq, d, chunk(1, off));
                if (sl == 0)
                    *reinterpret_cast<float2 *>(we + wrap(ws + (BACK + i) * WROW, WBYTES) + 8 * e) = make_float2(al[e], d);
            };
            if (par) {
                add(0, at(-pi), d_par);
                if constexpr (BIDIR) add(1, at(pi), d_par);
            }
#pragma unroll
            for (int x = 0; x < NW; ++x) {
                if (x < nw) add(NP + x, at(x - kw), d_loc);
            }
            const bool mine = t >= c0 && t < c1;
            store_row(bp.dq + (rbase + t) * D, dq, p.scale, mine);
            if (mine && sl == 0) {
                bp.dgate[rbase + t] = d_loc * gdv.local + d_par * gdv.partner;
                bp.rowterm[rbase + t] = r;
            }
        }
        __syncthreads();   // the weights are in place

        // ---- keys --------------------------------------------------------------
        const int j = t - reach;
        const bool mine = j >= c0 && j < c1;
        if (WHOLE || mine) {
            float dk[8], dv[8];
#pragma unroll
            for (int e = 0; e < 8; ++e) dk[e] = dv[e] = 0.0f;
            const int jb = tb - reach * ROWB, wb = ws + (BACK + i - reach) * WROW;
            // query j + d, of whose entries key j is number e (a query outside
            // the sequence is zeros, its weights too)
            auto visit = [&](int d, int e) __attribute__((always_inline)) {
                const int off = wrap(jb + d * ROWB, R::BYTES);
                const float2 ad = *reinterpret_cast<const float2 *>(we + wrap(wb + d * WROW, WBYTES) + 8 * e);
                axpy8(dk, ad.y, chunk(0, off));
                axpy8(dv, ad.x, chunk(3, off));
            };
            if (par) {
                visit(pi, 0);
                if constexpr (BIDIR) visit(-pi, 1);
            }
#pragma unroll
            for (int x = 0; x < NW; ++x) {   // queries j .. j + k, bidirectionally from j - k
                const int d = x - (BIDIR ? kw : 0);
                if (x < nw) visit(d, NP + kw - d);
            }
            store_row(bp.dk + (rbase + j) * D, dk, p.scale, mine);
            store_row(bp.dv + (rbase + j) * D, dv, 1.0f, mine);
        }
        if (n + 1 == steps) break;
        __syncthreads();   // rows [s - BACK, s) are done with
        os = wrap(os + STEP, R::ROWS);
        ws = wrap(ws + STEP * WROW, WBYTES);
        keep(nx, wrap(os + BACK + ahead + i, R::ROWS));
        __syncthreads();   // the next rows are in place
    }
}

template <bool BIDIR, int KMAX>
hipError_t launch_k(const BwdParams &p, hipStream_t stream) {
    const int64_t bh = (int64_t)p.f.B * p.f.H;
    Runs runs;
    // Runs: as many as are resident at once, three work-groups per CU (LDS
    // allows a fourth when causal, which pays where the VALU binds: 277
    // against 266 us with three at k4, 320 against 332 us at k8), but of no
    // fewer than 128 rows.
    const int64_t want = BIDIR || KMAX == 4 ? 768 : 1024;
    const int64_t n = std::max<int64_t>(1, std::min<int64_t>((want + bh - 1) / bh, (p.f.N + 127) / 128));
    runs.len = (int)((((int64_t)p.f.N + n - 1) / n + STEP - 1) / STEP * STEP);
    runs.n = (p.f.N + runs.len - 1) / runs.len;
    runs.n_logical = (uint32_t)(bh * runs.n);
    return launch_kernel(smallk_bwd_fused_kernel<BIDIR, KMAX>, dim3((unsigned)xcd_grid(runs.n_logical)), dim3(NT),
                         stream, p, runs);
}

}  // namespace

// One pass instead of two: for windows short enough that the weights of a
// step fit beside the ring (at k = 12 the two take 292 us at B8 H16 N4096, as
// one does) and launches that fill the chip (one run takes its steps one after
// the other: 22.7 against 20.4 us in two passes at 32000 rows, 31 against 38
// us at 64000).  A sequence of a tile or two takes more steps (N + reach rows,
// bidirectionally N + 2 reach) than the two passes have tiles, and a step costs
// the more the longer the window: at twice as many, k = 8, causal 1.09 times
// the two passes' time (N = 31, pi = 16), bidirectional k = 4 1.17 to 1.4 times
// (N = 4 to 32; N = 33 and 40, 3 steps for 2 tiles, equal), at 1.5 times as
// many, bidirectional k = 8 1.06 to 1.09 times (N = 50, 64; pi = 9).
// It takes a work-group for every (b, h) where the two passes take one for up
// to 32 heads, and a launch has fewer than 2^32 threads.
bool smallk_fused_takes(const BwdParams &p) {
    const FwdParams &f = p.f;
    const int reach = partner_enabled(f.k, f.pi) ? f.pi : f.k;
    if (f.D != 64 || f.k > 8 || reach > (f.causal ? Ring<false>::REACH : Ring<true>::REACH)) return false;
    const int64_t bh = (int64_t)f.B * f.H;
    if (bh * f.N < 49152 || xcd_grid(bh) * NT >= ((int64_t)1 << 32)) return false;
    const int64_t steps = (f.N + (f.causal ? 1 : 2) * (int64_t)reach + STEP - 1) / STEP, tiles = (f.N + TT - 1) / TT;
    if (f.causal) return f.k <= 4 || steps < 2 * tiles;
    return f.k <= 4 ? steps < 2 * tiles : 2 * steps < 3 * tiles;
}

hipError_t launch_backward_smallk_fused(const BwdParams &p, hipStream_t stream) {
    if (!p.f.causal) return p.f.k <= 4 ? launch_k<true, 4>(p, stream) : launch_k<true, 8>(p, stream);
    return p.f.k <= 4 ? launch_k<false, 4>(p, stream) : launch_k<false, 8>(p, stream);
}

}  // namespace pi_attn
