// attn_f32.hip -- float32 forward.
//
// v_mfma_f32_16x16x4f32 (float32 products and sums), tiles and layouts as in
// f32_tile.h.  A wavefront owns 16 queries; per block of 16 keys S^T = K Q^T
// lands with lane (c, g) holding the scores of query c for keys 4 g + r, the
// softmax reductions are in-lane plus two exchanges, and O^T += V^T P^T takes
// P^T straight from the score registers.  A partner run is one more block of
// which only the diagonal is valid.
//
// What bounds it: the float32 matrix rate (a block of 16 x 16 entries costs
// 2 x D / 4 instructions of 32 clocks, used by k + 1 of k + 16 keys) at large
// sizes, the dependent chain of a tile's blocks at small ones.  Measured
// against one wavefront per query with a cross-lane reduction per entry:
// 14.4 -> 5.9 us a launch at B1 H2 N256 D64 k32, 88 -> 13 us at B2 H8 N1000
// D64 k64, 2234 -> 152 us at B4 H16 N4096 D64 k128, 4696 -> 526 us at
// B2 H16 N8192 D128 k256.  Loading the next block ahead (two key blocks in registers,
// three wavefronts per SIMD instead of four) measured within 4% either way
// and is not used.
#include "f32_tile.h"
#include "kernels.h"
#include "pi_common.h"

namespace pi_attn {

namespace {

using namespace f32;

// Online softmax state of a tile: lane (c, g) keeps the sum over its own
// rows of every block (4 g + r); the maximum is the column's.
template <int D>
struct Soft {
    Acc<D> o;
    float m = -INFINITY;   // running max, log2 units
    float l = 0.0f;        // this lane's part of the running sum
};

template <int D>
struct KeyBlock {
    RowFrag<D> k;
    ColFrag<D> v;
};

template <int D, bool SPLIT>
__global__ __launch_bounds__(NT, D == 64 && !SPLIT ? 4 : 2) void forward_f32_kernel(FwdParams p, int n_qt, uint32_t n_tiles, uint32_t n_logical) {
    const uint32_t logical = xcd_remap(blockIdx.x, n_logical);
    if (logical >= n_logical) return;
    const int lane = __lane_id(), c = lane & 15, g = lane >> 4;
    const int w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const uint32_t tile = SPLIT ? logical : logical * WAVES + w;
    if (tile >= n_tiles) return;   // never with SPLIT: the whole work-group stays for the merge
    const DivMod tile_of = divmod(tile, n_qt), head_of = divmod(tile_of.quot, p.H);
    const int q0 = (int)tile_of.rem * TILE, h = (int)head_of.rem, b = (int)head_of.quot;
    const int64_t bh = tile_of.quot;
    const int t = q0 + c, N = p.N;
    const bool t_ok = t < N;
    const int tq = t_ok ? t : N - 1;
    const int64_t base = b * p.sb + h * p.sh;
    const float *kp = (const float *)p.k_ptr + base, *vp = (const float *)p.v + base;

    const bool par = partner_enabled(p.k, p.pi);
    const Walk walk(q0, N, p.k, p.causal ? 0 : p.k, p.pi, par, par && !p.causal);

    auto load = [&](KeyBlock<D> &kb, int i) __attribute__((always_inline)) {
        const int j = walk.block(i).j;
        load_row<D>(kb.k, kp + walk.clamp(j + c) * p.sn, g);
        load_cols<D>(kb.v, [&](int r) { return vp + walk.clamp(j + r) * p.sn; }, c, g);
    };
    const int first = SPLIT ? w : 0;
    constexpr int STEP = SPLIT ? WAVES : 1;
    KeyBlock<D> kb;
    if (first < walk.total) load(kb, first);   // flies with the query rows
    RowFrag<D> q;
    load_row<D>(q, (const float *)p.q + base + tq * p.sn, g);
    const bool clamp_on = p.clamp > 0.0f;
    const FusionBias fb = fusion_bias(p.gate[b * p.gsb + h * p.gsh + tq * p.gsn], clamp_on);
    const float c2 = p.scale * kLog2e;

    Soft<D> st;
#pragma unroll
    for (int d = 0; d < D / 16; ++d) st.o.a[d] = f32x4{};

    auto step = [&](const KeyBlock<D> &cur, int i) __attribute__((always_inline)) {
        const Block bl = walk.block(i);
        const bool edge = walk.edge(bl);
        const f32x4 dot = dot_rows<D>(cur.k, q);
        const float bias = bl.kind ? fb.partner : fb.local;
        float s[4];
        unsigned ok = 0xf;
#pragma unroll
        for (int r = 0; r < 4; ++r)
            s[r] = clamp_on ? fminf(fmaxf(dot[r] * p.scale + bias, -p.clamp), p.clamp) * kLog2e
                            : __builtin_fmaf(dot[r], c2, bias * kLog2e);
        if (edge) {
            ok = 0;
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                const bool in = t_ok && walk.has(bl, bl.j + 4 * g + r, t);
                s[r] = in ? s[r] : -INFINITY;
                ok |= (in ? 1u : 0u) << r;
            }
        }
        const float mx = col_max(fmaxf(fmaxf(s[0], s[1]), fmaxf(s[2], s[3])));
        if (__builtin_amdgcn_ballot_w64(mx > st.m)) {
            const float mn = fmaxf(st.m, mx);
            // lanes whose maximum stays scale by exactly 1 (also while it is -inf)
            const float f = mx > st.m ? __builtin_amdgcn_exp2f(st.m - mn) : 1.0f;
            st.m = mn;
            st.l *= f;
#pragma unroll
            for (int d = 0; d < D / 16; ++d) st.o.a[d] *= f;
        }
        const float mu = st.m == -INFINITY ? 0.0f : st.m;
        float pr[4];
#pragma unroll
        for (int r = 0; r < 4; ++r) pr[r] = __builtin_amdgcn_exp2f(s[r] - mu);
        st.l += (pr[0] + pr[1]) + (pr[2] + pr[3]);
        add_rows<D>(st.o, cur.v, pr, edge, ok, [&](int r) { return vp + walk.clamp(bl.j + r) * p.sn; }, lane);
    };
    for (int i = first; i < walk.total; i += STEP) {
        if (i != first) load(kb, i);
        step(kb, i);
    }

    float *out = (float *)p.out + b * p.osb + h * p.osh;
    float l = col_sum(st.l);
    if constexpr (!SPLIT) {
        if (t_ok) {
            store_acc<D>(out + t * p.osn, st.o, 1.0f / l, g);
            if (p.lse && g == 0) p.lse[bh * N + t] = (st.m + __log2f(l)) * kLn2 + fb.lse_shift;
        }
    } else {
        // merge the four wavefronts' states: thread (c, x) takes column c's
        // dims 4 x + [0, 4) (and 64 + ... at D = 128)
        __shared__ float s_m[WAVES][TILE], s_l[WAVES][TILE];
        __shared__ alignas(16) float s_o[WAVES][TILE][D + 4];
        store_acc<D>(&s_o[w][c][0], st.o, 1.0f, g);
        if (g == 0) {
            s_m[w][c] = st.m;
            s_l[w][c] = l;
        }
        __syncthreads();
        const int cc = threadIdx.x >> 4, x = threadIdx.x & 15, tt = q0 + cc;
        float m = s_m[0][cc];
#pragma unroll
        for (int i = 1; i < WAVES; ++i) m = fmaxf(m, s_m[i][cc]);
        float f[WAVES];
        l = 0.0f;
#pragma unroll
        for (int i = 0; i < WAVES; ++i) {
            // a wavefront with nothing valid for this column holds zeros
            f[i] = s_m[i][cc] == -INFINITY ? (s_l[i][cc] == 0.0f ? 0.0f : 1.0f)
                                           : __builtin_amdgcn_exp2f(s_m[i][cc] - m);
            l += s_l[i][cc] * f[i];
        }
        if (tt < N) {
#pragma unroll
            for (int hh = 0; hh < D / 64; ++hh) {
                f32x4 o = {};
#pragma unroll
                for (int i = 0; i < WAVES; ++i)
                    o += *reinterpret_cast<const f32x4 *>(&s_o[i][cc][64 * hh + 4 * x]) * f[i];
                *reinterpret_cast<f32x4 *>(out + tt * p.osn + 64 * hh + 4 * x) = o * (1.0f / l);
            }
            if (p.lse && x == 0) {
                const FusionBias fm = fusion_bias(p.gate[b * p.gsb + h * p.gsh + tt * p.gsn], clamp_on);
                p.lse[bh * N + tt] = (m + __log2f(l)) * kLn2 + fm.lse_shift;
            }
        }
    }
}

template <int D>
hipError_t launch_fwd(const FwdParams &p, hipStream_t stream) {
    const int n_qt = (p.N + TILE - 1) / TILE;
    const int64_t n_tiles = tiles_of((int64_t)p.B * p.H, p.N);
    const bool split = n_tiles <= kSplitTiles;
    const int64_t n_logical = split ? n_tiles : (n_tiles + WAVES - 1) / WAVES;
    return launch_kernel(split ? forward_f32_kernel<D, true> : forward_f32_kernel<D, false>,
                         dim3((unsigned)xcd_grid(n_logical)), dim3(NT), stream, p, n_qt, (uint32_t)n_tiles, (uint32_t)n_logical);
}

}  // namespace

hipError_t launch_forward_f32(const FwdParams &p, hipStream_t stream) {
    if ((int64_t)p.B * p.H * p.N == 0) return hipSuccess;
    if (one_per_row(p)) return launch_forward_rows_f32(p, stream);
    return p.D == 64 ? launch_fwd<64>(p, stream) : launch_fwd<128>(p, stream);
}

}  // namespace pi_attn
