// rows_f32.hip -- float32 forward and backward with one wavefront per row: for
// windows of a few entries and for sequences of a few rows, where a tile of 16
// columns (f32_tile.h) is mostly padding.
//
// Lane l holds elements l, l + 64, ... of the row.  The working set is visited
// entry by entry (partners, then the window oldest to newest); every score is a
// sum over the wavefront.  The backward's notation and formulas are those of
// backward_f32.hip: the query pass forms the row term, dq and the gate
// gradient, the key pass walks the queries whose working set holds its key.
#include <algorithm>

#include "f32_tile.h"
#include "kernels.h"
#include "pi_common.h"

namespace pi_attn {

namespace {

using f32::weight;

constexpr int NT = 256;   // four rows per work-group
constexpr int ROWS = NT / 64;

template <typename T>
__device__ inline T wave_sum(T x) {
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) x += __shfl_xor(x, o);
    return x;
}

template <int D>
struct Part {   // this lane's elements of a row
    float x[D / 64];
};

template <int D>
__device__ inline Part<D> load(const void *base, int64_t off, int lane) {
    Part<D> r;
#pragma unroll
    for (int e = 0; e < D / 64; ++e) r.x[e] = static_cast<const float *>(base)[off + lane + 64 * e];
    return r;
}

template <int D>
__device__ inline void store(float *row, const Part<D> &r, float f, int lane) {
#pragma unroll
    for (int e = 0; e < D / 64; ++e) row[lane + 64 * e] = r.x[e] * f;
}

template <int D>
__device__ inline float dot(const Part<D> &a, const Part<D> &b) {
    float s = 0.0f;
#pragma unroll
    for (int e = 0; e < D / 64; ++e) s += a.x[e] * b.x[e];
    return wave_sum(s);
}

template <int D>
__device__ inline void axpy(Part<D> &acc, float w, const Part<D> &r) {
#pragma unroll
    for (int e = 0; e < D / 64; ++e) acc.x[e] += w * r.x[e];
}

// This wavefront's row of a launch over B x H x N, if there is one.
struct Where {
    uint32_t row;
    int t, h, b;
    bool ok;

    __device__ explicit Where(const FwdParams &p) {
        row = __builtin_amdgcn_readfirstlane(blockIdx.x * ROWS + (threadIdx.x >> 6));
        ok = row < (uint32_t)p.B * p.H * p.N;
        const DivMod bh = divmod(row, p.N), head = divmod(bh.quot, p.H);
        t = (int)bh.rem;
        h = (int)head.rem;
        b = (int)head.quot;
    }
};

template <int D>
__global__ __launch_bounds__(NT) void forward_rows_f32_kernel(FwdParams p) {
    const Where w(p);
    if (!w.ok) return;
    const int lane = __lane_id(), t = w.t;
    const int64_t base = w.b * p.sb + w.h * p.sh;
    const Part<D> q = load<D>(p.q, base + t * p.sn, lane);
    const bool clamp_on = p.clamp > 0.0f;
    const FusionBias fb = fusion_bias(p.gate[w.b * p.gsb + w.h * p.gsh + t * p.gsn], clamp_on);

    const float c2 = p.scale * kLog2e;
    Part<D> acc = {};
    float m = -INFINITY, l = 0.0f;   // running max (log2 units) and sum
    auto visit = [&](int j, float bias) __attribute__((always_inline)) {
        const Part<D> k = load<D>(p.k_ptr, base + j * p.sn, lane), v = load<D>(p.v, base + j * p.sn, lane);
        const float x = dot<D>(q, k);
        const float s = clamp_on ? fminf(fmaxf(x * p.scale + bias, -p.clamp), p.clamp) * kLog2e
                                 : __builtin_fmaf(x, c2, bias * kLog2e);
        // a maximum that stays scales by exactly 1, also while it is -inf
        const float mn = fmaxf(m, s), c = s > m ? __builtin_amdgcn_exp2f(m - mn) : 1.0f;
        const float pr = __builtin_amdgcn_exp2f(s - (mn == -INFINITY ? 0.0f : mn));
        l = l * c + pr;
#pragma unroll
        for (int e = 0; e < D / 64; ++e) acc.x[e] = acc.x[e] * c + pr * v.x[e];
        m = mn;
    };
    const int jp = partner_of(t, p.k, p.pi), jf = p.causal ? -1 : partner_fwd_of(t, p.k, p.pi, p.N);
    if (jp >= 0) visit(jp, fb.partner);
    if (jf >= 0) visit(jf, fb.partner);
    const int hi = window_hi(t, p.k, p.N, p.causal);
    for (int j = window_lo(t, p.k); j <= hi; ++j) visit(j, fb.local);

    store<D>((float *)p.out + w.b * p.osb + w.h * p.osh + t * p.osn, acc, 1.0f / l, lane);
    if (p.lse && lane == 0) p.lse[w.row] = (m + __log2f(l)) * kLn2 + fb.lse_shift;
}

template <int D>
__global__ __launch_bounds__(NT) void backward_q_rows_f32_kernel(BwdParams bp) {
    const FwdParams &p = bp.f;
    const Where w(p);
    if (!w.ok) return;
    const int lane = __lane_id(), t = w.t;
    const int64_t base = w.b * p.sb + w.h * p.sh, obase = w.b * bp.osb + w.h * bp.osh + t * bp.osn;
    const Part<D> q = load<D>(p.q, base + t * p.sn, lane), o = load<D>(bp.dout, obase, lane);
    float r;
    {   // summed in 64 bits, as in the tiles: the gate gradient nearly cancels
        const Part<D> y = load<D>(bp.out, obase, lane);
        double s = 0.0;
#pragma unroll
        for (int e = 0; e < D / 64; ++e) s = __builtin_fma((double)o.x[e], (double)y.x[e], s);
        r = (float)wave_sum(s);
    }
    const float g = p.gate[w.b * p.gsb + w.h * p.gsh + t * p.gsn];
    const bool clamp_on = p.clamp > 0.0f;
    const FusionBias fb = fusion_bias(g, clamp_on);
    const float shift = fb.lse_shift - bp.lse[w.row];

    Part<D> dq = {};
    float d_win = 0.0f, d_par = 0.0f;   // sums of ddelta
    auto visit = [&](int j, float bias, float &sum) __attribute__((always_inline)) {
        const Part<D> k = load<D>(p.k_ptr, base + j * p.sn, lane), v = load<D>(p.v, base + j * p.sn, lane);
        bool cut;
        const float a = weight(dot<D>(q, k), bias, shift, p, clamp_on, cut), dp = dot<D>(o, v);
        const float dd = cut ? 0.0f : a * (dp - r);
        axpy<D>(dq, dd, k);
        sum += dd;
    };
    const int jp = partner_of(t, p.k, p.pi), jf = p.causal ? -1 : partner_fwd_of(t, p.k, p.pi, p.N);
    if (jp >= 0) visit(jp, fb.partner, d_par);
    if (jf >= 0) visit(jf, fb.partner, d_par);
    const int hi = window_hi(t, p.k, p.N, p.causal);
    for (int j = window_lo(t, p.k); j <= hi; ++j) visit(j, fb.local, d_win);

    store<D>(bp.dq + (int64_t)w.row * D, dq, p.scale, lane);
    if (lane == 0) {
        const GateDeriv gd = gate_deriv(g);
        bp.dgate[w.row] = d_win * gd.local + d_par * gd.partner;
        bp.rowterm[w.row] = r;
    }
}

template <int D>
__global__ __launch_bounds__(NT) void backward_kv_rows_f32_kernel(BwdParams bp) {
    const FwdParams &p = bp.f;
    const Where w(p);
    if (!w.ok) return;
    const int lane = __lane_id(), j = w.t;
    const int64_t base = w.b * p.sb + w.h * p.sh, obase = w.b * bp.osb + w.h * bp.osh;
    const float *gp = p.gate + w.b * p.gsb + w.h * p.gsh;
    const uint32_t row0 = w.row - j;   // of (b, h, 0)
    const Part<D> k = load<D>(p.k_ptr, base + j * p.sn, lane), v = load<D>(p.v, base + j * p.sn, lane);

    const bool clamp_on = p.clamp > 0.0f;
    Part<D> dk = {}, dv = {};
    auto visit = [&](int t, bool partner) __attribute__((always_inline)) {
        const Part<D> q = load<D>(p.q, base + t * p.sn, lane), o = load<D>(bp.dout, obase + t * bp.osn, lane);
        const FusionBias fb = fusion_bias(gp[t * p.gsn], clamp_on);
        bool cut;
        const float a = weight(dot<D>(q, k), partner ? fb.partner : fb.local, fb.lse_shift - bp.lse[row0 + t], p,
                               clamp_on, cut);
        const float dd = a * (dot<D>(o, v) - bp.rowterm[row0 + t]);
        axpy<D>(dk, cut ? 0.0f : dd, q);
        axpy<D>(dv, a, o);
    };
    // t in [j, j + k] and j + pi, bidirectionally also [j - k, j] and j - pi
    const int hi = window_hi(j, p.k, p.N, false);
    for (int t = p.causal ? j : window_lo(j, p.k); t <= hi; ++t) visit(t, false);
    const int tp = partner_fwd_of(j, p.k, p.pi, p.N), tm = p.causal ? -1 : partner_of(j, p.k, p.pi);
    if (tp >= 0) visit(tp, true);
    if (tm >= 0) visit(tm, true);

    store<D>(bp.dk + (int64_t)w.row * D, dk, p.scale, lane);
    store<D>(bp.dv + (int64_t)w.row * D, dv, 1.0f, lane);
}

dim3 grid_of(const FwdParams &p) { return dim3((unsigned)(((int64_t)p.B * p.H * p.N + ROWS - 1) / ROWS)); }

}  // namespace

// Which launches take these kernels: by estimates of a forward and a backward
// together, in units of about an entry's time where the chip is full (0.14 ns
// at D = 64, 0.08 at D = 128, less a common part).  Here a row's own chain, or
// all entries (at D = 64 also the rows).  In tiles, rounds of as many tiles as
// run at once (a wavefront per SIMD, or four per tile), each as long as the
// blocks of a tile's working sets.
//
// Both directions take the same way: a score then errs alike in the lse and in
// the weights made from it, and most of that cancels (otherwise dv errs 1.1 to
// 1.5 times as much).
//
// Measured with B H = 1 to 8192, N = 1 to 2048 and k = 0 to 24, causal and
// bidirectional, with and without partners (1602 pairs of launches): the two
// together take at most 1.15 (D = 64) and 1.26 (D = 128) times the shorter way,
// by more than 10 % in 32; a forward alone takes up to 1.05 and 1.33 times as
// long as in tiles where the backward gains more.  us, rows and tiles, D = 64
// causal unless given:
//   forward   B2 H8 N256 k1 4.5, 5.4;  k6 with partners 6.4, 5.5;
//             B1024 H8 N1 k0 5.5, 12.5;  B128 H8 N33 k0 14.5, 9.3
//   backward  B2 H8 N256 k1 9.7, 11.6;  k6 with partners 16.7, 12.1;
//             B1024 H8 N1 k0 11.6, 38.6;  B128 H8 N33 k4 54.6, 35.5
//   D = 128   B1 H8 N1000 k4 forward 7.4, 8.5, backward 21.4, 27.8;  k12 with
//             partners 15.2, 9.3 and 44.2, 29.5;  B8 H8 N2048 k1 52.7, 68.5 and
//             162, 264;  k12 with partners 167, 81 and 513, 310
bool one_per_row(const FwdParams &p) {
    const int64_t n = p.N, k = std::min<int64_t>(p.k, n - 1), sides = p.causal ? 1 : 2;
    const int64_t heads = p.B * (int64_t)p.H, rows = heads * n, tiles = f32::tiles_of(heads, p.N);
    if (rows * 64 + NT > (int64_t)UINT32_MAX) return false;   // the grid's threads must fit 32 bits
    const int64_t partners = partner_enabled(p.k, p.pi) ? std::max<int64_t>(0, n - p.pi) : 0;
    const int64_t entries = n + sides * (n * k - k * (k + 1) / 2 + partners);                  // of a head
    const int64_t blocks = (std::min(n, 16 + sides * k) + 15) / 16 + (partners ? sides : 0);   // of a tile
    if (entries > 64 * n) return false;   // far past every line below
    const bool split = tiles <= f32::kSplitTiles;
    const int64_t rounds = split ? (tiles + 255) / 256 : (tiles + 1023) / 1024;
    if (p.D == 64)
        return std::max(3800 * entries / n, 5 * rows / 2 + heads * entries) <=
               (split ? 8500 + rounds * (8700 + 3100 * blocks) : 8000 + rounds * (3700 + 12750 * blocks));
    return std::max(2000 * entries / n, heads * entries) <=
           (split ? 1000 + rounds * (7000 + 5100 * blocks) : rounds * (3100 + 17200 * blocks) + 7 * rows / 4);
}

hipError_t launch_forward_rows_f32(const FwdParams &p, hipStream_t stream) {
    return launch_kernel(p.D == 64 ? forward_rows_f32_kernel<64> : forward_rows_f32_kernel<128>, grid_of(p), dim3(NT),
                         stream, p);
}

hipError_t launch_backward_rows_f32(const BwdParams &p, hipStream_t stream) {
    const hipError_t e = launch_kernel(p.f.D == 64 ? backward_q_rows_f32_kernel<64> : backward_q_rows_f32_kernel<128>,
                                       grid_of(p.f), dim3(NT), stream, p);
    if (e != hipSuccess) return e;
    return launch_kernel(p.f.D == 64 ? backward_kv_rows_f32_kernel<64> : backward_kv_rows_f32_kernel<128>, grid_of(p.f),
                         dim3(NT), stream, p);
}

}  // namespace pi_attn
