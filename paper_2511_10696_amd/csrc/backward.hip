// backward.hip -- dispatch of the backward of the full-sequence operator, and
// the sum of the per-query gate gradients of a per-head gate.
#include "kernels.h"
#include "pi_common.h"
#include "smallk.h"

namespace pi_attn {

namespace {

// One work-group per head: thread i sums entries t = i, i + 1024, ... of
// every batch row of the head into four fp64 partial sums (a fixed order,
// independent additions in flight), then a fixed-shape tree in LDS.
constexpr int kGateRedThreads = 1024;

__global__ __launch_bounds__(kGateRedThreads) void gate_grad_per_head_kernel(int B, int H, int N,
                                                                              const float *dgate, float *out) {
    __shared__ double part[kGateRedThreads];
    const int h = blockIdx.x;
    double acc[4] = {0.0, 0.0, 0.0, 0.0};
    for (int b = 0; b < B; ++b) {
        const float *row = dgate + ((int64_t)b * H + h) * N;
        int64_t t = threadIdx.x;
        for (; t + 3 * kGateRedThreads < N; t += 4 * kGateRedThreads) {
#pragma unroll
            for (int u = 0; u < 4; ++u) acc[u] += (double)row[t + u * kGateRedThreads];
        }
        // at most three entries remain for this thread
#pragma unroll
        for (int u = 0; u < 3; ++u)
            if (t + u * kGateRedThreads < N) acc[u] += (double)row[t + u * kGateRedThreads];
    }
    part[threadIdx.x] = (acc[0] + acc[1]) + (acc[2] + acc[3]);
    __syncthreads();
    for (int w = kGateRedThreads / 2; w > 0; w >>= 1) {
        if ((int)threadIdx.x < w) part[threadIdx.x] += part[threadIdx.x + w];
        __syncthreads();
    }
    if (threadIdx.x == 0) out[h] = (float)part[0];
}

}  // namespace

hipError_t launch_gate_grad_per_head(int B, int H, int N, const float *dgate, float *out, hipStream_t stream) {
    if (H == 0) return hipSuccess;
    return launch_kernel(gate_grad_per_head_kernel, dim3((unsigned)H), dim3(kGateRedThreads), stream, B, H, N,
                         dgate, out);
}

hipError_t launch_backward(const BwdParams &p, hipStream_t stream) {
    if ((int64_t)p.f.B * p.f.H * p.f.N == 0) return hipSuccess;
    if (p.dtype != 1) return launch_backward_f32(p, stream);
    if (p.f.k <= kSmallK) return launch_backward_smallk(p, stream);
    // the query pass computes its row terms and writes the exact ones for the key pass
    const hipError_t e = launch_backward_q_bf16(p, stream);
    return e != hipSuccess ? e : launch_backward_kv_bf16(p, stream);
}

}  // namespace pi_attn
