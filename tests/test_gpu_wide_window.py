"""A window radius far past the sequence (k near INT32_MAX) is dense attention:
forward, backward and key shard give what k = N - 1 gives, to the bit, on both
key passes at D = 64 and at D = 128, causal and bidirectional."""
import pytest
import torch

import paper_2511_10696_amd as pa
from paper_2511_10696_amd import workloads as W
from tests.test_gpu_backward_kv64 import many

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dtype", [torch.bfloat16, torch.float32])
@pytest.mark.parametrize("D,times", [(64, 1), (64, 60), (128, 1)])   # 60: past the line between the key passes
@pytest.mark.parametrize("causal", [True, False])
@pytest.mark.parametrize("k", [2 ** 31 - 1, 2 ** 31 - 200])
def test_same_as_dense(device, dtype, D, times, causal, k):
    H, N = 2, 300
    cfg = W.ForwardConfig("custom", 1, H, N, D, N - 1, 0, dtype)
    q, kk, v, gate = (many(x, times) for x in W.forward_inputs(cfg, 71, device, per_query_gate=True))
    do = many(W.cotangent((1, H, N, D), dtype, 71, device), times)
    res = []
    for kw in (N - 1, k):
        out, lse = pa.pi_attn_forward(q, kk, v, gate, kw, 0, return_lse=True, causal=causal)
        res.append((out, lse, *pa.pi_attn_backward(q, kk, v, gate, kw, 0, out, lse, do, causal=causal)))
    for name, a, b in zip(("out", "lse", "dq", "dk", "dv", "dgate"), *res):
        assert torch.equal(a, b), name
    if dtype == torch.bfloat16:
        lse, rt = res[0][1], torch.rand((1, H * times, N), device="cuda")
        shard = lambda kw: pa.pi_attn_backward_shard_kv(q, kk[:, :, 40:], v[:, :, 40:], gate, kw, 0, N, 40, 0, lse, rt,
                                                        do, causal=causal)
        for a, b in zip(shard(N - 1), shard(k)):
            assert torch.equal(a, b)
