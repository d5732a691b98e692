"""The bf16 query pass's two ways of storing dq: launches of at least 256 tiles
of more than 32 rows store whole rows through LDS, others as the accumulator
lies.  The same heads, a few times and many times over, give the same gradients
to the bit: ragged tiles, both head dimensions, strided inputs, a shard."""
import pytest
import torch

import paper_2511_10696_amd as pa
from paper_2511_10696_amd import workloads as W
from tests.test_gpu_backward_kv64 import many

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("D", [64, 128])
@pytest.mark.parametrize("N,k,pi", [(300, 40, 100), (129, 17, 18), (33, 20, 0), (32, 20, 0)])
@pytest.mark.parametrize("causal", [True, False])
@pytest.mark.parametrize("strided", [True, False])
def test_rows_stored_alike(device, D, N, k, pi, causal, strided):
    H = 2
    times = 256 // (H * ((N + 127) // 128))   # at the line
    cfg = W.ForwardConfig("custom", 1, H, N, D, k, pi, torch.bfloat16)
    q, kk, v, gate = W.forward_inputs(cfg, 64, device, per_query_gate=True)
    do = W.cotangent(q.shape, q.dtype, 64, device)
    out, lse = pa.pi_attn_forward(q, kk, v, gate, k, pi, return_lse=True, causal=causal)
    few = pa.pi_attn_backward_shard_q(q, kk, v, gate, k, pi, N, 0, 0, out, lse, do, causal=causal)
    q, kk, v, gate, out, lse, do = (many(x, times) for x in (q, kk, v, gate, out, lse, do))
    if strided:
        q, kk, v, out, do = (x.transpose(1, 2).contiguous().transpose(1, 2) for x in (q, kk, v, out, do))
    got = pa.pi_attn_backward_shard_q(q, kk, v, gate, k, pi, N, 0, 0, out, lse, do, causal=causal,
                                      dq=torch.full(q.shape, float("nan"), device="cuda"))
    for name, a, b in zip(("dq", "dgate", "rowterm"), few, got):
        for i in (0, times - 1):
            assert torch.equal(a, b[:, H * i:H * (i + 1)]), name
