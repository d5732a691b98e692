"""The bf16 forward's two ways of storing its rows: a launch of at least 1024
query tiles stores whole rows through LDS, a smaller one as the accumulator
lies.  The same heads, a few times and many times over, give the same output
to the bit: ragged tiles, both head dimensions, strided outputs, with the lse."""
import pytest
import torch

import paper_2511_10696_amd as pa
from paper_2511_10696_amd import workloads as W
from tests.test_gpu_backward_kv64 import many

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("D", [64, 128])
@pytest.mark.parametrize("N,k,pi", [(300, 40, 100), (129, 17, 18), (65, 100, 0), (1, 20, 30), (40, 17, 18), (41, 17, 18)])
@pytest.mark.parametrize("causal", [True, False])
@pytest.mark.parametrize("strided", [True, False])
def test_rows_stored_alike(device, D, N, k, pi, causal, strided):
    H = 2
    times = 1024 // (H * ((N + 127) // 128)) + 1
    cfg = W.ForwardConfig("custom", 1, H, N, D, k, pi, torch.bfloat16)
    q, kk, v, gate = W.forward_inputs(cfg, 61, device, per_query_gate=True)
    few, lse = pa.pi_attn_forward(q, kk, v, gate, k, pi, return_lse=True, causal=causal)
    shape = (1, N, H * times, D) if strided else (1, H * times, N, D)
    out = torch.full(shape, float("nan"), dtype=torch.bfloat16, device="cuda")
    out = out.transpose(1, 2) if strided else out
    big = [many(x, times) for x in (q, kk, v, gate)]
    for with_lse in (False, True):
        got = pa.pi_attn_forward(*big, k, pi, out=out.fill_(float("nan")), return_lse=with_lse, causal=causal)
        got = got if with_lse else (got, None)
        for i in (0, times - 1):
            assert torch.equal(got[0][:, H * i:H * (i + 1)], few)
            assert not with_lse or torch.equal(got[1][:, H * i:H * (i + 1)], lse)


@pytest.mark.parametrize("causal", [True, False])
@pytest.mark.parametrize("H,k", [(64, 32), (64, 64), (64, 65), (128, 16), (1030, 3000)])
def test_heads_first_alike(device, causal, H, k):
    """Both sides of the line between the work-group orders at D = 64 (heads
    times the window's rows): the order changes no bit."""
    N, few = 1100, 2
    cfg = W.ForwardConfig("custom", 1, few, N, 64, max(k, 17), 90, torch.bfloat16)
    q, kk, v, gate = W.forward_inputs(cfg, 63, device, per_query_gate=True)
    ref = pa.pi_attn_forward(q, kk, v, gate, cfg.k, cfg.pi, causal=causal)
    out = pa.pi_attn_forward(*(many(x, H // few).repeat(2, *[1] * (x.dim() - 1)) for x in (q, kk, v, gate)), cfg.k, cfg.pi,
                             causal=causal)
    assert torch.equal(out, ref.repeat(2, H // few, 1, 1))


def test_shard_queries_and_gradients_of_stride_zero(device):
    """Query (and dL/dy) rows of a shard call that are one row, repeated."""
    H, N, D, k, pi = 130, 300, 64, 40, 100
    cfg = W.ForwardConfig("custom", 1, H, N, D, k, pi, torch.bfloat16)
    q, kk, v, gate = W.forward_inputs(cfg, 62, device, per_query_gate=True)
    q0, do0 = (x[:, :, :1].expand(1, H, N, D) for x in (q, W.cotangent(q.shape, q.dtype, 62, device)))
    call = lambda x: pa.pi_attn_forward_shard(x, kk, v, gate, k, pi, N, 0, 0, return_lse=True)
    (out, lse), (ref, rlse) = call(q0), call(q0.contiguous())
    assert torch.equal(out, ref) and torch.equal(lse, rlse)
    rt = torch.rand((1, H, N), device="cuda")
    back = lambda x, d: pa.pi_attn_backward_shard_kv(x, kk, v, gate, k, pi, N, 0, 0, lse, rt, d)
    for a, b in zip(back(q0, do0), back(q0.contiguous(), do0.contiguous())):
        assert torch.equal(a, b)
