"""The key pass at D = 64 of launches with more than 256 work-groups of 128
keys (one wavefront per 32 keys) against the wavefront pairs of smaller
launches: the same heads, a few times and many times over, give the same
gradients to the bit.  Ragged tiles, windows around a tile, partners next to
the window and past the band, the clamp, strided gradients, shards whose rows
start off the tile grid; and the oracle's gradients at the bf16 bar."""
import pytest
import torch

import paper_2511_10696_amd as pa
from paper_2511_10696_amd import workloads as W
from tests.grad_check import check_backward
from tests.test_gpu_shard import q_rows_for_keys

pytestmark = pytest.mark.gpu

SHAPES = [(500, 40, 100), (513, 17, 18), (129, 64, 65), (250, 300, 0), (1000, 128, 256), (97, 31, 50)]


def many(x, times, head_dim=1):
    """x with its heads `times` times over."""
    return x.repeat(times) if x.dim() == 1 else x.repeat([times if d == head_dim else 1 for d in range(x.dim())])


@pytest.mark.parametrize("N,k,pi", SHAPES)
@pytest.mark.parametrize("causal", [True, False])
@pytest.mark.parametrize("pq,clamp", [(True, 0.0), (False, 2.5)])
def test_same_as_pairs(device, N, k, pi, causal, pq, clamp):
    H = 2
    times = 256 // (H * ((N + 127) // 128)) + 1   # just past the line
    cfg = W.ForwardConfig("custom", 1, H, N, 64, k, pi, torch.bfloat16)
    q, kk, v, gate = W.forward_inputs(cfg, 41, device, per_query_gate=pq)
    do = W.cotangent(q.shape, q.dtype, 41, device)
    out, lse = pa.pi_attn_forward(q, kk, v, gate, k, pi, return_lse=True, causal=causal, logit_clamp=clamp)
    opt = dict(causal=causal, logit_clamp=clamp, gate_grad_per_query=True)
    few = pa.pi_attn_backward(q, kk, v, gate, k, pi, out, lse, do, **opt)
    big = [many(x, times) for x in (q, kk, v, gate, out, lse, do)]
    if pq:   # [B][N][H][D] storage of out and dL/dy
        big[4], big[6] = (x.transpose(1, 2).contiguous().transpose(1, 2) for x in (big[4], big[6]))
    got = pa.pi_attn_backward(*big[:4], k, pi, *big[4:], **opt)
    for name, a, b in zip(("dq", "dk", "dv", "dgate"), few, got):
        for i in (0, times - 1):
            assert torch.equal(a, b[:, H * i:H * (i + 1)]), name


@pytest.mark.parametrize("causal", [True, False])
def test_shards_same_as_pairs(device, causal):
    """Key shards of a sequence, the query rows held starting off the 32-row
    grid of the band."""
    H, N, k, pi = 2, 700, 40, 130
    cfg = W.ForwardConfig("custom", 1, H, N, 64, k, pi, torch.bfloat16)
    q, kk, v, gate = W.forward_inputs(cfg, 42, device, per_query_gate=True)
    do = W.cotangent(q.shape, q.dtype, 42, device)
    out, lse = pa.pi_attn_forward(q, kk, v, gate, k, pi, return_lse=True, causal=causal)
    rt = torch.empty((1, H, N), device="cuda")
    pa.pi_attn_backward(q, kk, v, gate, k, pi, out, lse, do, causal=causal, rowterm=rt)
    for s0, s1 in ((0, 100), (101, 450), (450, 700)):
        lo, hi = q_rows_for_keys(N, k, pi, causal, s0, s1 - s0)
        args = [q[:, :, lo:hi], kk[:, :, s0:s1], v[:, :, s0:s1], gate[:, :, lo:hi], lse[:, :, lo:hi].contiguous(),
                rt[:, :, lo:hi].contiguous(), do[:, :, lo:hi]]
        call = lambda a: pa.pi_attn_backward_shard_kv(*a[:4], k, pi, N, s0, lo, *a[4:], causal=causal)
        few, got = call(args), call([many(x, 130) for x in args])
        for a, b in zip(few, got):
            assert torch.equal(a, b[:, :H]) and torch.equal(a, b[:, -H:])


@pytest.mark.parametrize("causal", [True, False])
def test_against_the_oracle(device, causal):
    cfg = W.ForwardConfig("custom", 2, 44, 333, 64, 50, 120, torch.bfloat16)   # 264 work-groups
    q, kk, v, gate = W.forward_inputs(cfg, 43, device, per_query_gate=True)
    check_backward(q, kk, v, gate, 50, 120, 43, causal=causal, per_head_sum=False)
