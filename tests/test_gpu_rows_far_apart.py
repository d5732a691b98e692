"""Rows so far apart that a tile's span more than 1 GiB, or 2: positions before
the first row held still count as zeros, whatever lies in memory, and offsets
are right."""
import pytest
import torch

import paper_2511_10696_amd as pa
from paper_2511_10696_amd import workloads as W

pytestmark = pytest.mark.gpu


def test_key_shard(device):
    """dL/dy rows 4 MiB apart in a bidirectional key shard whose first row held
    lies off the 32-row grid of its band.  A row that is not finite, 1 GiB past
    the first one, reaches the keys within k of it and no block before them."""
    H, N, D, k, pi, step = 300, 420, 64, 70, 0, 1 << 21
    kpos0, nk = 128, 128
    qpos0, nqh = kpos0 - k, nk + 2 * k
    cfg = W.ForwardConfig("custom", 1, H, N, D, k, pi, torch.bfloat16)
    q, kk, v, gate = W.forward_inputs(cfg, 72, device, per_query_gate=True)
    q, gate = q[:, :, qpos0:qpos0 + nqh], gate[:, :, qpos0:qpos0 + nqh]
    kk, v = kk[:, :, kpos0:kpos0 + nk], v[:, :, kpos0:kpos0 + nk]
    lse, rt = torch.full((1, H, nqh), 3.0, device="cuda"), torch.zeros((1, H, nqh), device="cuda")
    far = torch.empty(((nqh - 1) * step + H * D,), dtype=torch.bfloat16, device="cuda").as_strided(
        (1, H, nqh, D), (0, D, step, 1))
    far.copy_(W.cotangent((1, H, nqh, D), torch.bfloat16, 72, device))
    far[:, :, 256] = float("nan")
    call = lambda d: pa.pi_attn_backward_shard_kv(q, kk, v, gate, k, pi, N, kpos0, qpos0, lse, rt, d, causal=False)
    for a, b in zip(call(far), call(far.contiguous())):
        assert torch.isfinite(b[:, :, :64]).all() and torch.equal(a[:, :, :64], b[:, :, :64])


@pytest.mark.parametrize("D", [64, 128])
@pytest.mark.parametrize("causal,k", [(True, 16), (False, 13), (False, 3)])
def test_small_window_backward(device, D, causal, k):
    """dL/dy and y rows that span 2 GiB per band of the small-window key pass:
    the gradients of the same rows side by side, to the bit."""
    H, N, pi = 2, 75, 20
    step = (1 << 30) // (31 + (1 if causal else 2) * k) // 128 * 128 + 128   # the band's rows: 32 + k or 32 + 2k
    cfg = W.ForwardConfig("custom", 1, H, N, D, k, pi, torch.bfloat16)
    q, kk, v, gate = W.forward_inputs(cfg, 73, device, per_query_gate=True)
    do = W.cotangent(q.shape, q.dtype, 73, device)
    y, lse = pa.pi_attn_forward(q, kk, v, gate, k, pi, return_lse=True, causal=causal)
    apart = [torch.empty(((N - 1) * step + H * D,), dtype=torch.bfloat16, device="cuda").as_strided(
        (1, H, N, D), (0, D, step, 1)) for _ in range(2)]
    apart[0].copy_(y)
    apart[1].copy_(do)
    got = pa.pi_attn_backward(q, kk, v, gate, k, pi, apart[0], lse, apart[1], causal=causal)
    for a, b in zip(got, pa.pi_attn_backward(q, kk, v, gate, k, pi, y, lse, do, causal=causal)):
        assert torch.equal(a, b)
