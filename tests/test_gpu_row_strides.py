"""Row strides below the head dimension: rows that are one row repeated (stride
0, an expanded tensor) and rows that overlap, in q, k, v, dL/dy and the forward
output.  Every path gives what the same values in contiguous storage give, to
the bit."""
import pytest
import torch

import paper_2511_10696_amd as pa
from paper_2511_10696_amd import workloads as W

pytestmark = pytest.mark.gpu


def rows(B, H, N, D, step, dtype, seed):
    """[B, H, N, D] whose rows start `step` elements apart."""
    g = torch.Generator("cuda").manual_seed(seed)
    x = torch.randn((B, H, (N - 1) * step + D), generator=g, device="cuda").to(dtype)
    return x.as_strided((B, H, N, D), (H * x.size(2), x.size(2), step, 1))


# banded (both head dimensions, few and many work-groups), small windows in two passes and in one
PATHS = [(64, 3, 300, 40, 100), (64, 90, 400, 40, 100), (128, 3, 300, 40, 100), (64, 3, 100, 4, 16), (128, 3, 100, 8, 30),
         (64, 3, 100, 16, 30), (64, 500, 100, 4, 16)]


@pytest.mark.parametrize("D,H,N,k,pi", PATHS)
@pytest.mark.parametrize("causal", [True, False])
@pytest.mark.parametrize("step", [0, 16])
def test_same_as_contiguous(device, D, H, N, k, pi, causal, step):
    q, kk, v, do = (rows(1, H, N, D, step, torch.bfloat16, 80 + i) for i in range(4))
    gate = torch.rand((1, H, N), device="cuda")
    u, w2 = (torch.randn(s, device="cuda").to(torch.bfloat16) for s in ((1, N, 64), (H, 64)))
    res = []
    for c in (lambda x: x, lambda x: x.contiguous()):
        args = [c(x) for x in (q, kk, v)]
        out, lse = pa.pi_attn_forward(*args, gate, k, pi, return_lse=True, causal=causal)
        gated = pa.pi_attn_forward_gated(*args, u, w2, None, k, pi, causal=causal)
        # y and dL/dy share strides: a row of each in the same storage form
        y = c(rows(1, H, N, D, step, torch.bfloat16, 90))
        grads = pa.pi_attn_backward(*args, gate, k, pi, y, lse, c(do), causal=causal)
        res.append((out, lse, *gated, *grads))
    for name, a, b in zip(("out", "lse", "gated", "gate", "dq", "dk", "dv", "dgate"), *res):
        assert torch.equal(a, b), name
