"""The decode step at the edges of its wavefront split: windows of one row more
and less than whole chunks (a chunk is 8 load instructions of 1 KiB), partner
present, absent and next to the window, with four and eight wavefronts per
work-group, both sides of each line of that choice.  Bars as in
test_gpu_parity.py."""
import numpy as np
import pytest
import torch

import oracle
import paper_2511_10696_amd as pa
from tests.test_gpu_parity import LSE_TOL, assert_close, np32

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dtype,D", [(torch.bfloat16, 64), (torch.bfloat16, 128), (torch.float32, 64),
                                     (torch.float32, 128)])
@pytest.mark.parametrize("S,H", [(8, 2), (8, 33)])   # 16 and 264 work-groups
@pytest.mark.parametrize("chunks", [4, 5, 8, 9])
def test_decode_chunk_edges(device, dtype, D, S, H, chunks):
    rpc = 8 * 1024 // (D * (2 if dtype == torch.bfloat16 else 4))   # rows per chunk
    k = chunks * rpc
    pi, cap = k + 1, k + 40
    lens_np = np.array([0, 1, rpc - 1, rpc, rpc + 1, k, k + 1, cap - 1], np.int32)
    g = torch.Generator(device="cuda").manual_seed(31)
    kc, vc = (torch.randn(S, H, cap, D, generator=g, device="cuda").to(dtype) for _ in range(2))
    gate = torch.rand(H, generator=g, device="cuda") * 2 - 1
    qn, kn, vn = (torch.randn(S, H, D, generator=g, device="cuda").to(dtype) for _ in range(3))
    # rows past the length are never read
    for s, t in enumerate(lens_np):
        kc[s, :, t:], vc[s, :, t:] = float("nan"), float("nan")
    kc_ref, vc_ref = np32(kc), np32(vc)
    lens, lse = torch.tensor(lens_np, device="cuda"), torch.empty(S, H, device="cuda")
    out = pa.pi_attn_decode_step(lens, qn, kn, vn, kc, vc, gate, k, pi, lse=lse)
    torch.cuda.synchronize()
    ref, lref = oracle.decode_step(lens_np, qn, kn, vn, kc_ref, vc_ref, gate, k, pi, want_lse=True)
    assert_close(np32(out), ref, dtype)
    assert np.abs(np32(lse) - lref).max() <= LSE_TOL
    for s, t in enumerate(lens_np):
        assert torch.equal(kc[s, :, t], kn[s]) and torch.equal(vc[s, :, t], vn[s])


@pytest.mark.parametrize("dtype", [torch.bfloat16, torch.float32])
def test_partner_of_weight_zero(device, dtype):
    """A partner whose logit is -inf has weight 0: of its value, an infinity
    makes NaN (0 times inf) where it stands, as it does in a window row, and
    nothing else shows."""
    D, k, pi, t = 64, 40, 70, 90
    g = torch.Generator(device="cuda").manual_seed(32)
    kc, vc = (torch.randn(1, 2, 128, D, generator=g, device="cuda").to(dtype) for _ in range(2))
    qn, kn, vn = (torch.randn(1, 2, D, generator=g, device="cuda").to(dtype) for _ in range(3))
    qn[..., 0] = 1.0
    kc[:, :, t - pi, 0], vc[:, :, t - pi, 5] = -float("inf"), float("inf")
    lens = torch.tensor([t], dtype=torch.int32, device="cuda")
    gate = torch.zeros(2, device="cuda")
    out = pa.pi_attn_decode_step(lens, qn, kn, vn, kc.clone(), vc.clone(), gate, k, pi)
    assert torch.isnan(out[..., 5]).all()
    out[..., 5] = 0
    assert torch.isfinite(out).all()
