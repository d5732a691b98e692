"""The decode step at the edges of its wavefront split: windows of one row more
and less than whole chunks (up to 8 load instructions of 1 KiB), partner
present, absent and next to the window, with one to eight wavefronts per (s, h),
both sides of each line of that choice.  Bars as in test_gpu_parity.py."""
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


@pytest.mark.parametrize("dtype,D", [(torch.bfloat16, 64), (torch.bfloat16, 128), (torch.float32, 64),
                                     (torch.float32, 128)])
@pytest.mark.parametrize("S,H", [(8, 4), (8, 129), (8, 256)])   # 32, 1032 and 2048 (s, h)
@pytest.mark.parametrize("loads", [0, 1, 2, 3, 5, 9])
def test_decode_short_windows(device, dtype, D, S, H, loads):
    """Windows of a few load instructions; the heads of a few (oracle) many
    times over give the same rows in every copy."""
    few = 4
    rpi = 1024 // (D * (2 if dtype == torch.bfloat16 else 4))   # rows per load instruction
    k = max(0, loads * rpi - (loads > 3))
    pi, cap = k + 1, k + 30
    lens_np = np.array([0, 1, max(k - 1, 2), k + 1, k + 2, k + 3, cap - 2, cap - 1], np.int32)
    g = torch.Generator(device="cuda").manual_seed(33)
    rnd = lambda *s: torch.randn(s, generator=g, device="cuda").to(dtype)
    kc, vc, qn, kn, vn = rnd(S, few, cap, D), rnd(S, few, cap, D), rnd(S, few, D), rnd(S, few, D), rnd(S, few, D)
    gate = torch.rand(few, generator=g, device="cuda") * 2 - 1
    for s, t in enumerate(lens_np):   # rows past the length are never read
        kc[s, :, t:], vc[s, :, t:] = float("nan"), float("nan")
    ref, lref = oracle.decode_step(lens_np, qn, kn, vn, np32(kc), np32(vc), gate, k, pi, want_lse=True)
    times = (H + few - 1) // few
    rep = lambda x: x.repeat_interleave(times, 1)[:, :H].contiguous()
    kcb, vcb, lse = rep(kc), rep(vc), torch.empty(S, H, device="cuda")
    lens, lout = torch.tensor(lens_np, device="cuda"), torch.empty(S, dtype=torch.int32, device="cuda")
    out = pa.pi_attn_decode_step(lens, rep(qn), rep(kn), rep(vn), kcb, vcb, gate.repeat_interleave(times)[:H], k, pi,
                                 lse=lse, len_out=lout)
    assert torch.equal(lout, lens + 1)
    for i in range(0, H, times):
        assert torch.equal(out[:, i:i + times], out[:, i:i + 1].expand(-1, min(times, H - i), -1))
        assert_close(np32(out[:, i]), ref[:, i // times], dtype)
        assert np.abs(np32(lse[:, i]) - lref[:, i // times]).max() <= LSE_TOL
    for s, t in enumerate(lens_np):
        assert torch.equal(kcb[s, :, t], rep(kn)[s]) and torch.equal(vcb[s, :, t], rep(vn)[s])


def test_rows_kept_or_not(device):
    """Steps of more and of less than 12 MB of window rows (kept in the caches
    or not): the same sequence in either gives the same output."""
    H, D, k, pi, t = 8, 128, 300, 400, 450
    g = torch.Generator(device="cuda").manual_seed(34)
    kc, vc = (torch.randn((1, H, 460, D), generator=g, device="cuda").to(torch.bfloat16) for _ in range(2))
    qn, kn, vn = (torch.randn((1, H, D), generator=g, device="cuda").to(torch.bfloat16) for _ in range(3))
    gate = torch.zeros(H, device="cuda")
    step = lambda S: pa.pi_attn_decode_step(torch.full((S,), t, dtype=torch.int32, device="cuda"), *(
        x.repeat(S, *([1] * (x.dim() - 1))) for x in (qn, kn, vn, kc, vc)), gate, k, pi)
    few, many = step(2), step(30)   # 2.5 and 37 MB
    assert torch.equal(few[:1].expand(30, -1, -1), many)


def test_more_heads_than_a_launch_of_wide_groups(device):
    """2^24 (s, h) of float32 caches of one row: the new row alone."""
    S, H, D = 1 << 20, 16, 64
    kc, vc = (torch.zeros((S, H, 1, D), device="cuda") for _ in range(2))
    x = torch.randn((S, H, D), generator=torch.Generator("cuda").manual_seed(35), device="cuda")
    lens, gate = torch.zeros(S, dtype=torch.int32, device="cuda"), torch.zeros(H, device="cuda")
    out = pa.pi_attn_decode_step(lens, x, x, x, kc, vc, gate, 0, 0)
    assert torch.equal(out, x) and torch.equal(kc[:, :, 0], x) and torch.equal(vc[:, :, 0], x)


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


@pytest.mark.parametrize("dtype,D,k", [(torch.bfloat16, 128, 517), (torch.float32, 64, 513)])
def test_decode_paced(device, dtype, D, k):
    """A step of more than 400 MB of window rows: three of its sequences, one
    shorter than a chunk, against the oracle."""
    S, H, pi, cap = 64, 32, k + 3, k + 20
    g = torch.Generator(device="cuda").manual_seed(37)
    kc, vc = (torch.randn(S, H, cap, D, generator=g, device="cuda", dtype=dtype) for _ in range(2))
    qn, kn, vn = (torch.randn(S, H, D, generator=g, device="cuda", dtype=dtype) for _ in range(3))
    gate = torch.rand(H, generator=g, device="cuda") * 2 - 1
    lens = torch.full((S,), cap - 1, device="cuda", dtype=torch.int32)
    lens[5], lens[63] = 3, k
    pick = [0, 5, 63]
    for s in pick:   # rows past the length are never read
        kc[s, :, lens[s]:], vc[s, :, lens[s]:] = float("nan"), float("nan")
    kc_ref, vc_ref = np32(kc[pick]), np32(vc[pick])
    out = pa.pi_attn_decode_step(lens, qn, kn, vn, kc, vc, gate, k, pi)
    ref = oracle.decode_step(lens[pick].cpu().numpy(), qn[pick], kn[pick], vn[pick], kc_ref, vc_ref, gate, k, pi)
    assert_close(np32(out[pick]), ref, dtype)
    assert torch.isfinite(out).all()
