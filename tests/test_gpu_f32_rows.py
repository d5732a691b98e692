"""The float32 forward and backward on either side of the lines between one
wavefront per row and tiles of 16: sequences of one row up, windows of a few
entries, both directions, clamps that cut, strided storage, and rows that are
not finite outside a working set.  Bars as in test_gpu_f32_tiles.py; sums are
over at most 2k + 3 unit-scale terms."""
import numpy as np
import pytest
import torch

import oracle
import paper_2511_10696_amd as pa
from paper_2511_10696_amd import workloads as W
from tests.grad_check import check_backward
from tests.test_gpu_parity import LSE_TOL, assert_close, np32

pytestmark = pytest.mark.gpu

# (B, H, N, D, k, pi): launches of up to 512 tiles (split over four wavefronts
# each) and of more, in one round and in two; most take rows causally and some
# tiles bidirectionally
SHAPES = [(1, 1, 1, 64, 0, 0), (2, 1, 2, 128, 1, 1), (1, 3, 5, 64, 2, 4), (1, 2, 16, 128, 7, 8), (1, 2, 17, 64, 2, 4),
          (1, 2, 130, 64, 5, 16), (1, 2, 130, 64, 6, 16), (1, 2, 130, 128, 9, 10), (1, 2, 130, 128, 12, 13),
          (1, 27, 150, 64, 4, 6), (1, 27, 150, 128, 7, 9), (2, 601, 1, 64, 0, 0), (1, 601, 18, 64, 2, 4),
          (1, 601, 18, 64, 6, 8), (1, 601, 18, 128, 1, 2), (1, 601, 18, 128, 10, 12), (1, 1040, 5, 64, 3, 4),
          (1, 1040, 12, 128, 8, 10)]


@pytest.mark.parametrize("B,H,N,D,k,pi", SHAPES)
@pytest.mark.parametrize("causal", [True, False])
@pytest.mark.parametrize("pq", [True, False])
def test_f32_rows(device, B, H, N, D, k, pi, causal, pq):
    cfg = W.ForwardConfig("custom", B, H, N, D, k, pi, torch.float32)
    q, kk, v, gate = W.forward_inputs(cfg, 21, device, per_query_gate=pq)
    if pq:   # [B][N][H][D] storage
        q, kk, v = (x.transpose(1, 2).contiguous().transpose(1, 2) for x in (q, kk, v))
    clamp = 1.0 if pq else 0.0   # cuts some of the unit-scale scores
    out, lse = pa.pi_attn_forward(q, kk, v, gate, k, pi, logit_clamp=clamp, return_lse=True, causal=causal)
    ref, lref = oracle.forward(q, kk, v, gate, k, pi, clamp=clamp, want_lse=True, causal=causal)
    assert_close(np32(out), ref, torch.float32)
    assert np.abs(np32(lse) - lref).max() <= LSE_TOL
    check_backward(q, kk, v, gate, k, pi, 21, causal=causal, clamp=20.0 if pq else 0.0, per_head_sum=False)


@pytest.mark.parametrize("D", [64, 128])
def test_f32_rows_minus_infinity(device, D):
    """Scores of -inf weigh nothing, the first of a set included."""
    cfg = W.ForwardConfig("custom", 1, 1, 40, D, 2, 7, torch.float32)
    q, kk, v, gate = W.forward_inputs(cfg, 23, device)
    q[..., 0] = 1.0
    kk[:, :, 5, 0] = -float("inf")   # first of t = 7's window, last of t = 5's, partner of t = 12
    out, lse = pa.pi_attn_forward(q, kk, v, gate, 2, 7, return_lse=True)
    kk[:, :, 5, 0] = -1e30
    ref, lref = oracle.forward(q, kk, v, gate, 2, 7, want_lse=True)
    assert_close(np32(out), ref, torch.float32)
    assert np.abs(np32(lse) - lref).max() <= LSE_TOL


@pytest.mark.parametrize("causal", [True, False])
@pytest.mark.parametrize("D", [64, 128])
def test_f32_rows_reach(device, causal, D):
    """A row that is not finite reaches the rows whose working sets meet it and
    no other, whose bits stay."""
    N, k, pi, x = 50, 2, 7, 20
    cfg = W.ForwardConfig("custom", 1, 1, N, D, k, pi, torch.float32)
    q, kk, v, gate = W.forward_inputs(cfg, 22, device)
    do = W.cotangent(q.shape, q.dtype, 22, device)
    idx = oracle.index_set(N, k, pi, causal=causal)
    meets = torch.from_numpy((idx == x).any(1)).to(device)
    held = torch.zeros(N, dtype=torch.bool, device=device)
    held[torch.from_numpy(idx[x][idx[x] >= 0].astype(np.int64)).to(device)] = True
    out, lse = pa.pi_attn_forward(q, kk, v, gate, k, pi, return_lse=True, causal=causal)

    def grads(q, kk, v, do):
        return pa.pi_attn_backward(q, kk, v, gate, k, pi, out, lse, do, gate_grad_per_query=True, causal=causal)

    def check(got, ref, rows):
        assert torch.equal(got[:, :, ~rows], ref[:, :, ~rows])
        assert not torch.isfinite(got[:, :, x]).all()

    def poison(t):
        p = t.clone()
        p[:, :, x] = float("nan")
        return p

    clean = grads(q, kk, v, do)
    for kx, vx in ((poison(kk), v), (kk, poison(v))):
        check(pa.pi_attn_forward(q, kx, vx, gate, k, pi, causal=causal), out, meets)
        check(grads(q, kx, vx, do)[0], clean[0], meets)
    for qx, dx in ((poison(q), do), (q, poison(do))):
        got = grads(qx, kk, v, dx)
        check(got[1], clean[1], held)
        if dx is not do:
            check(got[2], clean[2], held)
