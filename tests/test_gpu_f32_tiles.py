"""The float32 forward and backward at the edges of their 16-row tiles: tile
and block remainders, windows around a block, partners next to the window, the
two launch forms (one wavefront per tile, four wavefronts per tile), strided
storage, and rows that are not finite outside a query's working set.  Bars:
forward max-abs 1e-4 and the backward's of grad_check.py (float32 sums of at
most 2k + 3 unit-scale terms err by well under either)."""
import numpy as np
import pytest
import torch

import oracle
import paper_2511_10696_amd as pa
from paper_2511_10696_amd import workloads as W
from tests.grad_check import check_backward
from tests.test_gpu_parity import LSE_TOL, assert_close, np32

pytestmark = pytest.mark.gpu

SHAPES = [(1, 1, 1, 64, 0, 0), (1, 2, 15, 128, 15, 16), (2, 1, 16, 64, 16, 17), (1, 1, 17, 128, 0, 1),
          (1, 3, 33, 64, 31, 32), (1, 1, 130, 64, 17, 40), (1, 1, 77, 128, 100, 0),
          (1, 32, 256, 64, 20, 50),     # 512 tiles: the most that are split
          (1, 32, 257, 64, 20, 50),     # 544: one wavefront per tile
          (1, 27, 305, 128, 3, 16)]     # 540, tiles of several heads in one work-group


@pytest.mark.parametrize("B,H,N,D,k,pi", SHAPES)
@pytest.mark.parametrize("causal", [True, False])
@pytest.mark.parametrize("pq", [True, False])
def test_f32_tiles(device, B, H, N, D, k, pi, causal, pq):
    cfg = W.ForwardConfig("custom", B, H, N, D, k, pi, torch.float32)
    q, kk, v, gate = W.forward_inputs(cfg, 11, device, per_query_gate=pq)
    if pq:   # [B][N][H][D] storage
        q, kk, v = (x.transpose(1, 2).contiguous().transpose(1, 2) for x in (q, kk, v))
    clamp = 20.0 if pq else 0.0   # never saturates here: |scale <q, k>| < 12
    out, lse = pa.pi_attn_forward(q, kk, v, gate, k, pi, logit_clamp=clamp, return_lse=True, causal=causal)
    torch.cuda.synchronize()
    ref, lref = oracle.forward(q, kk, v, gate, k, pi, clamp=clamp, want_lse=True, causal=causal)
    assert_close(np32(out), ref, torch.float32)
    assert np.abs(np32(lse) - lref).max() <= LSE_TOL * (10 if clamp else 1)
    check_backward(q, kk, v, gate, k, pi, 11, causal=causal, clamp=clamp, per_head_sum=False)


@pytest.mark.parametrize("causal", [True, False])
@pytest.mark.parametrize("H", [1, 40])   # both launch forms
@pytest.mark.parametrize("bad", [float("nan"), float("inf")])
def test_f32_rows_not_finite(device, causal, H, bad):
    """A key, value, query or dL/dy row that is not finite reaches exactly the
    rows whose working sets meet it; the others keep their bits."""
    B, N, D, k, pi, x = 1, 300, 64, 21, 50, 120
    cfg = W.ForwardConfig("custom", B, H, N, D, k, pi, torch.float32)
    q, kk, v, gate = W.forward_inputs(cfg, 12, device)
    do = W.cotangent(q.shape, q.dtype, 12, device)
    idx = oracle.index_set(N, k, pi, causal=causal)
    meets = torch.from_numpy((idx == x).any(1)).to(device)          # queries whose set holds x
    held = torch.zeros(N, dtype=torch.bool, device=device)          # keys in x's set
    held[torch.from_numpy(idx[x][idx[x] >= 0].astype(np.int64)).to(device)] = True
    out, lse = pa.pi_attn_forward(q, kk, v, gate, k, pi, return_lse=True, causal=causal)
    clean = pa.pi_attn_backward(q, kk, v, gate, k, pi, out, lse, do, gate_grad_per_query=True, causal=causal)

    def same_but(got, ref, rows):
        assert torch.equal(got[:, :, ~rows], ref[:, :, ~rows])

    def poison(t):
        p = t.clone()
        p[:, :, x] = bad
        return p

    for kx, vx in ((poison(kk), v), (kk, poison(v))):
        o, l = pa.pi_attn_forward(q, kx, vx, gate, k, pi, return_lse=True, causal=causal)
        same_but(o, out, meets)
        same_but(l, lse, meets)
        assert not torch.isfinite(o[:, :, x]).all()
        dq, dk, dv, dg = pa.pi_attn_backward(q, kx, vx, gate, k, pi, out, lse, do, gate_grad_per_query=True,
                                             causal=causal)
        same_but(dq, clean[0], meets)
        same_but(dg, clean[3], meets)
    for qx, dx in ((poison(q), do), (q, poison(do))):
        dq, dk, dv, dg = pa.pi_attn_backward(qx, kk, v, gate, k, pi, out, lse, dx, gate_grad_per_query=True,
                                             causal=causal)
        one = torch.zeros_like(held)
        one[x] = True
        same_but(dq, clean[0], one)
        same_but(dk, clean[1], held)
        same_but(dv, clean[2], held)


@pytest.mark.parametrize("B,H,N,k,pi,bound", [(1, 4, 600, 32, 64, 2.82e-7), (2, 8, 1000, 64, 128, 3.33e-7)])
def test_f32_score_error(device, B, H, N, k, pi, bound):
    """The error of dk at D = 128, which shows that of the scores, in both
    launch forms: as with scores summed by a tree over 64 lanes (2.71e-7 and
    3.22e-7, 4.6e-9 and 1.6e-9 between seeds; the bounds are 4 and 12
    deviations of a mean of three above them), where one chain over all dims
    gives 2.94e-7 and 3.47e-7."""
    errs = []
    for seed in range(90, 93):
        cfg = W.ForwardConfig("custom", B, H, N, 128, k, pi, torch.float32)
        q, kk, v, gate = W.forward_inputs(cfg, seed, device, per_query_gate=True)
        do = W.cotangent(q.shape, q.dtype, seed, device)
        out, lse = pa.pi_attn_forward(q, kk, v, gate, k, pi, return_lse=True)
        dk = np32(pa.pi_attn_backward(q, kk, v, gate, k, pi, out, lse, do)[1])
        ref = oracle.backward(q, kk, v, gate, k, pi, do)[1]
        errs.append(np.linalg.norm(dk - ref) / np.linalg.norm(ref))
    assert np.mean(errs) <= bound, errs
