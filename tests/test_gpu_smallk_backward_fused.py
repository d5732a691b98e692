"""The one-pass small-window backward (D = 64, k <= 8, launches of at least
49152 rows, sequences of more than a tile or two) against the two passes that
other launches take: the same heads, a few times and many times over.  Both sum the same float32 terms, at most 19
a row and 64 dimensions a score, in another order: they agree to 2e-6 of the
largest gradient, and the one pass meets the oracle at the bar of the two.
Runs with ragged ends and of one and several steps, reaches of 0, k and pi up
to their largest, the clamp, both gate forms, strided storage, and rows that
are not finite."""
import pytest
import torch

import oracle
import paper_2511_10696_amd as pa
from paper_2511_10696_amd import workloads as W
from tests.grad_check import check_backward
from tests.test_gpu_backward_kv64 import many

pytestmark = pytest.mark.gpu

SHAPES = [(517, 4, 16, True), (1000, 4, 16, False), (300, 0, 0, True), (300, 0, 0, False), (129, 8, 32, True),
          (2049, 3, 9, False), (641, 8, 16, False), (96, 8, 5, True), (33, 4, 31, True), (40, 5, 6, False),
          (700, 1, 16, False), (5, 4, 16, True),
          # sequences of a tile or two, on both sides of the lines between one pass and two
          (31, 8, 16, True), (33, 8, 16, True), (24, 4, 4, False), (25, 4, 4, False), (33, 4, 16, False),
          (32, 8, 9, False), (64, 8, 9, False), (65, 8, 16, False)]


def inputs(device, N, k, pi, pq, seed=51):
    cfg = W.ForwardConfig("custom", 1, 2, N, 64, k, pi, torch.bfloat16)
    q, kk, v, gate = W.forward_inputs(cfg, seed, device, per_query_gate=pq)
    return q, kk, v, gate, W.cotangent(q.shape, q.dtype, seed, device)


@pytest.mark.parametrize("N,k,pi,causal", SHAPES)
@pytest.mark.parametrize("pq,clamp", [(True, 0.0), (False, 2.5)])
def test_same_as_two_passes(device, N, k, pi, causal, pq, clamp):
    H, times = 2, 49152 // (2 * N) + 1
    q, kk, v, gate, do = inputs(device, N, k, pi, pq)
    opt = dict(causal=causal, logit_clamp=clamp)
    out, lse = pa.pi_attn_forward(q, kk, v, gate, k, pi, return_lse=True, **opt)
    opt["gate_grad_per_query"] = True
    rts = [torch.full((1, H * n, N), float("nan"), device="cuda") for n in (1, times)]
    few = pa.pi_attn_backward(q, kk, v, gate, k, pi, out, lse, do, rowterm=rts[0], **opt) + (rts[0],)
    big = [many(x, times) for x in (q, kk, v, gate, out, lse, do)]
    if pq:   # [B][N][H][D] storage
        big = [x.transpose(1, 2).contiguous().transpose(1, 2) if x.dim() == 4 else x for x in big]
    got = pa.pi_attn_backward(*big[:4], k, pi, *big[4:], rowterm=rts[1], **opt) + (rts[1],)
    for name, a, b in zip(("dq", "dk", "dv", "dgate", "rowterm"), few, got):
        assert torch.isfinite(b).all(), name
        for i in (0, times - 1):
            err = (a - b[:, H * i:H * (i + 1)]).abs().max().item()
            assert err <= 2e-6 * max(1.0, a.abs().max().item()), (name, err)


@pytest.mark.parametrize("causal,k,pi", [(True, 4, 16), (False, 8, 16), (True, 8, 32)])
def test_against_the_oracle(device, causal, k, pi):
    cfg = W.ForwardConfig("custom", 2, 48, 520, 64, k, pi, torch.bfloat16)
    q, kk, v, gate = W.forward_inputs(cfg, 52, device, per_query_gate=True)
    check_backward(q, kk, v, gate, k, pi, 52, causal=causal, per_head_sum=False)


@pytest.mark.parametrize("causal", [True, False])
@pytest.mark.parametrize("N,x", [(600, 250), (600, 586), (600, 13), (16, 2)])
def test_rows_not_finite(device, causal, N, x):
    """A row that is not finite reaches the rows whose working sets meet it
    (586, 13 and 2: also the partners of positions outside the sequence, whose
    windows hold its last and first rows)."""
    k, pi, times = 4, 16, 49152 // (2 * N) + 1
    q, kk, v, gate, do = (many(t, times) for t in inputs(device, N, k, pi, False))
    idx = oracle.index_set(N, k, pi, causal=causal)
    meets = torch.from_numpy((idx == x).any(1)).to(device)   # queries whose set holds x
    held = torch.zeros(N, dtype=torch.bool, device=device)   # keys in x's set
    held[torch.from_numpy(idx[x][idx[x] >= 0].astype("int64")).to(device)] = True
    one = torch.zeros_like(held)
    one[x] = True
    # the keys of x's queries, the queries of x's keys
    near_k = torch.from_numpy(oracle.index_set(N, k, pi, causal=causal)).to(device)
    touched = torch.zeros_like(held)
    touched[near_k[meets][near_k[meets] >= 0].long()] = True
    out, lse = pa.pi_attn_forward(q, kk, v, gate, k, pi, return_lse=True, causal=causal)
    opt = dict(causal=causal, gate_grad_per_query=True)
    clean = pa.pi_attn_backward(q, kk, v, gate, k, pi, out, lse, do, **opt)

    def poison(t):
        p = t.clone()
        p[:, :, x] = float("nan")
        return p

    for args, rows in (((q, poison(kk), v, do), (meets, touched, touched, meets)),
                       ((q, kk, poison(v), do), (meets, touched, one, meets)),
                       ((poison(q), kk, v, do), (one, held, held, one)),
                       ((q, kk, v, poison(do)), (one, held, held, one))):
        got = pa.pi_attn_backward(*args[:3], gate, k, pi, out, lse, args[3], **opt)
        for name, a, b, r in zip(("dq", "dk", "dv", "dgate"), clean, got, rows):
            assert torch.equal(a[:, :, ~r], b[:, :, ~r]), name


def test_more_heads_than_a_launch_of_one_each(device):
    """2^24 (b, h) of two rows: the two passes, which group heads, take the
    call (its inputs one batch entry, expanded)."""
    B, H, N, D = 1 << 20, 16, 2, 64
    q, kk, v, do = (torch.randn((1, H, N, D), generator=torch.Generator("cuda").manual_seed(55 + i), device="cuda")
                    .to(torch.bfloat16) for i in range(4))
    gate = torch.rand(H, device="cuda")
    out, lse = pa.pi_attn_forward(q, kk, v, gate, 2, 0, return_lse=True)
    few = pa.pi_attn_backward(q, kk, v, gate, 2, 0, out, lse, do, gate_grad_per_query=True)
    wide = lambda x: x.expand(B, *x.shape[1:])
    got = pa.pi_attn_backward(*map(wide, (q, kk, v)), gate, 2, 0, wide(out), wide(lse).contiguous(), wide(do),
                              gate_grad_per_query=True)
    for name, a, b in zip(("dq", "dk", "dv", "dgate"), few, got):
        for part in b.split(1 << 17):
            assert torch.equal(part, a.expand(part.shape)), name
