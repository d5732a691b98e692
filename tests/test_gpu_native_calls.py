"""The native marshalling of the hot entry points (csrc/binding.cpp) against the
Python code that serves every other call: the same results to the bit over the
forms that it accepts (strides, gate shapes, given buffers, argument types), the
same error for what is refused, and the caller's stream."""
import threading

import pytest
import torch

import paper_2511_10696_amd as pa

pytestmark = pytest.mark.gpu


class NoNative:
    """Stands in for the native module: every call goes to the Python code."""

    def __getattr__(self, name):
        return lambda *a: None


def in_python(monkeypatch, call):
    pa._load_native()
    with monkeypatch.context() as m:
        m.setattr(pa, "_native", NoNative())
        return call()


def flat(x):
    return list(x) if isinstance(x, tuple) else [x]


def rnd(*shape, dtype=torch.bfloat16, seed=0):
    return torch.randn(shape, generator=torch.Generator("cuda").manual_seed(seed), device="cuda").to(dtype)


def qkv(B, H, N, D, dtype, layout):
    if layout == "bnhd":
        return tuple(rnd(B, N, H, D, dtype=dtype, seed=i).transpose(1, 2) for i in range(3))
    if layout == "rows":   # rows of a wider buffer
        return tuple(rnd(B, H, N, 3, D, dtype=dtype, seed=i)[:, :, :, i] for i in range(3))
    return tuple(rnd(B, H, N, D, dtype=dtype, seed=i) for i in range(3))


@pytest.mark.parametrize("dtype", [torch.float32, torch.bfloat16])
@pytest.mark.parametrize("layout", ["bhnd", "bnhd", "rows"])
@pytest.mark.parametrize("B,gate", [(2, "head"), (1, "head"), (2, "query"), (2, "head strided"), (2, "query expanded")])
@pytest.mark.parametrize("given", [False, True])
def test_sequence_calls(device, monkeypatch, dtype, layout, B, gate, given):
    H, N, D, k, pi = 3, 70, 64, 20, 33
    q, kk, v = qkv(B, H, N, D, dtype, layout)
    g = {"head": lambda: rnd(H, dtype=torch.float32), "query": lambda: rnd(B, H, N, dtype=torch.float32),
         "head strided": lambda: rnd(H, 2, dtype=torch.float32)[:, 1],
         "query expanded": lambda: rnd(B, 1, N, dtype=torch.float32).expand(B, H, N)}[gate]()
    opt = dict(causal=False, logit_clamp=5, scale=0.1) if given else {}
    buf = lambda *s, dt=torch.float32: torch.empty(s, dtype=dt, device="cuda")
    fwd = lambda: pa.pi_attn_forward(q, kk, v, g, k, pi, **(dict(
        out=buf(B, N, H, D, dt=dtype).transpose(1, 2), lse=buf(B, H, N)) if given else dict(return_lse=True)), **opt)
    out, lse = fwd()
    pout, plse = in_python(monkeypatch, fwd)
    assert torch.equal(out, pout) and torch.equal(lse, plse) and out.stride() == pout.stride()
    plain = pa.pi_attn_forward(q, kk, v, g, k, pi, **opt)
    assert isinstance(plain, torch.Tensor) and torch.equal(plain, in_python(
        monkeypatch, lambda: pa.pi_attn_forward(q, kk, v, g, k, pi, **opt)))
    do = rnd(B, H, N, D, dtype=dtype, seed=9)
    if given:
        do = do.transpose(1, 2).contiguous().transpose(1, 2)
    for per_query in (False, True):
        bwd = lambda: pa.pi_attn_backward(q, kk, v, g, k, pi, out, lse, do, gate_grad_per_query=per_query, **(dict(
            dq=buf(B, H, N, D), dgate=buf(B, H, N), rowterm=buf(B, H, N)) if given else {}), **opt)
        for a, b in zip(bwd(), in_python(monkeypatch, bwd)):
            assert a.shape == b.shape and a.dtype == b.dtype and torch.equal(a, b)
    native = pa._native.forward(q, kk, v, g, k, pi, None, 0.0, None, False, None, None, True)
    assert isinstance(native, torch.Tensor), "this call is plain"


@pytest.mark.parametrize("bias,k", [(True, 4), (False, 4), (True, 40)])
def test_gated_and_decode(device, monkeypatch, bias, k):
    B, H, N, D, dh = 2, 3, 50, 64, 32
    q, kk, v = qkv(B, H, N, D, torch.bfloat16, "bhnd")
    u, w2 = rnd(B, N, dh), rnd(H, dh, seed=1)
    b2 = rnd(H, dtype=torch.float32) if bias else None
    for opt in (dict(), dict(return_lse=True, causal=False)):
        call = lambda: pa.pi_attn_forward_gated(q, kk, v, u, w2, b2, k, 16, **opt)
        got, ref = flat(call()), flat(in_python(monkeypatch, call))
        assert len(got) == len(ref) and all(torch.equal(a, b) for a, b in zip(got, ref))
    assert pa._native.forward_gated(q, kk, v, u, w2, b2, k, 16, None, 0.0, None, False, None, None, None, True)
    for dtype in (torch.bfloat16, torch.float32):
        kc, vc = rnd(B, H, N, D, dtype=dtype), rnd(B, H, N, D, dtype=dtype, seed=1)
        qn, kn, vn = (rnd(B, H, D, dtype=dtype, seed=i) for i in range(3))
        ln, lo = torch.tensor([7, 30], dtype=torch.int32, device="cuda"), torch.empty(2, dtype=torch.int32, device="cuda")
        for gate in (rnd(H, dtype=torch.float32), rnd(B, H, dtype=torch.float32), rnd(H, B, dtype=torch.float32).t()):
            lse = [torch.empty(B, H, device="cuda") for _ in range(2)]
            a = pa.pi_attn_decode_step(ln, qn, kn, vn, kc, vc, gate, k, 16, len_out=lo, lse=lse[0])
            b = in_python(monkeypatch, lambda: pa.pi_attn_decode_step(ln, qn, kn, vn, kc, vc, gate, k, 16, lse=lse[1]))
            assert torch.equal(a, b) and torch.equal(lse[0], lse[1]) and torch.equal(lo, ln + 1)
        assert pa._native.decode_step(ln, qn, kn, vn, kc, vc, gate, k, 16, None, 0.0, None, None, None, None) is not None


def test_refused_calls(device, monkeypatch):
    """The same exception, to the word, whichever code meets the call first."""
    B, H, N, D = 1, 2, 40, 64
    q, kk, v = qkv(B, H, N, D, torch.bfloat16, "bhnd")
    g, f32 = rnd(H, dtype=torch.float32), torch.float32
    out, lse = pa.pi_attn_forward(q, kk, v, g, 20, 30, return_lse=True)
    F, G = pa.pi_attn_forward, pa.pi_attn_backward
    other = rnd(B, N, H, D).transpose(1, 2)
    cases = [lambda: F(q, kk, v.float(), g, 20, 30), lambda: F(q, other, v, g, 20, 30),
             lambda: F(q, kk, v[:, :, :8], g, 20, 30), lambda: F(q, kk, v, g.double(), 20, 30),
             lambda: F(q, kk, v, rnd(H + 1, dtype=f32), 20, 30), lambda: F(q.cpu(), kk, v, g, 20, 30),
             lambda: F(q, kk, v, g, -1, 30), lambda: F(q, kk, v, g, 20, 30, scale=-1.0),
             lambda: F(q, kk, v, g, 20, 30, logit_clamp=float("nan")),
             lambda: F(q, kk, v, g, 20, 30, logit_clamp=None),
             lambda: F(q, kk, v, g, 20, 30, out=rnd(B, H, N, D, dtype=f32)),
             lambda: F(q, kk, v, g, 20, 30, lse=rnd(B, H, N)), lambda: F(q[0], kk[0], v[0], g, 20, 30),
             lambda: F(*(rnd(B, H, N, 32),) * 3, g, 20, 30), lambda: F(*(rnd(B, H, N, 68)[..., 2:66],) * 3, g, 20, 30),
             lambda: F(q.half(), kk.half(), v.half(), g, 20, 30),
             lambda: G(q, kk, v, g, 20, 30, out, lse[..., :8], out), lambda: G(q, kk, v, g, 20, 30, out, lse, out.float()),
             lambda: G(q, kk, v, g, 20, 30, out, lse, out, dq=rnd(B, H, N, D)),
             lambda: pa.pi_attn_decode_step(torch.zeros(1, device="cuda"), q[:, :, 0], q[:, :, 0], q[:, :, 0], kk, v, g, 4, 9),
             lambda: pa.pi_attn_forward_gated(q, kk, v, rnd(B, N, 12), rnd(H, 12), None, 4, 16)]
    for i, call in enumerate(cases):
        with pytest.raises(Exception) as a:
            call()
        with pytest.raises(Exception) as b:
            in_python(monkeypatch, call)
        assert type(a.value) is type(b.value) and str(a.value) == str(b.value), i


def test_unusual_calls_take_python(device, monkeypatch):
    """Accepted as before, by the Python code: no rows, a given stream,
    arguments of other number types, strides that need a copy."""
    q, kk, v = qkv(1, 2, 40, 64, torch.bfloat16, "bhnd")
    g = rnd(2, dtype=torch.float32)
    ref, lse = pa.pi_attn_forward(q, kk, v, g, 20, 30, return_lse=True)
    assert pa.pi_attn_forward(q[:, :, :0], kk[:, :, :0], v[:, :, :0], g, 20, 30).shape == (1, 2, 0, 64)
    assert torch.equal(pa.pi_attn_forward(q, kk, v, g, 20.0, torch.tensor(30), causal=1), ref)
    side = torch.cuda.Stream()
    side.wait_stream(torch.cuda.current_stream())
    got = pa.pi_attn_forward(q, kk, v, g, 20, 30, stream=side)
    torch.cuda.synchronize()
    assert torch.equal(got, ref)
    do = rnd(1, 40, 2, 64).transpose(1, 2)   # other strides than out's
    a = pa.pi_attn_backward(q, kk, v, g, 20, 30, ref, lse, do)
    b = pa.pi_attn_backward(q, kk, v, g, 20, 30, ref, lse, do.contiguous())
    assert all(torch.equal(x, y) for x, y in zip(a, b))


def test_streams_threads_and_graphs(device):
    q, kk, v = qkv(1, 4, 300, 64, torch.bfloat16, "bhnd")
    g = rnd(4, dtype=torch.float32)
    ref = pa.pi_attn_forward(q, kk, v, g, 20, 30)
    torch.cuda.synchronize()
    got = {}

    def work(i):
        s = torch.cuda.Stream()
        with torch.cuda.stream(s):
            got[i] = [pa.pi_attn_forward(q, kk, v, g, 20, 30) for _ in range(20)]
            s.synchronize()

    ts = [threading.Thread(target=work, args=(i,)) for i in range(4)]
    [t.start() for t in ts]
    [t.join() for t in ts]
    assert all(torch.equal(x, ref) for xs in got.values() for x in xs)
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        out = pa.pi_attn_forward(q, kk, v, g, 20, 30)
    for i in range(3):
        q.mul_(0.5)
        graph.replay()
        torch.cuda.synchronize()
        assert torch.equal(out, pa.pi_attn_forward(q, kk, v, g, 20, 30))


def test_refused_launch_is_not_repeated(device, monkeypatch):
    """A launch that the HIP runtime refuses -- 2^24 work-groups of 256 -- ends
    the call in the native code: the Python code does not issue it again."""
    B, H = 1 << 20, 16
    q, kk, v = (rnd(1, 1, 1, 64, seed=i).expand(B, H, 1, 64) for i in range(3))
    entered = []
    monkeypatch.setattr(pa, "_stream_handle", lambda *a: entered.append(a))
    with pytest.raises(pa.PiAttnError, match="^pi_attn_forward: ") as e:
        pa.pi_attn_forward(q, kk, v, rnd(H, dtype=torch.float32), 17, 20)
    assert e.value.status == -3 and not entered
    try:   # the runtime's last error, which the next launch of torch reports
        torch.zeros(1, device="cuda")
    except RuntimeError:
        pass
    torch.cuda.synchronize()
