"""The binding's native calls against its Python path.

A call with no `stream` goes to the native module first, one that names the current stream takes
the Python path; both enqueue the same kernels, so outputs, caches and host positions are compared
bit for bit over the forms the entry points accept.  What the native module does not take
(subclasses, integers given as floats, other streams) still runs, and what was refused still raises.
"""
import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu

GH, GW, C, S, W, R, F0 = 5, 7, 2, 1, 4, 7, 9
T = GH * GW


def _u():
    import paper_2609_32518_amd as u
    return u


def _qkv(B, H, layout, seed):
    g = torch.Generator(device="cuda").manual_seed(seed)
    N = C * T
    if layout == "fused":
        return torch.randn((B, N, 3, H, 128), generator=g, device="cuda").bfloat16().unbind(2)
    if layout == "head_major":                       # head stride larger than the token stride is refused
        return [torch.randn((B, H, N, 128), generator=g, device="cuda").bfloat16().transpose(1, 2) for _ in range(3)]
    return [torch.randn((B, N, H, 128), generator=g, device="cuda").bfloat16() for _ in range(3)]


def _cache(u, B, H, seed):
    g = torch.Generator(device="cuda").manual_seed(seed)
    shape = (B, H, (S + R) * T, 128)
    k, v = (torch.randn(shape, generator=g, device="cuda").bfloat16() for _ in range(2))
    c = u.Cache(B, H, GH, GW, S, R, k_cache=k, v_cache=v)
    for f in range(F0):
        c.advance(f, 1)
    return c


def _same(a, b):
    assert torch.equal(a.view(torch.int16 if a.dtype == torch.bfloat16 else torch.int32),
                       b.view(torch.int16 if b.dtype == torch.bfloat16 else torch.int32))


@pytest.mark.parametrize("B,H,layout", [(1, 3, "contiguous"), (2, 2, "fused"), (1, 1, "fused"), (2, 5, "contiguous")])
@pytest.mark.parametrize("given", [False, True])
def test_native_equals_python(B, H, layout, given, monkeypatch):
    u = _u()
    cos, sin = u.unstep_rope_tables(F0, C, GH, GW)
    wq, wk = (torch.rand(H * 128, device="cuda").bfloat16() for _ in range(2))
    wo, x2 = torch.randn(64, H * 128, device="cuda").bfloat16(), torch.randn(64, device="cuda").bfloat16()
    taken = []
    for name in ("append", "append_qknorm", "window_attn", "step", "linear", "flow"):
        fn = getattr(u._calls, name)
        monkeypatch.setattr(u._calls, name, lambda *a, fn=fn, name=name: taken.append((name, r := fn(*a))) or r)
    res = []
    for stream in (None, torch.cuda.current_stream()):
        q, k, v = _qkv(B, H, layout, 1)
        c = _cache(u, B, H, 2)
        N = C * T
        mk = lambda: torch.empty((B, N, H, 128), dtype=torch.bfloat16, device="cuda") if given else None
        lse = torch.empty((B, H, N), device="cuda") if given else None
        kw = dict(stream=stream)
        out = [c.unstep_kv_append(F0, C, q, k, v, cos, sin, q_rot=mk(), **kw)]
        assert c.unstep_kv_append(F0, C, None, k, v, cos, sin, **kw) is None
        qr = c.unstep_kv_append_qknorm(F0, C, q, k, v, cos, sin, wq, wk, 1e-6, q_rot=mk(), **kw)
        for split in (True, False, True):            # the second split call finds the scratch the first one grew
            out.append(c.unstep_window_attn(F0, C, W, qr, out=mk(), lse=lse, use_split=split, **kw))
        o = c.unstep_step(F0, C, W, q, k, v, cos, sin, q_rot=mk(), out=mk(), lse=lse, **kw)
        y = u.unstep_linear(o.view(B, N, H * 128), wo, x2 if given else None,
                            out=torch.empty((B, N, 64), dtype=torch.bfloat16, device="cuda") if given else None, **kw)
        a, b = q.contiguous(), k.contiguous()
        rn = u.unstep_renoise(a, b, 0.02, out=mk(), **kw)
        em = u.unstep_emit(rn, b, 0.5, out=mk(), **kw)
        torch.cuda.synchronize()
        res.append(out + [qr, o, y, rn, em, c.k, c.v] + ([lse] if given else []))
        assert c.frame_map()[1] == F0 + C - 1
    for x, y in zip(*res):
        assert x.shape == y.shape
        _same(x, y)
    assert {n for n, r in taken} == {"append", "append_qknorm", "window_attn", "step", "linear", "flow"}
    assert all(r is not None for _, r in taken)


def test_other_forms_still_run_and_refusals_still_raise():
    u = _u()
    B, H, N = 1, 2, C * T
    cos, sin = u.unstep_rope_tables(F0, C, GH, GW)
    q, k, v = _qkv(B, H, "contiguous", 3)
    c = _cache(u, B, H, 4)
    want = c.unstep_step(F0, C, W, q, k, v, cos, sin)
    sub = lambda t: torch.nn.Parameter(t)
    _same(c.unstep_step(np.int32(F0), C, W, sub(q), k, v, cos, sin, softmax_scale=0), want)

    class Sub(torch.Tensor):
        pass

    _same(c.unstep_step(F0, C, W, q.as_subclass(Sub), k, v, cos, sin).as_subclass(torch.Tensor), want)
    side = torch.cuda.Stream()
    side.wait_stream(torch.cuda.current_stream())
    other = c.unstep_step(F0, C, W, q, k, v, cos, sin, stream=side)
    side.synchronize()
    _same(other, want)
    with torch.cuda.stream(side):                    # the current stream, wherever it is
        here = c.unstep_step(F0, C, W, q, k, v, cos, sin)
    side.synchronize()
    _same(here, want)

    step = lambda **kw: c.unstep_step(*[kw.get(n, d) for n, d in (("f0", F0), ("C", C), ("W", W), ("q", q), ("k", k),
                                                                  ("v", v), ("cos", cos), ("sin", sin))],
                                      **{n: kw[n] for n in ("out", "q_rot", "lse", "workspace") if n in kw})
    bad = [dict(q=None), dict(q=q.float()), dict(q=q[:, :-1]), dict(k=k.cpu()), dict(cos=cos.double()), dict(sin=sin[:-1]),
           dict(out=want[:, :-1]), dict(q_rot=want.float()), dict(lse=torch.empty(3, device="cuda")),
           dict(q=_qkv(B, H, "fused", 5)[0]), dict(workspace=torch.empty(8).cuda().expand(4, 8)[:, ::2])]
    for kw in bad:
        with pytest.raises(ValueError):
            step(**kw)
    for kw in (dict(f0=F0 + 5), dict(W=R + 1)):
        with pytest.raises(u.UnstepError):
            step(**kw)
    with pytest.raises(u.UnstepError):
        hq = _qkv(B, H, "head_major", 6)
        step(q=hq[0], k=hq[1], v=hq[2])
    x, w = torch.zeros(4, 16, device="cuda").bfloat16(), torch.zeros(8, 16, device="cuda").bfloat16()
    for args in ((x.float(), w), (x, w.t()), (x[:, :8], w), (x, w, torch.zeros(9, device="cuda").bfloat16()), (x, w.cpu())):
        with pytest.raises(ValueError):
            u.unstep_linear(*args)
    with pytest.raises(u.UnstepError):
        u.unstep_linear(torch.zeros(4, 12, device="cuda").bfloat16(), torch.zeros(8, 12, device="cuda").bfloat16())
    for args in ((x, x.float(), 0.5), (x, x[:2], 0.5), (x.t(), x.t(), 0.5)):
        with pytest.raises(ValueError):
            u.unstep_renoise(*args)
    with pytest.raises(u.UnstepError):
        u.unstep_emit(x, x, 1.5)
    torch.cuda.synchronize()
    assert c.frame_map()[1] == F0 + C - 1


@pytest.mark.parametrize("name", ["renoise", "emit"])
def test_update_in_place_is_applied_once_with_an_error_pending(name):
    """A HIP error that something else left on this thread is reported by the next launch, whose kernel has
    been enqueued: the call says so and does not enqueue it again."""
    import ctypes

    u = _u()
    f = getattr(u, f"unstep_{name}")
    x, y = (torch.randn(4096, device="cuda").bfloat16() for _ in range(2))
    once = f(x, y, 0.5)
    torch.cuda.synchronize()
    with open("/proc/self/maps") as maps:
        path = next(l.split()[-1] for l in maps if "libamdhip64" in l)
    hip, p = ctypes.CDLL(path), ctypes.c_void_p()
    assert hip.hipMalloc(ctypes.byref(p), ctypes.c_size_t(1 << 60)) != 0         # more than any device has
    try:
        with pytest.raises(u.UnstepError) as e:
            f(x, y, 0.5, out=x)
        assert e.value.code == u.E_HIP
    finally:
        hip.hipGetLastError()                                                   # leaves none behind
    torch.cuda.synchronize()
    _same(x, once)
    _same(f(x, y, 0.5, out=x), f(once, y, 0.5))
