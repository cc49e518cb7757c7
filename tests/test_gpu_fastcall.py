"""The binding's native call path (csrc/fastcall.cpp) against its general path:
every form the native path takes gives the general path's bits, and what is not
a plain call is left to the general path (which checks and raises)."""
import types

import pytest

pytestmark = pytest.mark.gpu

NAMES = ("attn_fwd", "attn_bwd", "attn_fwd_packed", "attn_bwd_packed", "proj")


def _modules(monkeypatch):
    from paper_2607_21624_amd import fbl
    native = fbl._FAST
    taken = []

    def counted(name):
        def f(*a):
            r = getattr(native, name)(*a)
            taken.append(r is not None)
            return r
        return f

    return fbl, taken, types.SimpleNamespace(**{n: counted(n) for n in NAMES}), \
        types.SimpleNamespace(**{n: (lambda *a: None) for n in NAMES})


def _both(monkeypatch, fbl, native, general, call):
    import torch
    out = []
    for path in (native, general):
        monkeypatch.setattr(fbl, "_FAST", path)
        r = call()
        torch.cuda.synchronize()
        out.append([t.clone() for t in (r if isinstance(r, tuple) else (r,))])
    assert all(torch.equal(a, b) and a.dtype == b.dtype and a.stride() == b.stride() for a, b in zip(*out))


def _qkv(dt, B, S, T, Hq, Hkv, d, seed):
    import torch
    g = torch.Generator(device="cpu").manual_seed(seed)
    mk = lambda s, h: torch.randn(B, s, h * d, generator=g).to("cuda", dt)
    return mk(S, Hq), mk(T, Hkv), mk(T, Hkv), mk(S, Hq)


@pytest.mark.parametrize("dt", ["bfloat16", "float32"])
@pytest.mark.parametrize("form", ["plain", "outputs", "views", "padded", "grad"])
def test_attention_forms(monkeypatch, dt, form):
    import torch
    fbl, taken, native, general = _modules(monkeypatch)
    dt = getattr(torch, dt)
    B, S, Hq, Hkv, d = 2, 161, 4, 2, 64
    q, k, v, do = _qkv(dt, B, S, S, Hq, Hkv, d, 3)
    kw = {}
    if form == "views":  # column and token views of wider buffers
        wide = lambda t: torch.nn.functional.pad(t, (0, 64, 0, 5))[:, :t.shape[1], :t.shape[2]]
        q, k, v, do = (wide(t) for t in (q, k, v, do))
    if form == "padded":
        kw = dict(kv_len=torch.tensor([S, 40], dtype=torch.int32, device="cuda"), scale=0.25)
    if form == "grad":
        q = torch.nn.Parameter(q)
        kw = dict(causal=True)
    outs = {}
    if form == "outputs":
        kw = dict(causal=True)
        outs = dict(out=torch.empty_like(q), lse=torch.empty(B, Hq, S, device="cuda"))
    _both(monkeypatch, fbl, native, general, lambda: fbl.attn_fwd(q, k, v, Hq, Hkv, **kw, **outs))
    o, lse = fbl.attn_fwd(q, k, v, Hq, Hkv, **kw)
    if form == "outputs":
        outs = dict(dq=torch.empty_like(q), dk=torch.empty_like(k), dv=torch.empty_like(v),
                    workspace=torch.empty(fbl.fbl_attn_bwd_workspace(fbl.layout_of(q, Hq), fbl.layout_of(k, Hkv)),
                                          dtype=torch.uint8, device="cuda"))
    _both(monkeypatch, fbl, native, general, lambda: fbl.attn_bwd(q, k, v, o, do, lse, Hq, Hkv, **kw, **outs))
    if form == "outputs" and dt == torch.bfloat16:  # named tiles, single phases
        _both(monkeypatch, fbl, native, general, lambda: fbl.attn_fwd(q, k, v, Hq, Hkv, causal=True, tile=2))
        for phase in (fbl.FBL_BWD_PREP, fbl.FBL_BWD_KV, fbl.FBL_BWD_Q):
            _both(monkeypatch, fbl, native, general,
                  lambda: fbl.attn_bwd(q, k, v, o, do, lse, Hq, Hkv, causal=True, phases=phase, kv_tile=5, **outs))
    assert taken and all(taken)


@pytest.mark.parametrize("causal", [False, True])
def test_packed_and_projection_forms(monkeypatch, causal):
    import torch
    fbl, taken, native, general = _modules(monkeypatch)
    g = torch.Generator(device="cpu").manual_seed(5)
    Hq, Hkv, d = 4, 2, 64
    qkv = torch.randn(2, 100, (Hq + 2 * Hkv) * d, generator=g).to("cuda", torch.bfloat16)
    do = torch.randn(2, 100, Hq * d, generator=g).to("cuda", torch.bfloat16)
    _both(monkeypatch, fbl, native, general, lambda: fbl.attn_fwd_packed(qkv, Hq, Hkv, causal=causal))
    o, lse = fbl.attn_fwd_packed(qkv, Hq, Hkv, causal=causal)
    for dqkv in (None, torch.empty_like(qkv)):
        _both(monkeypatch, fbl, native, general,
              lambda: fbl.attn_bwd_packed(qkv, o, do, lse, Hq, Hkv, causal=causal, dqkv=dqkv))
    for dt in (torch.bfloat16, torch.float32):
        x, w, dy = (torch.randn(s, generator=g).to("cuda", dt) for s in ((72, 144), (144, 200), (72, 200)))
        x, w, dy = x[:, 8:136], w[:128, :192], dy[:, :192]  # views: row strides above the widths
        wide = torch.empty(72, 256, dtype=dt, device="cuda")
        for args in ((0, x, w), (1, dy, w), (2, x, dy)):
            _both(monkeypatch, fbl, native, general, lambda: fbl.proj(*args))
        _both(monkeypatch, fbl, native, general, lambda: fbl.proj(0, x, w, out=wide[:, 8:200]))
    assert taken and all(taken)


def test_other_calls_go_to_the_general_path(monkeypatch):
    import torch
    from paper_2607_21624_amd import fbl
    F = fbl._FAST
    q, k, v, do = _qkv(torch.bfloat16, 1, 64, 64, 2, 2, 64, 1)
    fwd = lambda q=q, k=k, v=v, Hq=2, Hkv=2, scale=None, causal=False, kv_len=None, out=None, lse=None, stream=None, \
        tile=-1: F.attn_fwd(q, k, v, Hq, Hkv, scale, causal, kv_len, out, lse, stream, tile)
    assert fwd() is not None

    class Sub(torch.Tensor):
        pass

    lens = torch.tensor([64], device="cuda")
    for bad in (dict(q=q.cpu()), dict(q=q.as_subclass(Sub)), dict(q=q.half()), dict(q=q.transpose(1, 2)), dict(q=q[0]),
                dict(q=torch._neg_view(q)), dict(k=k.float()), dict(Hq=3), dict(Hq=0), dict(scale=1), dict(causal=1),
                dict(kv_len=lens), dict(kv_len=lens.int()[:0]), dict(lse=torch.empty(1, 2, 63, device="cuda")),
                dict(out=torch.empty_like(q).float()), dict(stream=torch.cuda.Stream()), dict(stream=0), dict(tile=99),
                dict(q=None), dict(q=q.data_ptr()), dict(out=q)):
        assert fwd(**bad) is None, bad
    x = q[0]
    for bad in ((3, x, x, None, -1, None), (0, x.half(), x, None, -1, None), (0, x.t(), x, None, -1, None),
                (0, x, x.float(), None, -1, None), (0, x, x, x, -1, None), (0, x, x.cpu(), None, -1, None)):
        assert F.proj(*bad) is None
    e = lambda *s: torch.empty(s, dtype=torch.bfloat16, device="cuda")
    X, W, dY = e(32, 64), e(64, 96), e(32, 96)  # operands that disagree, outputs of another shape: refused by both
    for bad in ((0, X, W[:56], None), (0, X, e(72, 96), None), (1, dY, W[:, :88], None), (1, dY[:, :88], W, None),
                (2, X, dY[:24], None), (2, X[:24], dY, None), (0, X, W, e(31, 96)), (0, X, W, e(33, 96)),
                (0, X, W, e(32, 104)), (1, dY, W, e(32, 72)), (2, X, dY, e(56, 96))):
        assert F.proj(*bad, -1, None) is None
        with pytest.raises(fbl.FblError) as err:
            fbl.proj(*bad)
        assert err.value.status == fbl.FBL_ERR_SHAPE
        if bad[3] is not None:
            with pytest.raises(fbl.FblError):
                fbl.proj_tune(*bad)
    with pytest.raises(fbl.FblError):
        fbl.attn_fwd(q, k, v, 2, 2, tile=99)
    with torch.cuda.stream(torch.cuda.Stream()):  # the current stream, whichever it is
        torch.cuda.current_stream().wait_stream(torch.cuda.default_stream())
        o, _ = fwd()
    torch.cuda.synchronize()
    assert torch.equal(o, fwd()[0])
