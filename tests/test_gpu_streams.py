"""The kernels of 32-row workgroups (small calls: bf16 forward, and the backward
in one launch beyond 128 keys) against the fp64 oracle and against an explicit
tile and the three separate passes on the same inputs."""
import math

import numpy as np
import pytest

import synth
from parity_util import TOL, compare, note, oracle_fwd_bwd, to_dev, to_np

pytestmark = pytest.mark.gpu

C, K, N = synth.MASK_CAUSAL, synth.MASK_KEY_PADDING, synth.MASK_NONE
CASES = [  # name, B, S_q, S_kv, Hq, Hkv, d, dtype, mask, launches of the backward
    ("below", 1, 135, 0, 4, 4, 64, "bf16", C, 3),          # 135 keys: three launches
    ("first", 1, 136, 0, 4, 4, 64, "bf16", C, 1),
    ("ragged", 2, 257, 0, 4, 2, 64, "bf16", C | K, 1),     # one row into a ninth block; a batch without keys
    ("one_query", 2, 1, 300, 4, 4, 64, "bf16", K, 1),      # fewer query blocks than wavefronts
    ("cross", 2, 95, 161, 4, 2, 32, "bf16", N, 1),
    ("wide", 1, 200, 0, 4, 4, 128, "bf16", C, 1),          # K and V rows in registers
    ("gqa_wide", 1, 70, 333, 8, 2, 128, "bf16", K, 1),
    ("f32_d64", 1, 161, 0, 4, 2, 64, "f32", C, 1),
    ("f32_d32", 2, 33, 400, 2, 1, 32, "f32", K, 1),
    ("f32_d128", 1, 150, 0, 2, 2, 128, "f32", C, 1),
    ("f32_short", 2, 65, 0, 2, 2, 64, "f32", K, 1),        # up to 128 keys
]


@pytest.mark.parametrize("name,B,Sq,Skv,Hq,Hkv,d,dt,mask,launches", CASES, ids=[c[0] for c in CASES])
def test_streams(name, B, Sq, Skv, Hq, Hkv, d, dt, mask, launches):
    import torch
    import paper_2607_21624_amd as fbl
    w = synth.Workload(name, B=B, S=Sq, Hq=Hq, Hkv=Hkv, d=d, dtype=dt, mask=mask, seed=Sq + d, len_lo=0,
                       len_hi=Skv or Sq, S_kv=Skv)
    inp = synth.make_inputs(w)
    if inp["kv_len"] is not None and B > 1:
        inp["kv_len"][0] = 0
    note(f"streams {name} B={B} Sq={Sq} Skv={w.Skv} Hq={Hq} Hkv={Hkv} d={d} {dt} mask={mask} kv_len={inp['kv_len']}")
    q, k, v, do = (to_dev(inp[n], dt) for n in ("q", "k", "v", "do"))
    kv_len = None if inp["kv_len"] is None else torch.from_numpy(inp["kv_len"].astype(np.int32)).to("cuda")
    causal, scale = bool(mask & C), 1.0 / math.sqrt(d)
    lq, lk = fbl.layout_of(q, Hq), fbl.layout_of(k, Hkv)
    ws_full = fbl.fbl_attn_bwd_workspace(lq, lk)
    assert fbl.attn_bwd_launches(lq, lk, mask, ws_full) == launches
    o, lse = fbl.attn_fwd(q, k, v, Hq, Hkv, scale, causal, kv_len)
    one = fbl.attn_bwd(q, k, v, o, do, lse, Hq, Hkv, scale, causal, kv_len)
    again = fbl.attn_bwd(q, k, v, o, do, lse, Hq, Hkv, scale, causal, kv_len)
    ws = torch.empty(ws_full, dtype=torch.uint8, device="cuda")
    outs = [torch.full_like(t, float("nan")) for t in (q, k, v)]
    for ph in (fbl.FBL_BWD_PREP, fbl.FBL_BWD_KV, fbl.FBL_BWD_Q):
        fbl.attn_bwd(q, k, v, o, do, lse, Hq, Hkv, scale, causal, kv_len, dq=outs[0], dk=outs[1], dv=outs[2],
                     workspace=ws, phases=ph)
    tiled = (o, lse)
    if dt == "bf16":
        tiled = fbl.attn_fwd(q, k, v, Hq, Hkv, scale, causal, kv_len, tile=0)
    torch.cuda.synchronize()
    for a_, b_ in zip(one, again):
        assert torch.equal(a_, b_), "not repeatable"
    ref = oracle_fwd_bwd(inp)
    for label, (oo, ll), res in (("automatic", (o, lse), one), ("tile 0, three passes", tiled, outs)):
        got = {"o": to_np(oo), "lse": to_np(ll), "dq": to_np(res[0]), "dk": to_np(res[1]), "dv": to_np(res[2])}
        errs, bad = compare(got, ref, dt)
        note(f"{label} rel errs {errs}")
        assert not bad, f"{name} {label}: {bad} (tol {TOL[dt]})"


def test_streams_rows_past_the_end_do_not_leak():
    """The last block's rows past S_q and S_kv lie in other tensors' memory: here
    NaN, which must not reach any result."""
    import torch
    import paper_2607_21624_amd as fbl
    S, T, H, d = 37, 141, 2, 64
    gen = torch.Generator(device="cuda")
    gen.manual_seed(3)
    for dt in (torch.bfloat16, torch.float32):
        def framed(rows):
            buf = torch.full((1, rows + 64, H * d), float("nan"), dtype=dt, device="cuda")
            buf[:, :rows] = torch.randn((1, rows, H * d), generator=gen, device="cuda").to(dt)
            return buf, buf[:, :rows]
        (bq, q), (bk, k), (bv, v), (bo, do) = framed(S), framed(T), framed(T), framed(S)
        ob, o = framed(S)
        o_, lse = fbl.attn_fwd(q, k, v, H, H, out=o)
        res = fbl.attn_bwd(q, k, v, o, do, lse, H, H)
        plain = [t.contiguous() for t in (q, k, v, o, do)]
        want = fbl.attn_bwd(*plain, lse, H, H)
        torch.cuda.synchronize()
        for got, ref in zip((o, lse) + tuple(res), (plain[3], lse) + tuple(want)):
            assert torch.isfinite(got).all() and torch.equal(got, ref)


@pytest.mark.parametrize("d", [32, 64, 128])
@pytest.mark.parametrize("dt", ["bfloat16", "float32"])
def test_streams_masked_rows_may_hold_anything_finite(dt, d):
    """Key padding over values so large that the masked scores and dP overflow
    to inf and nan: every result is that of zeros in their place, and the masked
    keys' gradients are zeros, also where dO is nan.  A causal pair (query 0, key
    100) whose dP overflows reaches no gradient either."""
    import torch
    import paper_2607_21624_amd as fbl
    dt = getattr(torch, dt)
    B, S, H = 2, 161, 2
    g = torch.Generator(device="cuda")
    g.manual_seed(d)
    q, k, v, do = (torch.randn(B, S, H * d, generator=g, device="cuda").to(dt) for _ in range(4))
    lens = torch.tensor([141, 40], dtype=torch.int32, device="cuda")
    big, zero = [], []
    for t, x in ((k, 1e30), (v, 3e38)):
        big.append(t.clone())
        zero.append(t.clone())
        for b in range(B):
            big[-1][b, lens[b]:] = x
            zero[-1][b, lens[b]:] = 0
    note(f"masked rows {dt} d={d}")

    def run(k, v, do=do, kv_len=lens, causal=False):
        o, lse = fbl.attn_fwd(q, k, v, H, H, causal=causal, kv_len=kv_len)
        r = (o, lse) + fbl.attn_bwd(q, k, v, o, do, lse, H, H, causal=causal, kv_len=kv_len)
        torch.cuda.synchronize()
        return r

    got, want = run(*big), run(*zero)
    for a, b in zip(got, want):
        assert torch.isfinite(a).all() and torch.equal(a, b)
    bad = do.clone()
    bad[:, 7] = float("nan")
    for name, t in zip(("dk", "dv"), run(*big, do=bad)[3:]):
        for b in range(B):
            assert (t[b, lens[b]:] == 0).all(), name
    far, wide = do.clone(), v.clone()
    far[:, 0], wide[:, 100] = 1e20, 1e20  # their product is past the fp32 range; every allowed pair's is not
    for t in run(k, wide, do=far, kv_len=None, causal=True):
        assert torch.isfinite(t).all()
