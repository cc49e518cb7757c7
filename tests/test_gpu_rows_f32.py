"""The fp32 kernels of 128-row workgroups (short walks over grids of whole rounds:
forward at d = 64 and 128, the backward's kv and dQ passes at d = 128) against the fp64
oracle, and that they are what such calls dispatch."""
import numpy as np
import pytest

import synth
from parity_util import compare, gpu_fwd_bwd, note, oracle_fwd_bwd, select_heads

pytestmark = pytest.mark.gpu

C, K, N = synth.MASK_CAUSAL, synth.MASK_KEY_PADDING, synth.MASK_NONE
CASES = [  # B, S_q, S_kv, Hq, Hkv, d, mask, kernels
    (16, 100, 33, 16, 16, 64, N, ("fwd",)),      # one tile of 64 keys, half of it past the end
    (16, 128, 128, 16, 4, 64, C, ("fwd",)),      # whole tiles, every mask on the diagonal
    (16, 250, 130, 16, 16, 64, K, ("fwd",)),     # two blocks of rows, three tiles, rows past S_q; a batch without keys
    (16, 97, 320, 16, 16, 64, N, ("fwd",)),      # the longest walk
    (16, 500, 50, 16, 4, 128, K, ("fwd",)),      # d = 128: one tile
    (16, 33, 33, 16, 16, 128, N, ("kv", "q")),   # two query blocks, wavefronts without rows
    (16, 100, 100, 16, 16, 128, C, ("kv", "q")),
    (16, 128, 128, 16, 16, 128, K, ("kv", "q")),
    (8, 250, 250, 16, 16, 128, N, ("kv", "q")),  # two blocks of rows, ragged
    (16, 70, 200, 16, 16, 128, K, ("kv",)),      # dQ in 32-row workgroups beside it
]


@pytest.mark.parametrize("B,Sq,Skv,Hq,Hkv,d,mask,kernels", CASES)
def test_rows_kernels(B, Sq, Skv, Hq, Hkv, d, mask, kernels):
    import bench
    w = synth.Workload("rows", B=B, S=Sq, S_kv=Skv, Hq=Hq, Hkv=Hkv, d=d, dtype="f32", mask=mask, seed=Sq + d, len_lo=1,
                       len_hi=Skv)
    inp = synth.make_inputs(w)
    if inp["kv_len"] is not None:
        inp["kv_len"][0] = 0
    note(f"rows B={B} Sq={Sq} Skv={Skv} Hq={Hq} Hkv={Hkv} d={d} mask={mask}")
    got = gpu_fwd_bwd(inp)
    heads = sorted({0, Hkv // 2, Hkv - 1})  # independent of each other; every batch
    errs, bad = compare(select_heads(got, w, heads), oracle_fwd_bwd(inp, heads), "f32")
    assert not bad, (bad, errs)
    again = gpu_fwd_bwd(inp)
    assert all(np.array_equal(got[n], again[n]) for n in got)
    ran = bench.dispatched_kernels(lambda: gpu_fwd_bwd(inp))
    if ran is not None:
        for k in kernels:
            assert any(f"_{k}_rows_f32" in n for n in ran), (k, ran)


@pytest.mark.parametrize("Sq,Skv,d", [(128, 128, 64), (128, 128, 128), (500, 50, 128)])
def test_rows_kernels_strides_and_masked_rows(Sq, Skv, d):
    """Views of packed buffers give the contiguous tensors' results bit for bit, and
    so do zeros in the place of padded keys whose scores and dP overflow; the padded
    keys' gradients are zeros, also where dO is nan."""
    import torch
    import paper_2607_21624_amd as fbl
    B, H = 16, 16
    W = H * d
    g = torch.Generator(device="cuda")
    g.manual_seed(Sq + d)
    qd = torch.randn(B, Sq, 2 * W, generator=g, device="cuda")
    kv = torch.randn(B, Skv, 2 * W, generator=g, device="cuda")
    lens = torch.randint(1, Skv + 1, (B,), generator=g, device="cuda", dtype=torch.int32)
    lens[0] = 0
    pad = torch.arange(Skv, device="cuda")[None, :] >= lens[:, None]
    note(f"rows, packed views Sq={Sq} Skv={Skv} d={d}")

    def run(q, k, v, do):
        out = torch.full_like(q, float("nan"))
        o, lse = fbl.attn_fwd(q, k, v, H, H, kv_len=lens, out=out)
        gr = [torch.full_like(t, float("nan")) for t in (q, k, v)]
        fbl.attn_bwd(q, k, v, o, do, lse, H, H, kv_len=lens, dq=gr[0], dk=gr[1], dv=gr[2])
        torch.cuda.synchronize()
        return [o, lse] + gr

    views = [qd[:, :, :W], kv[:, :, :W], kv[:, :, W:], qd[:, :, W:]]
    assert not any(t.is_contiguous() for t in views)
    want = run(*(t.contiguous() for t in views))
    for a, b in zip(run(*views), want):
        assert not a.isnan().any() and torch.equal(a, b)  # (LSE is -inf in the batch without keys)
    big, zero = kv.clone(), kv.clone()
    big[:, :, :W][pad], big[:, :, W:][pad], zero[pad] = 1e30, 3e38, 0.0
    want = run(views[0], zero[:, :, :W], zero[:, :, W:], views[3])
    for a, b in zip(run(views[0], big[:, :, :W], big[:, :, W:], views[3]), want):
        assert not a.isnan().any() and torch.equal(a, b)  # (LSE is -inf in the batch without keys)
    views[3] = views[3].clone()
    views[3][:, 7] = float("nan")
    for t in run(*views)[3:]:
        assert (t[pad] == 0).all()
