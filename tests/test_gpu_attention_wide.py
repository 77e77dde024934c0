"""GPU parity of the attention of more than 64 query rows per kv head, which share one copy of the keys
where the caller says how long the sequences are."""
import ctypes as C

import numpy as np
import pytest
import torch

import oracle
from paper_2604_05650_amd import synth
from parity import assert_rows_close, assert_scalars_close, bf16_out_to_f64, dev, t_bf16, t_i32

pytestmark = pytest.mark.gpu


def _call(q, k, v, kv_len, hint, mask=None, vis=None, narrow=False, host=False):
    from paper_2604_05650_amd import binding as L
    lens = t_i32(kv_len)
    ws = None
    if narrow:      # the records of equal splits of up to 64 rows, and no more
        a = L.verify_attn_args(q, k, v, lens, out=torch.empty_like(q), max_kv_len=hint, draft_mask=mask)
        p = L.describe_plan(attn=a)
        n = q.shape[0] * k.shape[1] * p["attn_row_chunks"] * p["attn_splits"] * p["attn_rows_padded"] * 131 * 4
        assert n < L.raw().lvspec_verify_attn_workspace(C.byref(a))
        ws = torch.empty((n,), dtype=torch.uint8, device=dev())
    out, lse, vm = L.verify_attn(q, k, v, lens, max_kv_len=hint, draft_mask=mask, workspace=ws,
                                 kv_len_host=list(kv_len) if host else None,
                                 vis_begin=None if vis is None else t_i32([x[0] for x in vis]),
                                 vis_end=None if vis is None else t_i32([x[1] for x in vis]),
                                 return_lse=True, return_vis_mass=vis is not None)
    torch.cuda.synchronize()
    return out, lse, vm


def _other_bits(a, b):
    return (a != b).float().mean().item()


# rows of a kv head: 65 (a third group of one row), 80, 96 (three groups), 100, 128 (four), 130, 256
# (two chunks); lengths: whole rounds of 64 keys, one key more, an odd tile at the end, much shorter than
# the hint (workgroups without a tile), nothing but the draft rows
@pytest.mark.parametrize("B,Hq,Hkv,gamma,hint,kv_len,branches", [
    (1, 80, 16, 13, 8300, [8300], 1),
    (1, 128, 16, 10, 8192 - 10, [8192 - 10], 1),
    (1, 96, 16, 16, 8200, [8192 - 15], 1),
    (1, 80, 16, 20, 8200, [8170], 2),
    (1, 128, 16, 16, 8200, [777], 1),
    (1, 64, 8, 16, 16400, [16384], 1),            # one split fewer, within the static scratch
    (1, 40, 8, 26, 3200, [3111], 2),
    (1, 64, 8, 32, 3200, [3200], 2),
    (1, 80, 16, 20, 8200, [0], 2),
    (8, 40, 8, 20, 3100, [3100, 5, 0, 800, 1601, 2016, 64, 3000], 2),
    (8, 40, 8, 16, 3100, [3100] * 8, 1),          # equal lengths
    (8, 64, 8, 9, 3100, [40, 90, 100, 7, 0, 33, 250, 64], 1),     # short ones: equal splits by the lengths
    (6, 40, 8, 30, 3100, [3100, 2000, 999, 31, 1024, 2777], 3),
])
def test_wide_rows(B, Hq, Hkv, gamma, hint, kv_len, branches):
    from paper_2604_05650_amd import binding as L
    D, rows = 128, hint + gamma
    key = (131, B, Hq, gamma, kv_len[0])
    q, k, v = (synth.normal_bf16((*key, i), s, 1.0) for i, s in
               enumerate([(B, gamma, Hq, D), (B, Hkv, rows, D), (B, Hkv, rows, D)]))
    mask = synth.branch_mask(branches, gamma // branches) if branches > 1 else None
    vis = [(min(n, 17), n * 3 // 4) for n in kv_len]
    tq, tk, tv = t_bf16(q), t_bf16(k), t_bf16(v)
    print(f"[wide] {key} hint {hint}", flush=True)
    out, lse, vm = _call(tq, tk, tv, kv_len, hint, mask, vis)
    narrow = _call(tq, tk, tv, kv_len, hint, mask, vis, narrow=True)[0]
    if max(kv_len) > 1000:    # other cuts of the keys than single tiles: the wide path it is
        assert _other_bits(out, narrow) > 1e-2
    o_out, o_lse, o_vm = oracle.verify_attn(q, k, v, kv_len, draft_mask=mask, vis_begin=[x[0] for x in vis],
                                            vis_end=[x[1] for x in vis])
    assert_rows_close(bf16_out_to_f64(out), o_out, "wide out")
    assert_rows_close(bf16_out_to_f64(narrow), o_out, "narrow out")
    assert_scalars_close(lse.cpu().numpy().astype(np.float64), o_lse, "wide lse")
    assert_scalars_close(vm.cpu().numpy().astype(np.float64), o_vm, "wide vis mass")
    # the same bits again, with the lengths on the host, and from the static scratch
    assert torch.equal(out, _call(tq, tk, tv, kv_len, hint, mask, vis, host=True)[0])
    st = torch.empty_like(tq)
    lens = t_i32(kv_len)
    a = L.verify_attn_args(tq, tk, tv, lens, out=st, max_kv_len=hint, draft_mask=mask)
    rc = L.raw().lvspec_verify_attn_static(C.byref(a), torch.cuda.current_stream().cuda_stream)
    torch.cuda.synchronize()
    assert rc == L.OK and torch.equal(out, st)


def test_wide_rows_of_a_token_major_cache():
    # rows of all kv heads side by side, row strides of 4 KiB; queries and results head-major
    B, Hq, Hkv, gamma, D, n = 1, 80, 16, 20, 128, 8200
    q, k, v = (synth.normal_bf16((132, i), s, 1.0) for i, s in
               enumerate([(B, gamma, Hq, D), (B, Hkv, n + gamma, D), (B, Hkv, n + gamma, D)]))
    tq, tk, tv = t_bf16(q), t_bf16(k), t_bf16(v)
    major = [t.transpose(1, 2).contiguous().transpose(1, 2) for t in (tk, tv)]
    hq = tq.transpose(1, 2).contiguous().transpose(1, 2)
    out = _call(tq, tk, tv, [n], n)[0]
    assert torch.equal(out, _call(hq, *major, [n], n)[0].contiguous())


def test_stale_lengths_stay_within_the_declared_rows():
    # device lengths outside [0, cap - gamma] are clamped to its ends
    B, Hq, Hkv, gamma, D, cap = 1, 80, 16, 16, 128, 8300
    gen = torch.Generator(device=dev())
    gen.manual_seed(133)
    q, k, v = (torch.randn(s, generator=gen, device=dev()).bfloat16() for s in
               [(B, gamma, Hq, D), (B, Hkv, cap, D), (B, Hkv, cap, D)])
    most = cap - gamma
    for stale, means in ((most + 999, most), (-5, 0)):
        assert torch.equal(_call(q, k, v, [stale], most)[0], _call(q, k, v, [means], most)[0])


@pytest.mark.parametrize("Hq,Hkv,gamma,hint,kv_len", [
    (28, 4, 14, 12000, [300] * 15 + [12000]),     # one long sequence among short ones
    (40, 8, 20, 6200, [6200, 3000, 700, 90]),     # eight records of a head, two groups merge them
    (40, 8, 20, 6200, [1900, 200, 60, 0]),        # far below the hint: equal splits
    (40, 8, 20, 12400, [12400, 11000]),           # sixteen records
    (28, 4, 16, 16400, [16400, 100, 9000]),       # more than sixteen: eight groups
    (64, 8, 10, 3100, [3100, 2, 0, 155, 3000, 640, 31, 33]),
])
def test_wide_batches_of_uneven_lengths(Hq, Hkv, gamma, hint, kv_len):
    from paper_2604_05650_amd import binding as L
    B, D = len(kv_len), 128
    key = (135, B, Hq, gamma, kv_len[0])
    q, k, v = (synth.normal_bf16((*key, i), s, 1.0) for i, s in
               enumerate([(B, gamma, Hq, D), (B, Hkv, hint + gamma, D), (B, Hkv, hint + gamma, D)]))
    tq, tk, tv = t_bf16(q), t_bf16(k), t_bf16(v)
    a = L.verify_attn_args(tq, tk, tv, t_i32(kv_len), out=torch.empty_like(tq), max_kv_len=hint)
    a.workspace_bytes = 1 << 40
    assert L.describe_plan(attn=a)["attn_rows_padded"] > 64
    vis = [(min(n, 17), n * 3 // 4) for n in kv_len]
    out, lse, vm = _call(tq, tk, tv, kv_len, hint, vis=vis)
    o_out, o_lse, o_vm = oracle.verify_attn(q, k, v, kv_len, vis_begin=[x[0] for x in vis],
                                            vis_end=[x[1] for x in vis])
    assert_rows_close(bf16_out_to_f64(out), o_out, "wide out")
    assert_scalars_close(lse.cpu().numpy().astype(np.float64), o_lse, "wide lse")
    assert_scalars_close(vm.cpu().numpy().astype(np.float64), o_vm, "wide vis mass")
    assert torch.equal(out, _call(tq, tk, tv, kv_len, hint, vis=vis, host=True)[0])


@pytest.mark.parametrize("B,Hq,Hkv,gamma,hint,kv_len", [
    (1, 80, 16, 20, 8300, [8170]),        # 100 rows; ends inside a tile, and an odd tile without a partner
    (1, 128, 16, 16, 8200, [777]),        # workgroups without a tile
    (1, 80, 16, 20, 8200, [0]),
    (8, 40, 8, 20, 3100, [3100, 5, 0, 800, 1601, 2016, 64, 3000]),
    (1, 40, 8, 5, 8200, [8170]),          # the cores of up to 64 rows: 32, 48 and 64
    (1, 64, 8, 5, 8200, [777]),
    (3, 64, 8, 8, 3100, [2900, 0, 95]),
])
def test_rows_behind_the_declared_ones_are_not_read(B, Hq, Hkv, gamma, hint, kv_len):
    # NaN from the last draft row on, in every kv head and behind the cache's rows: a masked key's row that is
    # read all the same gives 0 * NaN
    D, cap = 128, hint + gamma
    gen = torch.Generator(device=dev())
    gen.manual_seed(136)
    q = torch.randn((B, gamma, Hq, D), generator=gen, device=dev()).bfloat16()
    kv = [torch.randn((B, Hkv, cap + 64, D), generator=gen, device=dev()).bfloat16() for _ in "kv"]
    clean = _call(q, *(t[:, :, :cap] for t in kv), kv_len, hint)
    for t in kv:
        for b, n in enumerate(kv_len):
            t[b, :, n + gamma:] = float("nan")
    for got, want in zip(_call(q, *(t[:, :, :cap] for t in kv), kv_len, hint)[:2], clean[:2]):
        assert torch.equal(got, want)
