"""GPU parity: lvspec_verify_attn against oracle O1, element by element."""
import numpy as np
import pytest
import torch

import oracle
from paper_2604_05650_amd import synth
from parity import (assert_rows_close, assert_scalars_close, bf16_out_to_f64, dev, t_bf16,
                    t_i32)

pytestmark = pytest.mark.gpu


def _run(q, k, v, kv_len, vis_begin=None, vis_end=None, draft_mask=None, scale=0.0, **kw):
    from paper_2604_05650_amd import binding as L
    tq, tk, tv = t_bf16(q), t_bf16(k), t_bf16(v)
    out, lse, vm = L.verify_attn(
        tq, tk, tv, t_i32(kv_len),
        vis_begin=None if vis_begin is None else t_i32(vis_begin),
        vis_end=None if vis_end is None else t_i32(vis_end),
        draft_mask=draft_mask, scale=scale, return_lse=True,
        return_vis_mass=vis_begin is not None, **kw)
    torch.cuda.synchronize()
    return (bf16_out_to_f64(out), lse.cpu().numpy().astype(np.float64),
            None if vm is None else vm.cpu().numpy().astype(np.float64))


def _check(q, k, v, kv_len, vis_begin=None, vis_end=None, draft_mask=None, scale=0.0, tag=""):
    print(f"[attn] {tag} q{q.shape} k{k.shape} kv_len{list(kv_len)}", flush=True)
    g_out, g_lse, g_vm = _run(q, k, v, kv_len, vis_begin, vis_end, draft_mask, scale)
    o_out, o_lse, o_vm = oracle.verify_attn(q, k, v, kv_len, vis_begin, vis_end,
                                            scale=None if scale == 0.0 else scale,
                                            draft_mask=draft_mask)
    e1 = assert_rows_close(g_out, o_out, f"attn out {tag}")
    e2 = assert_scalars_close(g_lse, o_lse, f"attn lse {tag}")
    e3 = 0.0
    if vis_begin is not None:
        e3 = assert_scalars_close(g_vm, o_vm, f"attn vis_mass {tag}")
    print(f"[attn] {tag} ok: out {e1:.2e} lse {e2:.2e} vis {e3:.2e}", flush=True)


def test_config1_tiny():
    cfg = synth.CONFIGS["c1"]
    a = synth.attn_inputs(cfg)
    _check(a["q"], a["k"], a["v"], a["kv_len"], a["vis_begin"], a["vis_end"], tag="c1")


@pytest.mark.parametrize("gamma", [1, 2, 3, 5, 8, 16])
@pytest.mark.parametrize("L", [0, 1, 31, 33, 100, 777])
def test_ragged_lengths_and_gammas(gamma, L):
    B, Hq, Hkv, D = 1, 4, 2, 128
    cap = L + gamma + 3
    q = synth.normal_bf16((101, gamma, L, 0), (B, gamma, Hq, D), 1.0)
    k = synth.normal_bf16((101, gamma, L, 1), (B, Hkv, cap, D), 1.0)
    v = synth.normal_bf16((101, gamma, L, 2), (B, Hkv, cap, D), 1.0)
    _check(q, k, v, [L], [L // 4], [L // 2 + 1], tag=f"g{gamma} L{L}")


@pytest.mark.parametrize("Hq,Hkv,gamma", [(8, 8, 4), (10, 2, 5), (16, 2, 8), (16, 1, 8),
                                          (64, 8, 8), (7, 7, 3), (24, 2, 16)])
def test_head_groupings_and_row_chunks(Hq, Hkv, gamma):
    # G*gamma = 4, 25, 64, 128 (two row chunks), 64, 3, 192 (three row chunks)
    B, D, L = 2, 128, 300
    kv_len = [L, L - 77]
    cap = L + gamma
    q = synth.normal_bf16((102, Hq, Hkv, 0), (B, gamma, Hq, D), 1.0)
    k = synth.normal_bf16((102, Hq, Hkv, 1), (B, Hkv, cap, D), 1.0)
    v = synth.normal_bf16((102, Hq, Hkv, 2), (B, Hkv, cap, D), 1.0)
    _check(q, k, v, kv_len, [10, 0], [200, 223], tag=f"Hq{Hq} Hkv{Hkv} g{gamma}")


@pytest.mark.parametrize("Hq,Hkv,gamma,L", [(40, 8, 8, 1000), (6, 2, 16, 333), (7, 1, 5, 64),
                                            (12, 2, 16, 130), (66, 2, 1, 31), (9, 1, 5, 0)])
def test_between_33_and_48_rows_per_kv_head(Hq, Hkv, gamma, L):
    # row counts (or row-chunk sizes) that take the 48-row variant of the split kernel
    B, D = 2, 128
    cap = L + gamma + 1
    q = synth.normal_bf16((107, Hq, gamma, L, 0), (B, gamma, Hq, D), 1.0)
    k = synth.normal_bf16((107, Hq, gamma, L, 1), (B, Hkv, cap, D), 1.0)
    v = synth.normal_bf16((107, Hq, gamma, L, 2), (B, Hkv, cap, D), 1.0)
    _check(q, k, v, [L, L // 2], [0, 3], [L // 2, L // 2], tag=f"48 rows Hq{Hq} Hkv{Hkv} g{gamma} L{L}")


@pytest.mark.parametrize("Hq,Hkv,L", [(2, 1, 9000), (8, 4, 8200), (4, 2, 16500)])
def test_many_splits_per_kv_head(Hq, Hkv, L):
    # few kv heads and a long cache: more than 32 / more than 64 key-range splits per head, which
    # take the wider variants of the combine kernel
    B, D, gamma = 1, 128, 2
    q = synth.normal_bf16((106, Hq, L, 0), (B, gamma, Hq, D), 1.0)
    k = synth.normal_bf16((106, Hq, L, 1), (B, Hkv, L + gamma, D), 1.0)
    v = synth.normal_bf16((106, Hq, L, 2), (B, Hkv, L + gamma, D), 1.0)
    _check(q, k, v, [L], [100], [L - 50], tag=f"splits Hq{Hq} Hkv{Hkv} L{L}")


@pytest.mark.parametrize("Hq,Hkv,gamma", [(8, 8, 3), (32, 8, 5), (64, 8, 5), (64, 8, 8), (48, 4, 16)])
def test_workgroups_with_one_or_two_tiles_beyond_whole_rounds(Hq, Hkv, gamma):
    # 16-, 32-, 48-, 64-row variants and two row chunks; lengths chosen so that the key-range
    # splits hold 4q + 1 or 4q + 2 tiles of 32 keys (q >= 3): those workgroups keep the surplus
    # tiles in their extra LDS slots, among them the ragged last tile of a sequence
    from paper_2604_05650_amd import binding as L
    B, D = 4, 128
    kv_len = [3340, 3372, 3500, 1700]
    cap = max(kv_len) + gamma
    q = synth.normal_bf16((108, Hq, gamma, 0), (B, gamma, Hq, D), 1.0)
    k = synth.normal_bf16((108, Hq, gamma, 1), (B, Hkv, cap, D), 1.0)
    v = synth.normal_bf16((108, Hq, gamma, 2), (B, Hkv, cap, D), 1.0)
    a = L.verify_attn_args(t_bf16(q), t_bf16(k), t_bf16(v), t_i32(kv_len),
                           out=torch.empty((B, gamma, Hq, D), dtype=torch.bfloat16, device=dev()))
    n_split = L.describe_plan(attn=a)["attn_splits"]
    hit = set()
    for n in kv_len:
        tiles = (n + gamma + 31) // 32
        for t in {tiles // n_split, tiles // n_split + (1 if tiles % n_split else 0)}:
            if t >= 12 and t % 4 in (1, 2):
                hit.add(t % 4)
    assert hit == {1, 2}, (n_split, hit)
    _check(q, k, v, kv_len, [16, 0, 100, 5], [3000, 3372, 100, 1700],
           tag=f"extra tiles Hq{Hq} Hkv{Hkv} g{gamma} splits{n_split}")


def test_batch_with_different_lengths_and_spans():
    B, gamma, Hq, Hkv, D = 4, 5, 8, 2, 128
    kv_len = [1000, 37, 0, 515]
    cap = 1000 + gamma
    q = synth.normal_bf16((103, 0), (B, gamma, Hq, D), 1.0)
    k = synth.normal_bf16((103, 1), (B, Hkv, cap, D), 1.0)
    v = synth.normal_bf16((103, 2), (B, Hkv, cap, D), 1.0)
    # spans: interior, empty, beyond everything, whole context incl. drafts
    _check(q, k, v, kv_len, [16, 5, 0, 0], [900, 5, 0, 600], tag="ragged batch")


@pytest.mark.parametrize("Hq,Hkv,gamma", [(7, 1, 2), (16, 4, 5), (16, 2, 5), (40, 8, 8), (6, 1, 20)])
@pytest.mark.parametrize("kv_len", [
    [3, 0],                                  # fewer tiles than workgroups
    [4095, 31, 0, 64, 1],                    # one long sequence: units over many workgroups
    [250 + 13 * b for b in range(33)],       # workgroups over several units each
    [65 * (b % 3) for b in range(64)],       # the largest batch one line takes
    [4 * (b % 5) for b in range(65)],        # one more
])
def test_batches_share_the_workgroups(Hq, Hkv, gamma, kv_len):
    # 16-, 32-, 48- and 64-row variants and two row chunks; then equal splits per unit by a workspace
    # that holds only their partials: another summation order, so the bf16 results differ by roundings
    from paper_2604_05650_amd import binding as L
    B, D = len(kv_len), 128
    cap = max(kv_len) + gamma + 2
    q = synth.normal_bf16((109, Hq, B, 0), (B, gamma, Hq, D), 1.0)
    k = synth.normal_bf16((109, Hq, B, 1), (B, Hkv, cap, D), 1.0)
    v = synth.normal_bf16((109, Hq, B, 2), (B, Hkv, cap, D), 1.0)
    vb, ve = [n // 5 for n in kv_len], [n // 2 + 1 for n in kv_len]
    _check(q, k, v, kv_len, vb, ve, tag=f"line Hq{Hq} Hkv{Hkv} g{gamma} B{B}")
    tq, tk, tv = t_bf16(q), t_bf16(k), t_bf16(v)
    a = L.verify_attn_args(tq, tk, tv, t_i32(kv_len), out=torch.empty_like(tq))
    plan = L.describe_plan(attn=a)
    rows = B * Hkv * plan["attn_row_chunks"] * plan["attn_splits"] * plan["attn_rows_padded"]
    split = torch.empty((rows * 131 * 4,), dtype=torch.uint8, device=dev())
    out = L.verify_attn(tq, tk, tv, t_i32(kv_len), workspace=split)
    o_out, _, _ = oracle.verify_attn(q, k, v, kv_len)
    assert_rows_close(bf16_out_to_f64(out), o_out, "equal splits")


def test_draft_tree_mask():
    B, gamma, Hq, Hkv, D, L = 1, 6, 8, 2, 128, 200
    q = synth.normal_bf16((104, 0), (B, gamma, Hq, D), 1.0)
    k = synth.normal_bf16((104, 1), (B, Hkv, L + gamma, D), 1.0)
    v = synth.normal_bf16((104, 2), (B, Hkv, L + gamma, D), 1.0)
    # two branches of three tokens sharing the prefix: rows 0-2 and rows 3-5
    tree = [0b000001, 0b000011, 0b000111, 0b001000, 0b011000, 0b111000]
    _check(q, k, v, [L], [0], [L], draft_mask=tree, tag="tree")


def test_large_scores_and_custom_scale():
    # peaked softmax: large scale makes single keys dominate; running-max updates get exercised
    B, gamma, Hq, Hkv, D, L = 1, 4, 4, 1, 128, 500
    q = synth.normal_bf16((105, 0), (B, gamma, Hq, D), 1.0)
    k = synth.normal_bf16((105, 1), (B, Hkv, L + gamma, D), 1.0)
    v = synth.normal_bf16((105, 2), (B, Hkv, L + gamma, D), 1.0)
    _check(q, k, v, [L], [100], [400], scale=1.0, tag="scale1")
    # keys sorted by increasing score for row 0 would force a max update in every tile; emulate
    # by scaling key magnitudes up along the sequence
    k32 = synth.bf16_bits_to_f32(k) * np.linspace(0.1, 3.0, L + gamma,
                                                  dtype=np.float32)[None, None, :, None]
    _check(q, synth.f32_to_bf16_bits(k32), v, [L], [100], [400], tag="growing keys")


def test_strided_layouts():
    # K/V stored [B, cap, Hkv, D] (token-major) and q/out with padded head stride
    from paper_2604_05650_amd import binding as L_
    B, gamma, Hq, Hkv, D, L = 2, 3, 8, 4, 128, 130
    cap = L + gamma
    q = synth.normal_bf16((106, 0), (B, gamma, Hq, D), 1.0)
    k = synth.normal_bf16((106, 1), (B, Hkv, cap, D), 1.0)
    v = synth.normal_bf16((106, 2), (B, Hkv, cap, D), 1.0)
    tk = t_bf16(k).permute(0, 2, 1, 3).contiguous().permute(0, 2, 1, 3)   # strides of [B,cap,Hkv,D]
    tv = t_bf16(v).permute(0, 2, 1, 3).contiguous().permute(0, 2, 1, 3)
    qpad = torch.zeros((B, gamma, Hq, 2 * D), dtype=torch.bfloat16, device=dev())
    qpad[..., :D] = t_bf16(q)
    tq = qpad[..., :D]
    out = L_.verify_attn(tq, tk, tv, t_i32([L, L - 9]))
    torch.cuda.synchronize()
    o_out, _, _ = oracle.verify_attn(q, k, v, [L, L - 9])
    assert_rows_close(bf16_out_to_f64(out), o_out, "strided")


@pytest.mark.parametrize("B", [3, 5, 6, 20])
def test_host_lengths_give_identical_results(B):
    # lengths known to the host travel in the launch arguments (up to 5 sequences in the lines
    # the kernel fetches first, up to 32 in a table when there is no device array); every way
    # of passing them must give bit-identical results
    from paper_2604_05650_amd import binding as L
    gamma, Hq, Hkv, D = 5, 8, 2, 128
    kv_len = [int(x) for x in np.random.default_rng((107, B)).integers(0, 401, B)]
    kv_len[0], kv_len[-1] = 400, 33
    cap = 400 + gamma
    q = synth.normal_bf16((107, B, 0), (B, gamma, Hq, D), 1.0)
    k = synth.normal_bf16((107, B, 1), (B, Hkv, cap, D), 1.0)
    v = synth.normal_bf16((107, B, 2), (B, Hkv, cap, D), 1.0)
    tq, tk, tv = t_bf16(q), t_bf16(k), t_bf16(v)
    a = L.verify_attn(tq, tk, tv, t_i32(kv_len))
    b_ = L.verify_attn(tq, tk, tv, t_i32(kv_len), kv_len_host=kv_len)
    c_ = L.verify_attn(tq, tk, tv, None, kv_len_host=kv_len)
    torch.cuda.synchronize()
    assert torch.equal(a, b_) and torch.equal(a, c_)
    o_out, _, _ = oracle.verify_attn(q, k, v, kv_len)
    assert_rows_close(bf16_out_to_f64(c_), o_out, "host lengths")


@pytest.mark.parametrize("B", [1, 7])
def test_device_length_beyond_the_cache_is_clamped(B):
    # A stale device-side length must not send a copy past the rows the caller declared.  The
    # buffer is allocated larger than the declared cap, so even the unclamped kernel would read
    # mapped memory; the clamped one must give exactly the result of kv_len = cap - gamma, and a
    # negative length the result of an empty cache.
    from paper_2604_05650_amd import binding as L
    gamma, Hq, Hkv, D, cap, alloc = 4, 8, 2, 128, 300, 600
    q = synth.normal_bf16((108, B, 0), (B, gamma, Hq, D), 1.0)
    k = synth.normal_bf16((108, B, 1), (B, Hkv, alloc, D), 1.0)
    v = synth.normal_bf16((108, B, 2), (B, Hkv, alloc, D), 1.0)
    tq, tk, tv = t_bf16(q), t_bf16(k)[:, :, :cap], t_bf16(v)[:, :, :cap]
    lim = cap - gamma
    good = [lim] * B
    stale = [lim + 150] * B
    stale[-1] = -5
    good[-1] = 0
    a = L.verify_attn(tq, tk, tv, t_i32(good))
    b_ = L.verify_attn(tq, tk, tv, t_i32(stale))
    torch.cuda.synchronize()
    assert torch.equal(a, b_)
    o_out, _, _ = oracle.verify_attn(q, k[:, :, :cap], v[:, :, :cap], good)
    assert_rows_close(bf16_out_to_f64(b_), o_out, "clamped length")


def test_repeatable_bitwise():
    cfg = synth.CONFIGS["c1"]
    a = synth.attn_inputs(cfg)
    r1 = _run(a["q"], a["k"], a["v"], a["kv_len"], a["vis_begin"], a["vis_end"])
    r2 = _run(a["q"], a["k"], a["v"], a["kv_len"], a["vis_begin"], a["vis_end"])
    for x, y in zip(r1, r2):
        np.testing.assert_array_equal(x, y)


def _full_size(name, n_rows_checked):
    """Full-size config in the launch configuration the benchmark times; inputs generated on the
    device, copied to the host for the oracle, which computes a seeded sample of output rows."""
    from paper_2604_05650_amd import binding as L
    cfg = synth.CONFIGS[name]
    a = synth.attn_inputs(cfg, device=dev())
    kv_len = t_i32(a["kv_len"])
    vb, ve = t_i32(a["vis_begin"]), t_i32(a["vis_end"])
    print(f"[attn] {name} launching", flush=True)
    out, lse, vm = L.verify_attn(a["q"], a["k"], a["v"], kv_len, vis_begin=vb, vis_end=ve,
                                 return_lse=True, return_vis_mass=True,
                                 max_kv_len=max(cfg.kv_len), kv_len_host=list(cfg.kv_len))
    torch.cuda.synchronize()
    rng = np.random.default_rng(7)
    rows = np.stack([rng.integers(0, cfg.B, n_rows_checked),
                     rng.integers(0, cfg.gamma, n_rows_checked),
                     rng.integers(0, cfg.Hq, n_rows_checked)], 1).astype(np.int32)
    rows[0] = (cfg.B - 1, cfg.gamma - 1, cfg.Hq - 1)
    rows[1] = (0, 0, 0)
    qh, kh, vh = (synth.from_torch_bf16(a[x]) for x in ("q", "k", "v"))
    print(f"[attn] {name} oracle on {n_rows_checked} rows", flush=True)
    o_out, o_lse, o_vm = oracle.verify_attn(qh, kh, vh, a["kv_len"], a["vis_begin"],
                                            a["vis_end"], rows=rows)
    g = bf16_out_to_f64(out)
    gl = lse.cpu().numpy()
    gv = vm.cpu().numpy()
    g_rows = np.stack([g[b, i, h] for b, i, h in rows])
    e1 = assert_rows_close(g_rows, o_out, f"{name} out")
    e2 = assert_scalars_close([gl[b, h, i] for b, i, h in rows], o_lse, f"{name} lse")
    e3 = assert_scalars_close([gv[b, h, i] for b, i, h in rows], o_vm, f"{name} vis_mass")
    # properties that hold for every row: finite, visual mass within [0,1]
    assert np.isfinite(g).all() and np.isfinite(gl).all()
    assert (gv >= -1e-6).all() and (gv <= 1 + 1e-3).all()
    print(f"[attn] {name} ok: out {e1:.2e} lse {e2:.2e} vis {e3:.2e}", flush=True)


def test_config2_qwen32b_layer_full_size():
    _full_size("c2", 200)


def test_config3_llava72b_layer_full_size():
    _full_size("c3", 320)


def test_config5_long_video_full_size():
    _full_size("c5", 48)
