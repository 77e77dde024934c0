"""GPU parity of the merge of split partials, at the edges of its launch shapes."""
import numpy as np
import pytest
import torch

import oracle
from paper_2604_05650_amd import synth
from parity import assert_rows_close, assert_scalars_close, bf16_out_to_f64, t_bf16, t_i32

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("splits", [1, 2, 7, 8, 9, 31, 32, 33])
@pytest.mark.parametrize("short", [False, True])
def test_split_counts(splits, short):
    # up to 32 splits eight groups take every eighth one, beyond that four take every fourth; a sequence
    # much shorter than the hint leaves splits without a tile
    from paper_2604_05650_amd import binding as L
    Hq, Hkv, gamma, D = 20, 4, 5, 128
    hint = splits * 4 * 32 - gamma
    n = 40 if short else hint
    q, k, v = (synth.normal_bf16((134, splits, i), s, 1.0) for i, s in
               enumerate([(1, gamma, Hq, D), (1, Hkv, hint + gamma, D), (1, Hkv, hint + gamma, D)]))
    tq, tk, tv = t_bf16(q), t_bf16(k), t_bf16(v)
    lens = t_i32([n])
    a = L.verify_attn_args(tq, tk, tv, lens, out=torch.empty_like(tq), max_kv_len=hint)
    assert L.describe_plan(attn=a)["attn_splits"] == splits
    out, lse, vm = L.verify_attn(tq, tk, tv, lens, max_kv_len=hint, vis_begin=t_i32([3]), vis_end=t_i32([n // 2]),
                                 return_lse=True, return_vis_mass=True)
    torch.cuda.synchronize()
    o_out, o_lse, o_vm = oracle.verify_attn(q, k, v, [n], vis_begin=[3], vis_end=[n // 2])
    assert_rows_close(bf16_out_to_f64(out), o_out, "out")
    assert_scalars_close(lse.cpu().numpy().astype(np.float64), o_lse, "lse")
    assert_scalars_close(vm.cpu().numpy().astype(np.float64), o_vm, "vis mass")
