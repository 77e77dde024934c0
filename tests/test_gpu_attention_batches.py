"""GPU parity of the attention of batches: the cut of the line over all sequences, and the cut into
equal splits per unit, by the lengths, by the hint and by the workspace."""
import numpy as np
import pytest
import torch

import oracle
from paper_2604_05650_amd import synth
from parity import assert_rows_close, bf16_out_to_f64, dev, t_bf16, t_i32

pytestmark = pytest.mark.gpu


class Batch:
    """Inputs of one batched call, and what the library plans for it."""

    def __init__(self, key, kv_len, Hq, Hkv, gamma, cap=None):
        from paper_2604_05650_amd import binding as L
        import ctypes as C
        self.L, self.kv_len, self.gamma = L, list(kv_len), gamma
        B, D = len(kv_len), 128
        self.units, self.Hkv = B * Hkv, Hkv
        cap = cap or max(kv_len) + gamma
        self.q = t_bf16(synth.normal_bf16((121, *key, 0), (B, gamma, Hq, D), 1.0))
        # the rows in use, at the start of a cache that may be much larger
        rows = max(kv_len) + gamma
        self.kv = [torch.zeros((B, Hkv, cap, D), dtype=torch.bfloat16, device=dev()) for _ in "kv"]
        for i, t in enumerate(self.kv):
            t[:, :, :rows] = t_bf16(synth.normal_bf16((121, *key, 1 + i), (B, Hkv, rows, D), 1.0))
        a = L.verify_attn_args(self.q, *self.kv, t_i32(kv_len), out=torch.empty_like(self.q))
        plan = L.describe_plan(attn=a)
        self.n_split, self.n_rc = plan["attn_splits"], plan["attn_row_chunks"]
        self.rpad = plan["attn_rows_padded"]
        record = self.n_rc * self.rpad * 131 * 4          # bytes, all row chunks
        self.split_bytes = self.units * self.n_split * record
        asked = L.raw().lvspec_verify_attn_workspace(C.byref(a))
        # more than equal splits need: the line has records, one per stretch and one per unit
        self.stretches = asked // record - self.units if asked > self.split_bytes else 0

    def run(self, lens="device", split=False, **kw):
        ws = torch.empty((self.split_bytes,), dtype=torch.uint8, device=dev()) if split else None
        kv_len = None if lens == "host" else t_i32(self.kv_len)
        host = None if lens == "device" else self.kv_len
        out = self.L.verify_attn(self.q, *self.kv, kv_len, kv_len_host=host, workspace=ws, **kw)
        torch.cuda.synchronize()
        return out

    def check(self, out, what):
        rows = max(self.kv_len) + self.gamma
        o, _, _ = oracle.verify_attn(synth.from_torch_bf16(self.q),
                                     *(synth.from_torch_bf16(t[:, :, :rows].contiguous())
                                       for t in self.kv), self.kv_len)
        assert_rows_close(bf16_out_to_f64(out), o, what)


# bf16 results of the same partial sums, merged in another order: a 32-bit rounding (1e-7) moves a
# value over a bf16 boundary (4e-3 apart) in about one of 1e4; another cut gives other bf16
# probabilities and moves about a third of them
def _other_bits(a, b):
    return (a != b).float().mean().item()


@pytest.mark.parametrize("Hq,Hkv,gamma,kv_len,cap", [
    (40, 8, 5, [256, 256], 16384),                # fewer tiles than splits
    (28, 4, 5, [1024] * 4, 16384),
    (64, 8, 5, [700, 40, 1900], 16384),           # 48-row variant, units no multiple of XCDs' eight
    (64, 8, 8, [0, 2000, 33], 16384),             # 64-row variant
    (48, 4, 16, [600, 40, 900], 16384),           # three row chunks
    (16, 1, 5, [900, 1500, 2], 40000),            # 85 splits
    (8, 2, 5, [3000, 100, 1, 31, 64, 500, 7], 40000),
    (8, 1, 4, [6100, 17], 70000),                 # 128 splits
    (16, 8, 4, [1200] * 16, 1300),                # equal lengths, two splits
    (40, 8, 5, [4100] * 4, 4200),                 # equal lengths, twelve tiles and more each
])
def test_short_or_equal_sequences_take_equal_splits(Hq, Hkv, gamma, kv_len, cap):
    b = Batch((Hq, cap, len(kv_len)), kv_len, Hq, Hkv, gamma, cap)
    assert b.stretches > 0
    line = b.run()
    assert _other_bits(line, b.run(split=True)) < 2e-3
    assert torch.equal(line, b.run(lens="host")) and torch.equal(line, b.run(lens="both"))
    b.check(line, "equal splits")
