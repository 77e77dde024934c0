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

    def segments(self):
        """Tiles of every workgroup's parts of units, as the line cuts them."""
        pad = 5 if self.rpad <= 32 else 10
        tiles = [(n + self.gamma + 31) // 32 for n in self.kv_len for _ in range(self.Hkv)]
        total = sum(t + pad for t in tiles)
        n_pos = max(1, min(self.stretches, total // 4))
        cuts = [total * p // n_pos for p in range(n_pos + 1)]
        ends = np.cumsum([t + pad for t in tiles])
        parts = []
        for lo, hi in zip(cuts, cuts[1:]):
            for u in range(int(np.searchsorted(ends, lo, "right")), len(tiles)):
                at = int(ends[u]) - tiles[u] - pad
                if at >= hi:
                    break
                parts.append(min(hi - at, tiles[u]) - max(lo - at, 0))
        return [t for t in parts if t > 0]


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


@pytest.mark.parametrize("Hq,Hkv,gamma,n", [(8, 8, 3, 4100), (32, 8, 5, 4100), (64, 8, 5, 3600),
                                            (64, 8, 8, 3600), (48, 4, 16, 3600)])
def test_surplus_tiles_on_the_line_and_in_equal_splits(Hq, Hkv, gamma, n):
    # 16-, 32-, 48-, 64-row variants and two row chunks: parts of 4q + 1 and 4q + 2 tiles (q >= 3)
    # keep the surplus in extra LDS slots, whichever kernel has them
    b = Batch((Hq, gamma), [n, 3372, 3500, 1700], Hq, Hkv, gamma)
    assert b.stretches > 0
    parts = b.segments()
    assert sum(parts) == sum((x + gamma + 31) // 32 for x in b.kv_len) * Hkv
    assert {t % 4 for t in parts if t >= 12} >= {1, 2}, parts
    b.check(b.run(), "line")
    tiles = [(x + gamma + 31) // 32 for x in b.kv_len]
    each = {t // b.n_split + more for t in tiles for more in ((0, 1) if t % b.n_split else (0,))}
    assert {t % 4 for t in each if t >= 12} >= {1, 2}, each
    b.check(b.run(split=True), "equal splits")


@pytest.mark.parametrize("B,Hq,Hkv,gamma,n", [(3, 8, 8, 5, 4000), (5, 24, 8, 5, 2400), (6, 40, 4, 4, 4000),
                                              (20, 16, 2, 8, 2400), (32, 8, 2, 5, 1700)])
def test_the_line_is_the_same_however_the_lengths_arrive(B, Hq, Hkv, gamma, n):
    # in the launch arguments (up to five sequences), in a table (without a device array) and on the
    # device: the same stretches
    kv_len = [int(x) for x in np.random.default_rng((122, B)).integers(1, n, B)]
    kv_len[B // 2] = n
    b = Batch((B, n), kv_len, Hq, Hkv, gamma)
    assert b.stretches > 0
    out = b.run()
    # the line it is, not the equal splits
    assert _other_bits(out, b.run(split=True)) > 1e-2
    assert torch.equal(out, b.run(lens="host")) and torch.equal(out, b.run(lens="both"))
    b.check(out, "line")


@pytest.mark.parametrize("Hq,Hkv,gamma", [(8, 8, 5), (40, 8, 8)])
def test_equal_splits_do_not_look_at_the_other_sequences(Hq, Hkv, gamma):
    # the stretches of the line follow from all lengths; with a workspace for equal splits, or one
    # sequence, a sequence's bits follow from the shapes and its own length
    lens = [4000, 1300, 2500]
    a = Batch((Hq, 1), lens, Hq, Hkv, gamma)
    out = a.run(split=True)
    a.kv_len = [4000, 17, 3100]
    other = a.run(split=True)
    assert torch.equal(out[0], other[0]) and not torch.equal(out[1], other[1])
    assert_rows_close(bf16_out_to_f64(a.run()[0]), bf16_out_to_f64(other[0]), "line, same sequence")


@pytest.mark.parametrize("Hq,Hkv,gamma,kv_len,cap", [
    (28, 4, 10, [1500] * 4, 20000),               # two row chunks of 35 rows, eight splits
    (8, 2, 32, [2100, 2099, 2098, 2097], 20000),  # two of 64, as many tiles each
    (64, 8, 9, [900, 900], 16384),                # two, eight kv heads
    (40, 8, 32, [1000] * 3, 16384),               # three, and nine workgroups to a head
    (16, 4, 20, [0, 0], 16384),                   # one tile, most splits empty
    (28, 4, 10, [3000, 900, 40, 1], 60000),       # short ones of unequal lengths
])
def test_row_chunks_of_equal_splits(Hq, Hkv, gamma, kv_len, cap):
    # all row chunks of a kv head on one XCD, whichever kernel divides the keys: the same records
    b = Batch((Hq, gamma, len(kv_len)), kv_len, Hq, Hkv, gamma, cap)
    assert b.stretches > 0 and b.n_rc > 1 and b.units % 8 == 0
    out = b.run()
    assert _other_bits(out, b.run(split=True)) < 2e-3
    b.check(out, "row chunks")
