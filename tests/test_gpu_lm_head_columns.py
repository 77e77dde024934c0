"""GPU parity at the edges of the lm_head pass and its merge: vocabularies that end inside a block,
long candidate lists, many hidden rows per sequence, and rows whose maxima tie everywhere."""
import numpy as np
import pytest
import torch

import test_gpu_accept as acc
from paper_2604_05650_amd import synth
from parity import t_bf16, t_f32, t_i32

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("B,K,n_br,bonus,V,d,topk", [
    (1, 1, 1, False, 40, 128, 16),        # fewer rows than a block, one hidden row
    (1, 5, 1, False, 193, 128, 1),        # one row beyond three blocks
    (1, 5, 1, True, 33000, 256, 16),      # several blocks per workgroup, k * k candidates
    (2, 16, 1, True, 20001, 128, 4),      # more hidden rows than waves of the merge
    (8, 8, 8, False, 8192, 256, 5),       # 64 hidden rows of one sequence
    (33, 1, 1, False, 33333, 256, 4),     # smallest of the wide pass, second half one column
    (7, 5, 1, False, 8192, 384, 4),       # 64-row blocks
    (12, 5, 1, True, 33000, 256, 4),      # two groups of 36 columns
    (17, 5, 1, False, 65, 128, 16),       # two groups of 45 and 40, one row beyond a block
    (8, 16, 1, False, 40001, 128, 2),     # 128 columns
    (8, 16, 1, False, 16384, 128, 4),     # ... in 64-row blocks, the most there are of them
    (26, 5, 1, False, 33000, 256, 4),     # three groups: a full pass and a narrower one
    (6, 10, 2, True, 20001, 256, 4),      # trees: two groups of four and two chains
    (14, 5, 1, False, 8192, 128, 4),      # two groups of 35, 64-row blocks
    (9, 16, 1, False, 5000, 128, 1),      # a last pass of 16 columns
])
def test_edges(B, K, n_br, bonus, V, d, topk):
    rows = K + (1 if bonus else 0)
    key = (611, B, K, V, topk)
    h = synth.normal_bf16(key + (0,), (B, rows, d), 1.0)
    w = synth.normal_bf16(key + (1,), (V, d), 0.1)
    h, planted = synth.plant_target_rows(h, w, 24.0, key + (2,))
    draft = synth.draft_ids_from_target(planted[:, :K], key + (3,), p_wrong=0.3, V=V)
    rel = np.random.default_rng(611).random((B, K)).astype(np.float32)
    acc._check(h, w, draft, rel, int(0.7 * K), K, topk=topk, bonus_row=bonus, n_branches=n_br,
               tag=f"edges V{V} d{d} rows{B * rows}")


@pytest.mark.parametrize("V,topk,step", [(38400, 4, 1), (38400, 16, 1), (152064, 16, 64 * 512)])
def test_equal_logits_take_the_lowest_ids(V, topk, step):
    # every `step`-th vocabulary row is the same vector and the others are zero: the best logit
    # occurs in all records (step 1: more of them than the short selection takes) or in a few,
    # and the k best are the k lowest ids among them, exactly
    from paper_2604_05650_amd import binding as L
    d = 128
    w = torch.zeros((V, d), dtype=torch.bfloat16, device="cuda:0")
    w[::step] = 0.5
    h = np.full((1, 3, d), 0x3F80, np.uint16)     # ones
    outs = L.loose_accept(t_bf16(h), w, t_i32([[0, 1, 2]]), t_f32([[0.0, 0.1, 0.2]]), 0, 0,
                          topk=topk, return_entropy=True)
    torch.cuda.synchronize()
    best = list(range(0, V, step))
    rest = [i for i in range(2 * topk) if i not in best]
    want = (best + rest)[:topk]
    assert outs["target_ids"].cpu().tolist() == [[0, 0, 0]]
    assert outs["topk_ids"].cpu().tolist() == [[want] * 3]
    # the softmax of `len(best)` logits 64 and V - len(best) zeros
    np.testing.assert_allclose(outs["topk_probs"][0, 0, 0].item(), 1.0 / len(best), rtol=1e-5)


@pytest.mark.parametrize("B,K,V,d,room", [
    (9, 5, 65500, 384, 1.0),      # one group over both halves, 128-row tasks, three chunks
    (13, 5, 65500, 1152, 1.0),    # two groups in a pass, 48 columns each at most
    (8, 16, 65500, 128, 1.0),     # 128 columns, one chunk
    (13, 5, 8192, 384, 1.0),      # 64-row tasks
    (13, 5, 65500, 384, 0.6),     # a workspace that holds one group only
    (26, 5, 65500, 384, 1.0),     # a full pass and a narrower one
])
def test_logits_do_not_depend_on_the_other_rows(B, K, V, d, room):
    # every kernel adds up a vocabulary row's products in the same order: the same bits
    import ctypes as C
    from paper_2604_05650_amd import binding as L
    h = t_bf16(synth.normal_bf16((613, B, K, d), (B, K, d), 1.0))
    w = t_bf16(synth.normal_bf16((614, V, d), (V, d), 0.1))
    draft = t_i32(np.zeros((B, K)))
    rel = t_f32(np.zeros((B, K)))
    outs = L.alloc_accept_outputs(B, K, V, 4, h.device, True)
    args = L.loose_accept_args(h, w, draft, rel, 0, K, topk=4, loose_topk_gate=0, outs=outs)
    full = L.raw().lvspec_loose_accept_workspace(C.byref(args))
    ws = torch.empty((int(full * room),), dtype=torch.uint8, device=h.device)
    args.workspace, args.workspace_bytes = ws.data_ptr(), ws.numel()
    assert L.raw().lvspec_loose_accept(C.byref(args), torch.cuda.current_stream().cuda_stream) == L.OK
    for b in (0, 1, B // 2, B - 1):
        one = L.loose_accept(h[b:b + 1], w, draft[b:b + 1], rel[b:b + 1], 0, K, topk=4,
                             return_logits=True)
        assert torch.equal(one["logits"][0], outs["logits"][b])
        assert torch.equal(one["topk_ids"][0], outs["topk_ids"][b])


@pytest.mark.parametrize("B,K,V,topk", [(1, 3, 33000, 4), (1, 3, 33000, 16), (7, 5, 33000, 4),
                                        (17, 5, 9000, 16)])
def test_nan_logits_keep_their_places(B, K, V, topk):
    # NaN ranks as its bits do: equal ones by id, and behind every number as the products leave it
    # (sign bit set).  A row of nothing but NaN has token 0, as argmax gives; the rows beside it
    # have the bits that they have without it.
    from paper_2604_05650_amd import binding as L
    d = 256
    h = t_bf16(synth.normal_bf16((615, B, K, 0), (B, K, d), 1.0))
    w = t_bf16(synth.normal_bf16((615, V, 1), (V, d), 0.1))
    draft, rel = t_i32(np.zeros((B, K))), t_f32(np.zeros((B, K)))

    def call(h, w):
        outs = L.loose_accept(h, w, draft, rel, 0, 0, topk=topk, return_entropy=True)
        torch.cuda.synchronize()
        return {k: v.cpu() for k, v in outs.items()}

    clean = call(h, w)
    bad = h.clone()
    bad[-1, 1] = float("nan")
    outs = call(bad, w)
    assert outs["topk_ids"][-1, 1].tolist() == list(range(topk))
    assert outs["target_ids"][-1, 1] == 0 and torch.isnan(outs["topk_probs"][-1, 1]).all()
    keep = torch.ones((B, K), dtype=torch.bool)
    keep[-1, 1] = False
    for name in ("target_ids", "topk_ids", "topk_probs", "entropy"):
        assert torch.equal(outs[name][keep], clean[name][keep]), name
    # three rows of lm_head that are not NaN: they come first, then the lowest ids
    left = [5, V // 2, V - 2]
    holes = torch.full_like(w, float("nan"))
    holes[left] = w[left]
    outs = call(h, holes)
    logits = (h.double() @ w[left].double().T).cpu()
    for b in (0, B - 1):
        for i in range(K):
            order = [left[j] for j in torch.argsort(logits[b, i], descending=True)]
            rest = [j for j in range(topk) if j not in left]
            assert outs["topk_ids"][b, i].tolist() == (order + rest)[:topk]


@pytest.mark.parametrize("S,n_br,K,bonus,V", [
    (3, 2, 8, False, 8192),      # 16 rows of a sequence: merge and rule in one kernel
    (3, 3, 6, False, 8192),      # 18: two kernels; 128 records per row
    (2, 2, 16, True, 8300),      # 34, chains of 17 rows; 130 records
    (1, 8, 8, False, 33000),     # the most rows and chains
    (5, 8, 2, True, 40),         # one record, rows that end inside a workgroup of the merge
])
def test_chains_of_a_tree_are_judged_as_chains(S, n_br, K, bonus, V):
    # the same hidden rows as trees and as single chains: the same bits, and the longest chain is kept
    from paper_2604_05650_amd import binding as L
    B, d, rows = S * n_br, 256, K + (1 if bonus else 0)
    key = (616, S, n_br, K, V)
    h = synth.normal_bf16(key + (0,), (B, rows, d), 1.0)
    w = synth.normal_bf16(key + (1,), (V, d), 0.1)
    h, planted = synth.plant_target_rows(h, w, 24.0, key + (2,))
    draft = t_i32(synth.draft_ids_from_target(planted[:, :K], key + (3,), p_wrong=0.3, V=V))
    rel = t_f32(np.random.default_rng(key).random((B, K)))
    h, w = t_bf16(h), t_bf16(w)
    seen = set()
    for kw in (dict(), dict(loose_topk_gate=3), dict(rule=L.RULE_ENTROPY_GATE, entropy_threshold=0.05),
               dict(rule=L.RULE_ENTROPY_WINDOW, entropy_threshold=0.01, defer_window=1)):
        tree, chains = (L.loose_accept(h, w, draft, rel, K // 2, K, topk=5, return_entropy=True,
                                       n_branches=n, bonus_row=bonus, **kw) for n in (n_br, 1))
        torch.cuda.synchronize()
        for name, v in chains.items():
            assert torch.equal(tree[name], v), (name, kw)
        taus = chains["accept_len"].view(S, n_br).cpu().numpy()
        assert tree["best_branch"].cpu().tolist() == taus.argmax(1).tolist()
        seen |= set(chains["verdict"].unique().tolist())
    assert seen >= {0, 1, 2}


@pytest.mark.parametrize("V,d,topk", [(5000, 4096, 4), (5000, 8192, 4), (152064, 128, 16), (152064, 128, 4)])
def test_logits_in_calls_of_few_and_of_many_rows(V, d, topk):
    # where the order of the sums is another one for up to 32 hidden rows (row pitches of 8 KiB, many
    # candidates): the same bits in every call of up to 32 rows, and in every call of more
    from paper_2604_05650_amd import binding as L
    B, K = 20, 4
    h = t_bf16(synth.normal_bf16((617, V, d, 0), (B, K, d), 1.0))
    w = t_bf16(synth.normal_bf16((617, V, d, 1), (V, d), 0.1))

    def logits(chains):
        n = len(chains)
        outs = L.loose_accept(h[chains].contiguous(), w, t_i32(np.zeros((n, K))), t_f32(np.zeros((n, K))),
                              0, 0, topk=topk, return_logits=True)
        return outs["logits"], outs["topk_ids"]

    few, few_ids = logits([0])                                   # 4 rows
    for chains in ([3, 0], [5, 1, 2, 6, 0], list(range(7, -1, -1))):     # 8, 20, 32
        z, ids = logits(chains)
        assert torch.equal(z[-1], few[0]) and torch.equal(ids[-1], few_ids[0])
    many, many_ids = logits(list(range(8, -1, -1)))              # 36: both halves of one group
    for chains in (list(range(15, -1, -1)), list(range(19, -1, -1))):    # 64; 80: two groups
        z, ids = logits(chains)
        assert torch.equal(z[-1], many[-1]) and torch.equal(ids[-1], many_ids[-1])
    # two orders of the same 32-bit sum
    scale = (h[0].float().abs() @ w.float().abs().T).max().item()
    assert (few[0] - many[-1]).abs().max().item() <= 2 * d * 2.0 ** -24 * scale
    if topk <= 4 and d < 4096:
        assert torch.equal(few[0], many[-1])


@pytest.mark.parametrize("rows,V,d,topk", [
    (1, 16, 128, 16), (5, 40, 128, 7), (5, 33000, 256, 16), (5, 70001, 128, 8), (32, 40001, 256, 12),
    (16, 20001, 4096, 7), (36, 16384, 128, 16), (100, 40001, 128, 9), (128, 66000, 128, 16),
])
@pytest.mark.parametrize("ramp", [0.0, 4.0])
def test_long_lists_are_those_of_the_logits(rows, V, d, topk, ramp):
    # k = 7 to 16, single tasks and several per workgroup, in every stage size and column count; with
    # the ramp later rows beat earlier ones, so that many enter every list to the last.  The lists
    # against the logits that the same call returns, exactly: value descending, id ascending.
    from paper_2604_05650_amd import binding as L
    gen = torch.Generator(device="cuda:0")
    gen.manual_seed(612 + rows + V)
    w = torch.randn((V, d), generator=gen, device="cuda:0")
    w += ramp * torch.arange(V, device="cuda:0")[:, None] / V
    h = torch.rand((rows, 1, d), generator=gen, device="cuda:0") * 0.2
    ids = torch.zeros((rows, 1), dtype=torch.int32, device="cuda:0")
    outs = L.loose_accept(h.bfloat16(), w.bfloat16(), ids, torch.zeros((rows, 1), device="cuda:0"), 0, 0,
                          topk=topk, return_logits=True)
    torch.cuda.synchronize()
    z = outs["logits"].view(rows, V).cpu().numpy()
    want = np.argsort(-z, axis=1, kind="stable")[:, :topk]
    np.testing.assert_array_equal(outs["topk_ids"].view(rows, topk).cpu().numpy(), want)
