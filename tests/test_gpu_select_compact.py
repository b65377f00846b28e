"""Selection and gather in one launch against the separate calls, which the oracle tests hold: at the edges of what the one
launch takes (256, 1024 and 4096 chunks per head, workgroups) and beyond, ragged tails, whole chunks, nothing kept, everything
kept.  The caller's log-sum-exps make the scores the same bits on both ways."""
import pytest
import torch

import paper_2502_00299_amd as ckv

pytestmark = pytest.mark.gpu
DEV = "cuda:0"

# (prefix tokens per sequence, chunk, percent kept, kv-heads, layers that share the selection)
CASES = [
    ([255], 1, 30, 2, 1), ([256], 1, 100, 2, 3), ([257], 1, 50, 1, 2), ([1024 * 3 - 1], 3, 20, 2, 1), ([1024 * 3 + 1], 3, 20, 2, 1),
    ([4095 * 2 + 1], 2, 10, 2, 1), ([4097 * 2 - 1], 2, 10, 2, 2), ([4096], 1, 90, 4, 1),      # many workgroups of a wide head
    ([1030], 4, 50, 4, 25), ([1030], 4, 50, 4, 26),      # 1400 and 1456 workgroups of 258 chunks
    ([1024], 4, 50, 16, 18),      # 4032 of 256
    ([7, 500, 33], 33, 30, 2, 2), ([1000, 10, 2000], 10, 0, 1, 1), ([999], 500, 60, 1, 1), ([0, 640], 16, 25, 2, 1),
    ([3000], 10, 30, 32, 33),      # more layers than one launch carries
]


@pytest.mark.parametrize("whole", [False, True])
@pytest.mark.parametrize("prefix,c,pct,hkv,layers", CASES)
def test_equals_separate_calls(prefix, c, pct, hkv, layers, whole):
    gen = torch.Generator(device=DEV).manual_seed(sum(prefix) + c)
    g, w, d = 2, 9, 64
    lens = [p + w for p in prefix]
    B, total = len(lens), sum(lens) * hkv * d
    base = [sum(lens[:i]) * hkv * d for i in range(B)]
    prob = ckv.Problem(hkv * g, hkv, d, w, c, ckv.BF16, lens, [p * pct // 100 for p in prefix], base, d, hkv * d,
                       flags=ckv.FLAG_WHOLE_CHUNKS if whole else 0)
    k = [torch.randn(total, generator=gen, device=DEV).bfloat16() for _ in range(layers)]
    v = [torch.randn(total, generator=gen, device=DEV).bfloat16() for _ in range(layers)]
    q = torch.randn((B, hkv * g, w, d), generator=gen, device=DEV).bfloat16()
    lse = torch.rand((B, hkv * g, w), generator=gen, device=DEV) + 5

    def outputs(n):
        sel = [torch.full((1, B, hkv, prob.sel_cap), -7, dtype=torch.int32, device=DEV) for _ in range(2)]
        cnt = torch.full((1, B, hkv), -7, dtype=torch.int32, device=DEV)
        return sel, cnt, [torch.zeros(prob.out_elements(), dtype=torch.bfloat16, device=DEV) for _ in range(2 * n)]

    sel, cnt, want = outputs(layers)
    ws = torch.full((ckv.chunkkv_workspace_bytes(prob, layers, layers),), 0xFF, dtype=torch.uint8, device=DEV)
    scores = torch.full((B, hkv, prob.score_cap), float("nan"), device=DEV)
    ckv.chunkkv_score_lse(prob, q, k[0], lse, scores, None, ws)
    ckv.chunkkv_chunk_topk(prob, scores, sel[0], sel[1], cnt)
    for i in range(layers):
        ckv.chunkkv_compact(prob, k[i], v[i], sel[0], sel[1], cnt, want[i], want[layers + i])

    got_sel, got_cnt, got = outputs(layers)
    ckv.chunkkv_compress_stack_lse(prob, layers, [q] + [None] * (layers - 1), k, v, [lse] + [None] * (layers - 1), got[:layers], got[layers:],
                                   *got_sel, got_cnt, ws)
    layer_sel, layer_cnt, layer = outputs(1)
    ckv.chunkkv_compress_layer(prob, 0, layers, q, lse, k[0], v[0], layer[0], layer[1], *layer_sel, layer_cnt, ws)
    for s, n, out in ((got_sel, got_cnt, got), (layer_sel, layer_cnt, layer)):
        assert torch.equal(n, cnt)
        for x, y in zip(s, sel):
            live = torch.arange(prob.sel_cap, device=DEV) < cnt[..., None]
            assert torch.equal(torch.where(live, x, 0), torch.where(live, y, 0))
    for i in range(2 * layers):
        assert torch.equal(got[i], want[i])
    assert torch.equal(layer[0], want[0]) and torch.equal(layer[1], want[layers])
