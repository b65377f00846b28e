"""Decode attention over fp32 caches where its launches differ: one range per head (no merge), 16, 8 and 4 wavefronts per
workgroup, one, two and four heads, at the edges of a step, against float64."""
import math

import pytest
import torch

import paper_2502_00299_amd as ckv

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


def reference(q, k, v):
    """[Hq][d] output and [Hq] log-sum-exp in float64 of one sequence: q [Hq][d], k and v [Hkv][n][d]."""
    g = q.shape[0] // k.shape[0]
    s = torch.einsum("hgd,hnd->hgn", q.double().view(k.shape[0], g, -1), k.double()) / math.sqrt(q.shape[1])
    out = torch.softmax(s, 2) @ v.double()
    return out.reshape(q.shape), torch.logsumexp(s, 2).reshape(-1)


def workgroups(lens, hkv, g):
    """Workgroups that have rows: ranges of one length, about 1024 of them, 256 rows or more."""
    batches = -(-g // 4) if g > 2 else 1
    rows = -(-(sum(lens) * hkv * batches) // 1024)
    rows = 256 if rows < 256 else -(-rows // 128) * 128
    return sum(-(-n // rows) for n in lens) * hkv * batches


# rows of the sequences, kv-heads, heads per kv-head, workgroups
@pytest.mark.parametrize("d", [64, 128])
@pytest.mark.parametrize("lens,hkv,g,wgs", [
    ([1], 1, 1, 1), ([31], 2, 2, 2), ([129, 256, 64], 2, 4, 6), ([255], 8, 3, 8),                   # one range per head
    # up to a workgroup per CU: 16 wavefronts (d = 128 and three heads or more: 8)
    ([257], 2, 1, 4), ([513, 1, 256], 2, 4, 10), ([3000], 8, 2, 96), ([2049, 700], 4, 5, 96), ([8192], 8, 1, 256),
    ([8000] + [300] * 7, 4, 2, 184), ([8000] + [300] * 7, 4, 4, 184), ([300, 1, 700] * 6, 2, 2, 72),
    # up to two: 8 at d = 128, 4 at d = 64
    ([8193], 8, 1, 264), ([12000], 8, 2, 376), ([9000, 3001], 8, 4, 384), ([16384], 8, 1, 512),
    # more: 4
    ([16385], 8, 1, 520), ([20000], 8, 1, 632), ([20000, 13], 8, 4, 640),
])
def test_matches_float64(d, lens, hkv, g, wgs):
    assert workgroups(lens, hkv, g) == wgs
    gen = torch.Generator().manual_seed(sum(lens) + g)
    B, hq, total = len(lens), hkv * g, sum(lens)
    k, v = (torch.randn((total, hkv, d), generator=gen) for _ in range(2))
    q = torch.randn((B, hq, d), generator=gen) * 2
    starts = [sum(lens[:b]) for b in range(B)]
    prob = ckv.Problem(hq, hkv, d, 1, 1, ckv.F32, lens, [0] * B, [s * hkv * d for s in starts], d, hkv * d)
    ws = torch.full((max(256, ckv.chunkkv_decode_workspace_bytes(prob, False)),), 0xFF, dtype=torch.uint8, device=DEV)
    out, lse = torch.full((B, hq, d), float("nan"), device=DEV), torch.full((B, hq), float("nan"), device=DEV)
    short = torch.tensor([[max(0, n - 40 * h) for h in range(hkv)] for n in lens], dtype=torch.int32)   # rows of every head
    for kv_len in (None, short):
        ckv.chunkkv_decode_attention(prob, False, None if kv_len is None else kv_len.to(DEV), q.to(DEV), k.to(DEV), v.to(DEV), out, lse, ws)
        got, got_lse = out.cpu().double(), lse.cpu().double()
        for b, n in enumerate(lens):
            for h in range(hkv):
                m = n if kv_len is None else int(kv_len[b, h])
                rows, heads = slice(starts[b], starts[b] + m), slice(h * g, (h + 1) * g)
                if m == 0:
                    assert (got[b, heads] == 0).all() and (got_lse[b, heads] == float("-inf")).all()
                    continue
                want, want_lse = reference(q[b, heads], k[rows, h][None], v[rows, h][None])
                # a logit is a sum of 128 products with 24 bits, the largest about 10: 1e-6 of a weight
                assert float(((got[b, heads] - want).abs().amax(1) / want.abs().amax(1)).max()) < 1e-5
                assert float((got_lse[b, heads] - want_lse).abs().max()) < 1e-5
