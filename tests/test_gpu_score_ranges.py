"""Single-pass scoring where its kernel can go wrong: the ragged last period, a range that holds window keys alone, the
largest window, workgroups that share the rows of a range and ones that hold 256 of them, wavefronts without rows, and every
compiled chunk size; scores against plain float64."""
import math

import pytest
import torch

import paper_2502_00299_amd as ckv

pytestmark = pytest.mark.gpu
DEV = "cuda:0"
KIND = {ckv.BF16: torch.bfloat16, ckv.F16: torch.float16}


def oracle_scores(q, k, w, c):
    """[Hkv][C] chunk scores of one sequence in float64: q [Hq][w][d], k [Hkv][L][d]."""
    g, (hkv, L, d) = q.shape[0] // k.shape[0], k.shape
    P = L - w
    seen = torch.arange(L)[None, :] <= P + torch.arange(w)[:, None]
    out = torch.zeros(hkv, (P + c - 1) // c, dtype=torch.float64)
    for h in range(hkv):
        s = (q[h * g:(h + 1) * g].double() @ k[h].double().T) / math.sqrt(d)
        p = torch.softmax(s.masked_fill(~seen, float("-inf")), dim=2)[:, :, :P].sum((0, 1))
        out[h].index_add_(0, torch.arange(P) // c, p)
    return out


# (prefix tokens, window, query heads per kv-head, chunk size): periods are 160 keys, ranges four of them or more
CASES = [
    (1, 64, 4, 20), (100, 64, 4, 10),        # 256 rows: a ragged first period
    (1, 32, 4, 5), (159, 32, 4, 10), (160, 32, 4, 20), (161, 64, 4, 5),
    (640, 96, 2, 10),        # four whole periods, then a range that holds window keys alone
    (639, 32, 7, 5), (641, 32, 7, 10), (2000, 32, 7, 20),   # 224 rows: the last wavefront of the second row group has none
    (1281, 64, 4, 5), (1439, 64, 4, 10), (1440, 64, 4, 20),
    (1290, 256, 1, 10),      # the largest window one head can have
    (3333, 17, 4, 5), (3333, 16, 5, 10), (3333, 25, 3, 20),
    (9001, 64, 4, 5),        # more than one round of ranges
]


@pytest.mark.parametrize("dtype", [ckv.BF16, ckv.F16])
@pytest.mark.parametrize("P,w,g,c", CASES)
def test_scores_match_float64(dtype, P, w, g, c):
    gen = torch.Generator().manual_seed(P * 7 + w)
    hkv, d, L = 2, 128, P + w
    q = torch.randn((hkv * g, w, d), generator=gen).to(KIND[dtype])
    k = torch.randn((hkv, L, d), generator=gen).to(KIND[dtype])
    want = oracle_scores(q, k, w, c)
    prob = ckv.Problem(hkv * g, hkv, d, w, c, dtype, [L], [0], [0], L * d, d)
    ws = torch.full((ckv.chunkkv_workspace_bytes(prob),), 0xFF, dtype=torch.uint8, device=DEV)   # NaNs: nothing may be read unwritten
    scores = torch.full((hkv, prob.score_cap), float("nan"), device=DEV)
    ckv.chunkkv_score(prob, q.to(DEV), k.to(DEV), scores, None, ws)
    got = scores.cpu().double()[:, :want.shape[1]]
    # sums are stored with 12 mantissa bits, 2^-13 each, which up to 256 rows average out; fp32 around that is 1e-6
    assert float(((got - want).abs() / want).max()) < 1.3e-4
    # the same head over and over, until the launch is too large for workgroups to share rows: the same scores
    ranges = -(-(-(-L // 160)) // 4)      # of four periods: no case is long enough for longer ones
    n = 128 // (ranges * hkv) + 1 if g * w > 128 else 5
    assert ranges <= 32 and (g * w <= 128 or ranges * hkv <= 128 < ranges * hkv * n)
    many = ckv.Problem(n * hkv * g, n * hkv, d, w, c, dtype, [L], [0], [0], L * d, d)
    ws = torch.full((ckv.chunkkv_workspace_bytes(many),), 0xFF, dtype=torch.uint8, device=DEV)
    more = torch.full((n * hkv, many.score_cap), float("nan"), device=DEV)
    ckv.chunkkv_score(many, q.to(DEV).repeat(n, 1, 1), k.to(DEV).repeat(n, 1, 1), more, None, ws)
    assert torch.equal(more[:, :want.shape[1]], scores[:, :want.shape[1]].repeat(n, 1))


# The grids count the ranges of all sequences: ragged batches, sequences without a prefix first, last and in between, 16 and 17
# of them (two launches), with shared rows and without, against every sequence alone, to the bit.
@pytest.mark.parametrize("prefixes,w,g,c,hkv", [
    ([0, 700, 0, 0, 5121, 20, 0], 64, 4, 5, 2), ([20400] + [300] * 11, 64, 4, 20, 2), ([641, 1, 160, 2000], 32, 4, 10, 3),
    ([100 * i for i in range(16)], 32, 7, 10, 2), ([161 * (i * 5 % 17) for i in range(17)], 64, 4, 20, 1), ([0, 0], 64, 4, 10, 2),
])
def test_ragged_batch_equals_sequences_alone(prefixes, w, g, c, hkv):
    gen = torch.Generator(device=DEV).manual_seed(len(prefixes))
    d, lens = 128, [p + w for p in prefixes]
    k = torch.randn((max(lens), hkv, d), generator=gen, device=DEV).bfloat16()      # every sequence is a prefix of the same cache
    q = torch.randn((len(lens), hkv * g, w, d), generator=gen, device=DEV).bfloat16()

    def score(lens, q):
        prob = ckv.Problem(hkv * g, hkv, d, w, c, ckv.BF16, lens, [0] * len(lens), [0] * len(lens), d, hkv * d)
        ws = torch.full((ckv.chunkkv_workspace_bytes(prob),), 0xFF, dtype=torch.uint8, device=DEV)
        scores = torch.full((len(lens), hkv, max(1, prob.score_cap)), -1.0, device=DEV)
        ckv.chunkkv_score(prob, q, k, scores, None, ws)
        return scores

    got = score(lens, q)
    for b, p in enumerate(prefixes):
        n = (p + c - 1) // c
        assert torch.equal(got[b, :, :n], score(lens[b:b + 1], q[b:b + 1].contiguous())[0, :, :n]), b
        assert (got[b, :, n:] == -1.0).all()


# The row totals keep the bits of their ranges' sums: all prefix logits are X and scale * log2(e) is one, so the sums are whole
# numbers, every score is 65 c / P, and the only rounding is that of X + log2(P) at 2^13.. (its last bit is 2^-10).  A rounding
# per range on top of it takes all of these prefixes past the bound.
@pytest.mark.parametrize("dtype", [ckv.BF16, ckv.F16])
@pytest.mark.parametrize("P", [2561, 6400, 19200, 25600, 25000])
def test_row_totals_are_rounded_once(P, dtype):
    hkv, d, w, c, X = 2, 128, 65, 5, 8448.0
    q, k = torch.zeros((hkv, w, d), dtype=KIND[dtype], device=DEV), torch.zeros((hkv, P + w, d), dtype=KIND[dtype], device=DEV)
    q[..., 3], k[:, :P, 3] = 1.0, X
    prob = ckv.Problem(hkv, hkv, d, w, c, dtype, [P + w], [0], [0], (P + w) * d, d, softmax_scale=0.6931472)
    ws = torch.full((ckv.chunkkv_workspace_bytes(prob),), 0xFF, dtype=torch.uint8, device=DEV)
    scores = torch.full((hkv, prob.score_cap), float("nan"), device=DEV)
    ckv.chunkkv_score(prob, q, k, scores, None, ws)
    got = scores[:, :P // c].cpu().double()
    # half of the last bit, as a weight; the sum of 65 weights and the hardware's log2 and exp2 are 1e-5 of that at most
    assert float((got / (w * c / P) - 1).abs().max()) < (2.0 ** 2.0 ** -11 - 1) * 1.03


# Two passes, where pass 1 merges the row statistics of the ranges itself: one range, a whole number of loads of eight ranges
# and one more, 63 and 64 ranges (the most), a batch whose sequences have different numbers of them, and the last and first sizes
# on either side of the line from which a kernel merges them.
TWO_PASS = [
    (ckv.F32, 64, [40], 2, 2, 16, 3), (ckv.F32, 64, [8 * 64, 33], 2, 2, 16, 1), (ckv.BF16, 128, [9 * 64, 640, 65], 2, 4, 16, 8),
    (ckv.F16, 64, [64 * 128 + 1, 500], 1, 4, 32, 16), (ckv.F32, 128, [16000], 4, 1, 16, 33), (ckv.F32, 128, [16384], 4, 1, 16, 33),
    (ckv.BF16, 128, [20011], 1, 8, 32, 300),
    (ckv.F16, 64, [33 + 97 * (i * 7 % 17) for i in range(17)], 2, 4, 32, 7),     # two launches of up to 16 sequences
    (ckv.BF16, 128, [131072], 8, 1, 16, 10), (ckv.BF16, 128, [131073], 8, 1, 16, 10),
]


@pytest.mark.parametrize("dtype,d,lens,hkv,g,w,c", TWO_PASS)
def test_two_pass_scores_match_float64(dtype, d, lens, hkv, g, w, c):
    kind = {ckv.F32: torch.float32, **KIND}[dtype]
    gen = torch.Generator().manual_seed(sum(lens))
    q = torch.randn((len(lens), hkv * g, w, d), generator=gen).to(kind)
    k = torch.randn((sum(lens), hkv, d), generator=gen).to(kind)      # packed
    base = [sum(lens[:i]) * hkv * d for i in range(len(lens))]
    prob = ckv.Problem(hkv * g, hkv, d, w, c, dtype, lens, [0] * len(lens), base, d, hkv * d, flags=ckv.FLAG_TWO_PASS)
    ws = torch.full((ckv.chunkkv_workspace_bytes(prob),), 0xFF, dtype=torch.uint8, device=DEV)
    scores = torch.full((len(lens), hkv, prob.score_cap), float("nan"), device=DEV)
    ckv.chunkkv_score(prob, q.to(DEV), k.to(DEV), scores, None, ws)
    for b, n in enumerate(lens):
        at = sum(lens[:b])
        want = oracle_scores(q[b], k[at:at + n].transpose(0, 1).contiguous(), w, c)
        got = scores[b].cpu().double()[:, :want.shape[1]]
        # the reference of a row is one float below 32 (2^-20 in the exponent of every weight), the sums are fp32
        assert float(((got - want).abs() / want).max()) < 4e-6


# An infinity in a window key that some rows do not see: minus infinity as the logit of those that do (weight 0), nothing
# for the others, though their products with it are plus infinity.
@pytest.mark.parametrize("flags", [0, ckv.FLAG_TWO_PASS])
@pytest.mark.parametrize("dtype", [ckv.BF16, ckv.F16])
@pytest.mark.parametrize("P,w,g,c", [(1, 32, 4, 5), (159, 32, 4, 10), (641, 32, 7, 10), (1281, 64, 4, 20), (1290, 256, 1, 10)])
def test_infinite_key_that_rows_do_not_see(P, w, g, c, dtype, flags):
    gen = torch.Generator().manual_seed(P)
    hkv, d, L, at = 2, 128, P + w, w // 2
    q = torch.randn((hkv * g, w, d), generator=gen)
    k = torch.randn((hkv, L, d), generator=gen)
    q[:, :at, 3], q[:, at:, 3] = 0.5, -0.5
    k[:, P + at, 3] = float("inf")
    q, k = q.to(KIND[dtype]), k.to(KIND[dtype])
    want = oracle_scores(q, k, w, c)
    assert torch.isfinite(want).all()
    prob = ckv.Problem(hkv * g, hkv, d, w, c, dtype, [L], [0], [0], L * d, d, flags=flags)
    ws = torch.full((ckv.chunkkv_workspace_bytes(prob),), 0xFF, dtype=torch.uint8, device=DEV)
    scores = torch.full((hkv, prob.score_cap), float("nan"), device=DEV)
    ckv.chunkkv_score(prob, q.to(DEV), k.to(DEV), scores, None, ws)
    got = scores.cpu().double()[:, :want.shape[1]]
    assert float(((got - want).abs() / want).max()) < 1.3e-4   # as above; a NaN fails as well


# Launches on either side of the line from which the ranges of a head are neighbours (16384 key tiles, of 128 keys here): a ragged batch
# with sequences without a prefix, against every sequence alone.  Both are within 1e-6 of float64.
@pytest.mark.parametrize("lens", [[90000, 16, 150000, 16, 17, 40000], [16, 90000, 60000], [40000, 16] * 9])
def test_long_ragged_launches_equal_sequences_alone(lens):
    hkv, g, w, d, c = 8, 2, 16, 64, 33
    gen = torch.Generator(device=DEV).manual_seed(3)
    k = torch.randn((max(lens), hkv, d), generator=gen, device=DEV).bfloat16()      # every sequence is a prefix of the same cache
    q = torch.randn((len(lens), hkv * g, w, d), generator=gen, device=DEV).bfloat16()

    def score(lens, q):
        prob = ckv.Problem(hkv * g, hkv, d, w, c, ckv.BF16, lens, [0] * len(lens), [0] * len(lens), d, hkv * d)
        ws = torch.full((ckv.chunkkv_workspace_bytes(prob),), 0xFF, dtype=torch.uint8, device=DEV)
        scores = torch.full((len(lens), hkv, max(1, prob.score_cap)), -1.0, device=DEV)
        ckv.chunkkv_score(prob, q, k, scores, None, ws)
        return scores

    got = score(lens, q)
    for b, n in enumerate((L - w + c - 1) // c for L in lens):
        alone = score(lens[b:b + 1], q[b:b + 1].contiguous())[0, :, :n]
        assert n == 0 or float(((got[b, :, :n] - alone).abs() / alone).max()) < 2e-6, b
        assert (got[b, :, n:] == -1.0).all()
