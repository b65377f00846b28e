"""Importance pass in short launches: smaller super-tiles against the largest ones, which the oracle tests hold.  The caller's
log-sum-exps make both the same bits: chunks shorter than, as long as and longer than a super-tile, prefixes that end inside
one and at its edge, each key-tile size (d=64, 128, each type, few and many rows)."""
import pytest
import torch

import paper_2502_00299_amd as ckv

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


def stride(prefixes, hkv, c, row_bytes):
    """Keys of a super-tile in a launch over these prefixes (at most 16 sequences): whole chunks of at most 256 keys, halved
    down to 64 or the key tile (16 KB) until there are 256 of them."""
    keys = 256
    while True:
        n = keys // c * c if c <= keys else c
        if sum(-(-p // n) for p in prefixes) * hkv >= 256 or keys // 2 < 16384 // row_bytes or keys <= 64:
            return n
        keys //= 2


@pytest.mark.parametrize("dtype", [ckv.BF16, ckv.F16, ckv.F32])
@pytest.mark.parametrize("d,g,w", [(64, 1, 8), (64, 8, 32), (128, 4, 32), (128, 1, 33)])
@pytest.mark.parametrize("c", [1, 3, 10, 33, 64, 65, 100, 128, 129, 256])
def test_same_bits_as_a_large_launch(c, d, g, w, dtype):
    gen = torch.Generator(device=DEV).manual_seed(c * d + g)
    # the large launch holds twelve more sequences of 11 * 256 prefix tokens: 264 super-tiles of them alone
    hkv, lens, fill = 2, [513 + w, 1 + w, 64 * c + w, 700], [11 * 256 + w] * 12
    td = {ckv.BF16: torch.bfloat16, ckv.F16: torch.float16, ckv.F32: torch.float32}[dtype]
    k = torch.randn((max(lens + fill) + 1, hkv, d), generator=gen, device=DEV).to(td)
    q = torch.randn((len(lens), hkv * g, w, d), generator=gen, device=DEV).to(td)
    lse = torch.rand((len(lens), hkv * g, w), generator=gen, device=DEV) + 5

    def score(lens, q, lse):      # every sequence is a prefix of the same cache
        prob = ckv.Problem(hkv * g, hkv, d, w, c, dtype, lens, [0] * len(lens), [0] * len(lens), d, hkv * d)
        scores = torch.full((len(lens), hkv, prob.score_cap), -1.0, device=DEV)
        ws = torch.full((ckv.chunkkv_workspace_bytes(prob, 1, 1),), 0xFF, dtype=torch.uint8, device=DEV)
        ckv.chunkkv_score_lse(prob, q, k, lse, scores, None, ws)
        return scores

    n, row_bytes = len(lens), d * td.itemsize
    largest = 256 // c * c
    assert stride([m - w for m in lens + fill], hkv, c, row_bytes) == largest
    alone_strides = [stride([m - w], hkv, c, row_bytes) for m in lens]
    # every call alone is cut finer, as far as it can be; above 128 tokens a super-tile is one chunk either way
    assert alone_strides == [max(64, 16384 // row_bytes) // c * c or c] * n
    assert c > 128 or max(alone_strides) < largest
    many = score(lens + fill, torch.cat([q, q[:1].expand(len(fill), -1, -1, -1)]).contiguous(),
                 torch.cat([lse, lse[:1].expand(len(fill), -1, -1)]).contiguous())
    for b in range(n):
        alone = score(lens[b:b + 1], q[b:b + 1].contiguous(), lse[b:b + 1].contiguous())
        chunks = (lens[b] - w + c - 1) // c
        assert torch.equal(alone[0, :, :chunks], many[b, :, :chunks])
