"""Calls on either side of the lines from which K and V are read, and K' and V' written, with streaming accesses, for rows of 128, 256
and 512 bytes: the stack call (192 MB of K and V, 128 MB of K' and V') and the per-layer call (64 MB, 4 MB) give the same selections and
the same gathered bytes, which are rows of the caches."""
import pytest
import torch

import paper_2502_00299_amd as ckv

pytestmark = pytest.mark.gpu
DEV = "cuda:0"
TOKEN = 4096   # bytes of K and V of a token in a layer, in every case
KIND = {ckv.BF16: torch.bfloat16, ckv.F16: torch.float16, ckv.F32: torch.float32}


@pytest.mark.parametrize("chunk,window,dtype,d", [(10, 64, ckv.BF16, 128), (20, 32, ckv.F16, 128), (5, 64, ckv.F16, 128), (7, 32, ckv.BF16, 128),
                                                  (16, 32, ckv.BF16, 64), (9, 32, ckv.F32, 128)])
@pytest.mark.parametrize("n,kept", [(16383, 1001), (16385, 1001),      # two layers of 64 MB: the per-layer call's loads
                                    (9001, 1024), (9001, 1025),        # 4 MB of K' and V': its stores
                                    (24575, 2521), (24577, 2521),      # two layers of 96 MB: the stack call's loads
                                    (17001, 16384), (17001, 16385)])   # 128 MB of K' and V': its stores
def test_stack_equals_layers(n, kept, chunk, window, dtype, d):
    kind = KIND[dtype]
    g, N, hkv = 4, 2, TOKEN // (2 * d * torch.empty(0, dtype=kind).element_size())
    mb = 1 << 20
    edges = [n * TOKEN > 64 * mb, kept * TOKEN > 4 * mb, N * n * TOKEN > 192 * mb, N * kept * TOKEN > 128 * mb]
    assert edges == {16383: [False, False, False, False], 16385: [True, False, False, False], 9001: [False, kept == 1025, False, False],
                     24575: [True, True, False, False], 24577: [True, True, True, False], 17001: [True, True, False, kept == 16385]}[n]
    gen = torch.Generator(device=DEV).manual_seed(n)
    k, v = ([torch.randn((hkv, n, d), generator=gen, device=DEV).to(kind) for _ in range(N)] for _ in range(2))
    q = torch.randn((1, hkv * g, window, d), generator=gen, device=DEV).to(kind)
    keep = kept - window
    prob = ckv.Problem(hkv * g, hkv, d, window, chunk, dtype, [n], [keep], [0], n * d, d)

    def fresh():
        sel = [torch.zeros((1, 1, hkv, prob.sel_cap), dtype=torch.int32, device=DEV) for _ in range(2)] + [torch.zeros((1, 1, hkv), dtype=torch.int32, device=DEV)]
        return sel, [torch.zeros(prob.out_elements(), dtype=kind, device=DEV) for _ in range(2 * N)]

    sel, out = fresh()
    ws = torch.empty(ckv.chunkkv_workspace_bytes(prob, N, N), dtype=torch.uint8, device=DEV)
    ckv.chunkkv_compress_stack(prob, N, [q, None], k, v, out[:N], out[N:], *sel, ws)
    sel1, out1 = fresh()
    ws1 = torch.empty(ckv.chunkkv_workspace_bytes(prob, 1, 1), dtype=torch.uint8, device=DEV)
    for layer in range(N):
        ckv.chunkkv_compress_layer(prob, layer, N, q if layer == 0 else None, None, k[layer], v[layer], out1[layer], out1[N + layer], *sel1, ws1)
    count = sel[2][0, 0]
    assert torch.equal(sel[2], sel1[2])
    for h in range(hkv):
        m = int(count[h])
        chunks, lens = sel[0][0, 0, h, :m].long(), sel[1][0, 0, h, :m].long()
        assert torch.equal(chunks, sel1[0][0, 0, h, :m].long()) and torch.equal(lens, sel1[1][0, 0, h, :m].long()) and int(lens.sum()) == keep
        first = torch.cumsum(lens, 0) - lens   # place of every entry's first row
        rows = torch.repeat_interleave(chunks * chunk - first, lens) + torch.arange(keep, device=DEV)
        rows = torch.cat([rows, torch.arange(n - window, n, device=DEV)])
        for x, src in zip(out, k + v):
            assert torch.equal(x.view(hkv, kept, d)[h], src[h][rows])
    for a, b in zip(out, out1):
        assert torch.equal(a, b)
