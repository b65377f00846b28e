"""Calls on either side of the lines from which K and V are read with streaming loads: the stack call (192 MB) and the per-layer
call (64 MB) give the same selections and the same gathered bytes, which are rows of the caches."""
import pytest
import torch

import paper_2502_00299_amd as ckv

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


@pytest.mark.parametrize("chunk,window,dtype", [(10, 64, ckv.BF16), (20, 32, ckv.F16), (5, 64, ckv.F16), (7, 32, ckv.BF16)])
@pytest.mark.parametrize("n", [8191, 8193, 24575, 24577])   # 8 kv-heads of 128: 32 MB and 96 MB of K and V a layer, and a little more
def test_stack_equals_layers(n, chunk, window, dtype):
    hkv, g, d, N = 8, 4, 128, 2
    kind = {ckv.BF16: torch.bfloat16, ckv.F16: torch.float16}[dtype]
    gen = torch.Generator(device=DEV).manual_seed(n)
    k, v = ([torch.randn((hkv, n, d), generator=gen, device=DEV).to(kind) for _ in range(N)] for _ in range(2))
    q = torch.randn((1, hkv * g, window, d), generator=gen, device=DEV).to(kind)
    keep = (n - window) // 10
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
        chunks, lens = sel[0][0, 0, h, :m], sel[1][0, 0, h, :m]
        assert torch.equal(chunks, sel1[0][0, 0, h, :m]) and torch.equal(lens, sel1[1][0, 0, h, :m]) and int(lens.sum()) == keep
        rows = torch.cat([torch.arange(int(c) * chunk, int(c) * chunk + int(m_), device=DEV) for c, m_ in zip(chunks.cpu(), lens.cpu())] +
                         [torch.arange(n - window, n, device=DEV)])
        for x, src in zip(out, k + v):
            assert torch.equal(x.view(hkv, keep + window, d)[h], src[h][rows])
    for a, b in zip(out, out1):
        assert torch.equal(a, b)
