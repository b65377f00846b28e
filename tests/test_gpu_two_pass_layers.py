"""Two-pass scoring gives the same bits however many layers share its launches: the stack call, the call with a chunk size per group and
the per-layer calls select the same chunks, on keys whose chunks differ by rounding alone (every chunk holds the same keys in
another order), also where the workspace holds the statistics of a few of the stack's layers at a time."""
import pytest
import torch

import paper_2502_00299_amd as ckv

pytestmark = pytest.mark.gpu
DEV = "cuda:0"
KIND = {ckv.F32: torch.float32, ckv.BF16: torch.bfloat16, ckv.F16: torch.float16}


@pytest.mark.parametrize("lens,layers,hkv,g,window,d,chunk,dtype", [
    ([2048], 8, 8, 2, 32, 128, 7, ckv.BF16),                 # statistics merged by the second pass in the layer call ...
    ([4097], 16, 8, 2, 32, 128, 7, ckv.BF16),                # ... by a kernel between the passes in the stack call
    ([4096], 32, 8, 4, 16, 128, 9, ckv.F16),
    ([513], 16, 2, 2, 16, 64, 5, ckv.F32),
    ([6000], 8, 4, 4, 32, 128, 6, ckv.F32),
    ([3000, 700, 65, 1900, 5000], 8, 4, 7, 32, 64, 11, ckv.BF16),
    ([700, 130, 2500] * 6, 6, 2, 2, 32, 128, 7, ckv.BF16),   # more sequences than a launch takes
    ([20011], 32, 16, 1, 32, 64, 33, ckv.BF16),              # sets of layers
    ([9000, 400], 40, 8, 8, 64, 128, 3, ckv.F16),            # 512 rows, more layers than a launch takes
    ([70001], 2, 32, 1, 16, 128, 13, ckv.BF16),              # the kernel merges in the layer call, too
    ([140001], 2, 8, 1, 16, 128, 13, ckv.BF16),              # 122 ranges, more than the second pass merges
])
def test_layers_equal_stack(lens, layers, hkv, g, window, d, chunk, dtype):
    gen = torch.Generator(device=DEV).manual_seed(sum(lens) + layers)
    B, hq, total = len(lens), hkv * g, sum(lens)
    starts = [sum(lens[:b]) * hkv * d for b in range(B)]
    keep = [3 * (n - window) // 10 for n in lens]
    few = torch.randn((hkv, chunk, d), generator=gen, device=DEV)    # a head's keys: every chunk is a permutation of them
    order = torch.rand((total // chunk + B, chunk), generator=gen, device=DEV).argsort(1)
    k, first = torch.empty((total, hkv, d), device=DEV), 0
    for b, n in enumerate(lens):
        rows = order[first:first + n // chunk + 1].reshape(-1)[:n]
        first += n // chunk + 1
        k[sum(lens[:b]):sum(lens[:b]) + n] = few[:, rows].transpose(0, 1)
    k = k.to(KIND[dtype])
    q = [torch.randn((B, hq, window, d), generator=gen, device=DEV).to(KIND[dtype]) for _ in range(layers)]
    prob = ckv.Problem(hq, hkv, d, window, chunk, dtype, lens, keep, starts, d, hkv * d, flags=ckv.FLAG_TWO_PASS)
    ks = [k] * layers
    ko, vo = ([torch.zeros(prob.out_elements(), dtype=KIND[dtype], device=DEV) for _ in range(layers)] for _ in range(2))

    def selection():
        sel = [torch.zeros((layers, B, hkv, prob.sel_cap), dtype=torch.int32, device=DEV) for _ in range(2)]
        return sel + [torch.zeros((layers, B, hkv), dtype=torch.int32, device=DEV)]

    one, stack, mixed = selection(), selection(), selection()
    ws = torch.full((ckv.chunkkv_workspace_bytes(prob, 1, 1),), 0xFF, dtype=torch.uint8, device=DEV)
    for layer in range(layers):
        ckv.chunkkv_compress_layer(prob, layer, 1, q[layer], None, k, k, ko[layer], vo[layer], *one, ws)
    ws = torch.full((ckv.chunkkv_workspace_bytes(prob, layers, 1),), 0xFF, dtype=torch.uint8, device=DEV)
    ckv.chunkkv_compress_stack(prob, 1, q, ks, ks, ko, vo, *stack, ws)
    assert int(one[2].min()) > 0 and int(one[1].sum()) == layers * hkv * sum(keep)
    for a, b in zip(one, stack):
        assert torch.equal(a, b)
    table = [chunk + (layer % 3 == 1) for layer in range(layers)]
    ws = torch.full((ckv.chunkkv_workspace_bytes_hybrid(prob, layers, 1, table),), 0xFF, dtype=torch.uint8, device=DEV)
    ckv.chunkkv_compress_stack_hybrid(prob, 1, table, q, ks, ks, None, ko, vo, *mixed, ws)
    same = [layer for layer in range(layers) if table[layer] == chunk]
    for a, b in zip(one, mixed):
        assert torch.equal(a[same], b[same])
