"""Launches that the timing aid reports, per kind, against those each call makes: a kernel that is not launched leaves no record."""
import pytest
import torch

import paper_2502_00299_amd as ckv

pytestmark = pytest.mark.gpu
DEV = "cuda:0"
STATS, COMBINE, COLSUM, CHUNK_SUMS, SELECT, COMPACT = range(6)

# (prefix tokens, chunk, layers that share a selection, head_dim, caller's log-sum-exps): launches by kind
CASES = [
    ((500, 10, 2, 64, False), {STATS: 1, COLSUM: 1, COMPACT: 1}),                      # selects while it gathers
    ((500, 10, 2, 64, True), {COLSUM: 1, COMPACT: 1}),
    ((5000, 1, 2, 64, False), {STATS: 1, COLSUM: 1, SELECT: 1, COMPACT: 1}),           # too many chunks for that
    ((2560, 10, 32, 64, False), {STATS: 1, COLSUM: 1, COMPACT: 1}),                    # 256 chunks, one per thread: 1152 workgroups
    ((2570, 10, 27, 64, False), {STATS: 1, COLSUM: 1, COMPACT: 1}),                    # four per thread: 972 workgroups, ...
    ((10240, 10, 10, 64, False), {STATS: 1, COLSUM: 1, COMPACT: 1}),                   # ... 1320 ...
    ((10240, 10, 11, 64, False), {STATS: 1, COLSUM: 1, SELECT: 1, COMPACT: 1}),        # ... and 1452, where selecting apart is faster
    ((500, 10, 40, 64, False), {STATS: 1, COLSUM: 1, SELECT: 1, COMPACT: 2}),          # two launches' worth of layers
    ((700, 300, 1, 64, False), {STATS: 1, COLSUM: 1, CHUNK_SUMS: 1, COMPACT: 1}),
    ((3000, 10, 1, 128, False), {STATS: 1, COLSUM: 1, COMPACT: 1}),                    # single pass
    ((0, 10, 1, 128, False), {STATS: 1, COMPACT: 1}),                                  # nothing before the window
    ((0, 10, 1, 64, False), {STATS: 1, COMPACT: 1}),
    ((0, 300, 1, 64, True), {COMPACT: 1}),
]


@pytest.mark.parametrize("case,want", CASES)
def test_records_are_launches(case, want):
    P, c, layers, d, with_lse = case
    hkv, g, w = 2, 4, 32
    L = P + w
    prob = ckv.Problem(hkv * g, hkv, d, w, c, ckv.BF16, [L], [P // 4], [0], L * d, d)
    k = [torch.randn((hkv, L, d), device=DEV).bfloat16() for _ in range(layers)]
    q, lse = torch.randn((1, hkv * g, w, d), device=DEV).bfloat16(), torch.full((1, hkv * g, w), 6.0, device=DEV)
    sel = [torch.zeros((1, 1, hkv, prob.sel_cap), dtype=torch.int32, device=DEV) for _ in range(2)]
    cnt = torch.zeros((1, 1, hkv), dtype=torch.int32, device=DEV)
    out = [torch.zeros(prob.out_elements(), dtype=torch.bfloat16, device=DEV) for _ in range(2 * layers)]
    ws = torch.empty(ckv.chunkkv_workspace_bytes(prob, layers, layers), dtype=torch.uint8, device=DEV)
    rest = [None] * (layers - 1)
    ckv.chunkkv_timing_begin(64)
    for _ in range(3):
        if with_lse:
            ckv.chunkkv_compress_stack_lse(prob, layers, [q] + rest, k, k, [lse] + rest, out[:layers], out[layers:], *sel, cnt, ws)
        else:
            ckv.chunkkv_compress_stack(prob, layers, [q] + rest, k, k, out[:layers], out[layers:], *sel, cnt, ws)
    got = [n for _, n in ckv.chunkkv_timing_end().values()]
    assert got == [3 * want.get(kind, 0) for kind in range(len(got))]
