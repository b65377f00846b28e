"""Chunk selection at the sizes and score patterns where its kernels change form: one, four and sixteen stripes of
chunks per thread, registers or re-reading, few or many candidates in the threshold's bin, more equal scores than the
list of candidates holds, the ragged tail at the threshold.  Bit-exact against the oracle on the same fp32 scores."""
import numpy as np
import pytest
import torch

from oracle import chunkkv_oracle as orc

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


def scores_of(kind, C, heads, rng):
    if kind == "spread":         # five orders of magnitude
        s = np.exp(2.5 * rng.standard_normal((heads, C)))
    elif kind == "narrow":       # around a power of two, a few thousand distinct values
        s = 2.0 + 1e-4 * rng.standard_normal((heads, C))
    elif kind == "ties":         # seven values: hundreds to thousands of equal scores at the threshold
        s = rng.integers(0, 7, (heads, C)).astype(np.float64)
    elif kind == "outlier":      # one score far above the rest, which are within a few ulp of one another
        s = 1.0 + 2.0 ** -23 * rng.integers(0, 40, (heads, C))
        s[:, rng.integers(0, C)] = 1e20
    else:                        # all zero
        s = np.zeros((heads, C))
    return s.astype(np.float32)


@pytest.mark.parametrize("whole", [False, True])
@pytest.mark.parametrize("kind", ["spread", "narrow", "ties", "outlier", "zero"])
@pytest.mark.parametrize("C", [1, 2, 255, 256, 257, 1023, 1025, 4096, 4097, 16384, 16385, 40001])
def test_selection_is_exact(lib, C, kind, whole):
    heads, c, w = 3, 3, 2
    rng = np.random.default_rng(C)
    P = C * c - (C % 3)          # ragged tail of 1 or 2 tokens, or none
    for keep in sorted({1, min(2, P), P // 10 or 1, P // 2 or 1, P - 1 or 1, P}):
        s = scores_of(kind, C, heads, rng)
        prob = lib.Problem(heads, heads, 64, w, c, lib.F32, [P + w], [keep], [0], (P + w) * 64, 64,
                           flags=lib.FLAG_WHOLE_CHUNKS if whole else 0)
        sc = torch.full((heads, prob.sel_cap), -7, dtype=torch.int32, device=DEV)
        sl, n = torch.full_like(sc, -7), torch.full((heads,), -7, dtype=torch.int32, device=DEV)
        t = torch.zeros((heads, prob.score_cap), dtype=torch.float32, device=DEV)
        t[:, :C] = torch.from_numpy(s).to(DEV)
        print(f"C={C} {kind} whole={whole} keep={keep}", flush=True)
        lib.chunkkv_chunk_topk(prob, t, sc, sl, n)
        torch.cuda.synchronize()
        for h in range(heads):
            want = orc.chunk_topk_whole(s[h], P, c, keep) if whole else orc.chunk_topk(s[h], P, c, keep)
            k = int(n[h])
            assert k == len(want[0])
            assert np.array_equal(sc[h, :k].cpu().numpy(), want[0]) and np.array_equal(sl[h, :k].cpu().numpy(), want[1])
            assert (sc[h, k:] == -7).all() and (sl[h, k:] == -7).all()


@pytest.mark.parametrize("C", [100, 3000, 20000])
def test_the_lowest_nan_is_selected_last(lib, C):
    """A score whose bits are all ones is the lowest of all keys: never ahead of a number, in no form of the kernel."""
    c, w, keep = 3, 2, 3 * (C // 2)
    s = scores_of("spread", C, 1, np.random.default_rng(C))
    t = torch.from_numpy(s).to(DEV)
    t.view(torch.int32)[0, 5] = -1
    prob = lib.Problem(1, 1, 64, w, c, lib.F32, [C * c + w], [keep], [0], (C * c + w) * 64, 64)
    sc = torch.full((1, prob.sel_cap), -7, dtype=torch.int32, device=DEV)
    sl, n = torch.full_like(sc, -7), torch.full((1,), -7, dtype=torch.int32, device=DEV)
    full = torch.zeros((1, prob.score_cap), dtype=torch.float32, device=DEV)
    full.view(torch.int32)[:, :C] = t.view(torch.int32)
    lib.chunkkv_chunk_topk(prob, full, sc, sl, n)
    torch.cuda.synchronize()
    s[0, 5] = -1.0
    want = orc.chunk_topk(s[0], C * c, c, keep)
    k = int(n[0])
    assert k == len(want[0]) and np.array_equal(sc[0, :k].cpu().numpy(), want[0]) and np.array_equal(sl[0, :k].cpu().numpy(), want[1])
