"""Decode attention of 16-bit caches where its matrix-core kernel can go wrong: the edges of a 32-row step, of the
one-range and the many-range forms and of a range, padded head batches, the parts a weight is cut into, and strides
its 32-bit offsets cannot hold."""
import numpy as np
import pytest
import torch

from oracle import chunkkv_oracle as orc

pytestmark = pytest.mark.gpu
DEV = "cuda:0"
# fp32 accumulation of 128 products, an exponential and n weighted rows: a few 2^-24 of the logits' size (up to about
# 100 before scaling, 1e-6 of a weight) and about sqrt(n) 2^-24 of the row for the sums; 20 times that
TOL = 2e-5


def bits(t):
    t = t.cpu().contiguous()
    return t.view(torch.int16).numpy().view(np.uint16) if t.dtype == torch.bfloat16 else t.numpy()


def run(lib, dtype, n, hq, hkv, d, k, v, q, kv_len=None, stride_tok=None, scale=0.0):
    """Compacted-cache call over k, v [hkv][n][d] (strided copies when stride_tok is given)."""
    stride_tok = stride_tok or d
    stride_head = n * stride_tok if stride_tok == d else d
    prob = lib.Problem(hq, hkv, d, 1, 1, {torch.bfloat16: lib.BF16, torch.float16: lib.F16}[dtype], [n], [n - 1], [0], n * d, d,
                       [0], stride_head, stride_tok, softmax_scale=scale)
    kk, vv = k, v
    if stride_tok != d:
        kk, vv = (torch.zeros((n - 1) * stride_tok + hkv * d, dtype=dtype, device=DEV) for _ in range(2))
        for src, dst in ((k, kk), (v, vv)):
            torch.as_strided(dst, (hkv, n, d), (stride_head, stride_tok, 1)).copy_(src)
    out = torch.full((1, hq, d), 7.0, dtype=torch.float32, device=DEV)
    lse = torch.full((1, hq), 7.0, dtype=torch.float32, device=DEV)
    ws = torch.empty(lib.chunkkv_decode_workspace_bytes(prob, True), dtype=torch.uint8, device=DEV)
    lib.chunkkv_decode_attention(prob, True, kv_len, q, kk, vv, out, lse, ws)
    torch.cuda.synchronize()
    return out[0].cpu().numpy(), lse[0].cpu().numpy()


def check(out, lse, q, k, v, n, scale=None):
    hq, hkv = q.shape[0], k.shape[0]
    g = hq // hkv
    for h in range(hkv):
        o_ref, l_ref = orc.decode_attention(bits(q[h * g:(h + 1) * g]), bits(k[h:h + 1, :n]), bits(v[h:h + 1, :n]), scale)
        err = np.abs(out[h * g:(h + 1) * g] - o_ref).max(axis=1) / np.abs(o_ref).max(axis=1)
        assert err.max() <= TOL, (h, err)
        assert np.abs(lse[h * g:(h + 1) * g] - l_ref).max() <= TOL * 10


@pytest.mark.parametrize("dtype", [torch.bfloat16, torch.float16])
@pytest.mark.parametrize("n,hq,hkv,d", [(1, 4, 1, 128), (31, 8, 2, 64), (33, 7, 1, 128), (255, 3, 3, 128), (256, 8, 1, 64), (257, 4, 1, 128),
                                        (257, 10, 2, 64), (1025, 8, 1, 128), (5000, 9, 1, 128), (4097, 36, 9, 64), (20011, 8, 2, 128)])
def test_edges(lib, dtype, n, hq, hkv, d):
    gen = torch.Generator(device=DEV).manual_seed(n)
    q, k, v = (torch.randn(s, generator=gen, device=DEV).mul_(a).to(dtype) for s, a in (((hq, d), 2.0), ((hkv, n, d), 1.0), ((hkv, n, d), 1.0)))
    print(f"n={n} hq={hq} hkv={hkv} d={d} {dtype}", flush=True)
    out, lse = run(lib, dtype, n, hq, hkv, d, k, v, q)
    check(out, lse, q, k, v, n)
    if n > 40:   # fewer tokens than the cache holds: the rows behind them must not count
        m = n - 37
        out, lse = run(lib, dtype, n, hq, hkv, d, k, v, q, kv_len=torch.full((1, hkv), m, dtype=torch.int32, device=DEV))
        check(out, lse, q, k, v, m)


@pytest.mark.parametrize("dtype", [torch.bfloat16, torch.float16])
@pytest.mark.parametrize("peak", [0, 300, 599])
def test_one_token_far_above_many(lib, dtype, peak):
    """One token 25 nats above 599 equal ones, wherever it comes: the others' weights (1.4e-11) stay in the sums."""
    n, d, hq = 600, 128, 4
    u = torch.zeros(d, device=DEV)
    u[5] = 1.0
    k = torch.zeros((1, n, d), device=DEV)
    k[0, peak] = 25.0 * u
    q = u.repeat(hq, 1)
    v = torch.zeros((1, n, d), device=DEV)
    v[0, :, 1] = 30000.0
    v[0, peak] = 0.0
    v[0, peak, 2] = 1.0
    q, k, v = q.to(dtype), k.to(dtype), v.to(dtype)
    out, lse = run(lib, dtype, n, hq, 1, d, k, v, q, scale=1.0)
    p = np.exp(-25.0) / (1.0 + 599 * np.exp(-25.0))
    want = 599 * p * float(v[0, (peak + 1) % n, 1].float())
    assert np.abs(out[:, 1] / want - 1).max() <= 1e-5 and np.abs(out[:, 2] - 1).max() <= 1e-6
    assert np.abs(lse - 25.0).max() <= 1e-5


@pytest.mark.parametrize("n,stride_tok", [(3, 1 << 22), (300, 1 << 22), (33, (1 << 25) - 128), (33, 1 << 25)])
def test_strides_past_32_bit_offsets(lib, n, stride_tok):
    """Rows 8 and 64 MB apart: the offsets of a head, and past 64 MB those of a step, do not fit 32 bits."""
    d, hq, hkv = 128, 8, 2
    gen = torch.Generator(device=DEV).manual_seed(3)
    q, k, v = (torch.randn(s, generator=gen, device=DEV).to(torch.bfloat16) for s in ((hq, d), (hkv, n, d), (hkv, n, d)))
    out, lse = run(lib, torch.bfloat16, n, hq, hkv, d, k, v, q, stride_tok=stride_tok + 64)
    check(out, lse, q, k, v, n)


def test_cache_past_32_bit_offsets(lib):
    """Rows 64 KB apart, as in a cache that holds all layers of a token together: 2.6 GB."""
    n, d, hq, hkv = 40000, 128, 8, 2
    gen = torch.Generator(device=DEV).manual_seed(4)
    q, k, v = (torch.randn(s, generator=gen, device=DEV).to(torch.bfloat16) for s in ((hq, d), (hkv, n, d), (hkv, n, d)))
    out, lse = run(lib, torch.bfloat16, n, hq, hkv, d, k, v, q, stride_tok=32768)
    check(out, lse, q, k, v, n)


@pytest.mark.parametrize("dtype", [torch.bfloat16, torch.float16])
@pytest.mark.parametrize("n,hq,d", [(200, 4, 128), (1000, 7, 128), (5000, 4, 64)])
def test_infinite_values_stay_infinite(lib, dtype, n, hq, d):
    """An infinity in V under an ordinary weight, under an exact power of two (parts of it are zero) and under a tiny
    one reaches the output as that infinity; everything else stays what it is."""
    gen = torch.Generator(device=DEV).manual_seed(n)
    q, k, v = (torch.randn(s, generator=gen, device=DEV).to(dtype) for s in ((hq, d), (1, n, d), (1, n, d)))
    q[:, 0], k[0, :, 0] = 4.0, 0.0
    k[0, n // 2, 0], k[0, 7, 0] = 0.0, -40.0 if d == 128 else -30.0   # token 7: 14 or 15 nats below its like
    k[0, n - 1] = 0.0
    inf_at = {1: (n // 2, float("inf")), 2: (7, float("-inf")), 3: (n - 1, float("inf")), 5: (0, float("inf"))}
    finite = v.clone()
    for col, (tok, val) in inf_at.items():
        v[0, tok, col] = val
    out, lse = run(lib, dtype, n, hq, 1, d, k, v, q)
    for col, (_, val) in inf_at.items():
        assert (out[:, col] == val).all(), (col, out[:, col])
    cols = [i for i in range(d) if i not in inf_at]
    want, _ = orc.decode_attention(bits(q), bits(k), bits(finite))
    assert (np.abs(out - want)[:, cols].max(axis=1) / np.abs(want).max(axis=1)).max() <= TOL


@pytest.mark.parametrize("dtype", [torch.bfloat16, torch.float16])
@pytest.mark.parametrize("nats", [25.0, 30.0, 40.0, 60.0])
@pytest.mark.parametrize("n,hq,d", [(200, 4, 128), (600, 8, 128), (5000, 4, 64)])
def test_weights_far_below_the_reference(lib, dtype, n, hq, d, nats):
    """Every 32nd token `nats` above the rest, its value zero where theirs is not: the small weights keep their size.  fp16
    cuts a weight off below 2^-72; otherwise it is rounded as its exponent is, by 2^-19 (half an ulp of 60 log2 e) and
    half an ulp of v_exp.  An infinity under such a weight, cut off or not, is an infinity."""
    k = torch.zeros((1, n, d), device=DEV)
    k[0, ::32, 5] = nats
    q = torch.zeros((hq, d), device=DEV)
    q[:, 5] = 1.0
    v = torch.zeros((1, n, d), device=DEV)
    v[0, :, 1] = 30000.0
    v[0, ::32, 1] = 0.0
    v[0, ::32, 2] = 1.0
    v[0, 5, 7], v[0, 64, 9] = float("inf"), float("-inf")
    q, k, v = q.to(dtype), k.to(dtype), v.to(dtype)
    out, lse = run(lib, dtype, n, hq, 1, d, k, v, q, scale=1.0)
    peaks = (n + 31) // 32
    total = peaks + (n - peaks) * np.exp(-nats)
    value = float(v[0, 1, 1].float())
    want = (n - peaks) * np.exp(-nats) * value / total
    cut = (n - peaks) * 2.0 ** -72 * value / total if dtype == torch.float16 else 0.0
    assert np.abs(out[:, 1] - want).max() <= cut + 1e-5 * want, (out[:, 1], want)
    assert np.abs(out[:, 2] * total / peaks - 1).max() <= 1e-6
    assert (out[:, 7] == np.inf).all() and (out[:, 9] == -np.inf).all()
    assert (np.delete(out, (1, 2, 7, 9), axis=1) == 0).all()
    assert np.abs(lse - nats - np.log(total) + 0.0).max() <= 1e-5


@pytest.mark.parametrize("dtype", [torch.bfloat16, torch.float32])
@pytest.mark.parametrize("lens,hq,hkv", [([4111] + [61] * 15, 32, 32), ([50, 3000, 1, 700, 513, 2999], 14, 2), ([900] * 16 + [4000, 33], 8, 8)])
def test_uneven_batches(lib, dtype, lens, hq, hkv):
    """Sequences cut into different numbers of ranges share the places of the workspace; 18 sequences take two launches."""
    d, B = 64, len(lens)
    gen = torch.Generator(device=DEV).manual_seed(B)
    base = [sum(lens[:i]) * hkv * d for i in range(B)]
    q = torch.randn((B, hq, d), generator=gen, device=DEV).to(dtype)
    k, v = (torch.randn(sum(lens) * hkv * d, generator=gen, device=DEV).to(dtype) for _ in range(2))
    prob = lib.Problem(hq, hkv, d, 1, 1, lib.F32 if dtype == torch.float32 else lib.BF16, lens, [0] * B, base, d, hkv * d)
    out, lse = torch.full((B, hq, d), 7.0, device=DEV), torch.full((B, hq), 7.0, device=DEV)
    room = lib.chunkkv_decode_workspace_bytes(prob, False)
    ws = torch.full((room + 4096,), 0x5A, dtype=torch.uint8, device=DEV)
    lib.chunkkv_decode_attention(prob, False, None, q, k, v, out, lse, ws[:room])
    torch.cuda.synchronize()
    assert (ws[room:] == 0x5A).all()
    for b, n in enumerate(lens):
        kk, vv = (x[base[b]:base[b] + n * hkv * d].view(n, hkv, d).transpose(0, 1).contiguous() for x in (k, v))
        check(out[b].cpu().numpy(), lse[b].cpu().numpy(), q[b], kk, vv, n)
