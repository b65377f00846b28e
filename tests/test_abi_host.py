"""Host-side checks of the C-ABI library that need no GPU: it loads, exports every symbol the header
declares, and every argument check returns its status before anything is enqueued."""
import copy
import ctypes as C
import os
import pickle
import re

import numpy as np
import pytest
import torch

import paper_2502_00299_amd as pkg

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


@pytest.fixture(scope="module")
def lib():
    if not os.path.exists(pkg.LIB_PATH):
        from paper_2502_00299_amd import build
        build.build(verbose=False)
    return pkg.load_library()


def header_functions():
    text = open(os.path.join(ROOT, "include", "chunkkv.h")).read()
    text = re.sub(r"/\*.*?\*/", "", text, flags=re.S)
    return sorted(set(re.findall(r"\b(chunkkv_[a-z_]+)\s*\(", text)))


def test_every_declared_symbol_is_exported(lib):
    names = header_functions()
    assert set(names) == set(pkg.SYMBOLS)
    for n in names:
        assert getattr(lib, n) is not None


def test_status_strings(lib):
    seen = {lib.chunkkv_status_string(i).decode() for i in range(6)}
    assert len(seen) == 6 and "ok" in seen
    assert lib.chunkkv_status_string(99).decode() == "unknown status"


def good(**kw):
    d = dict(n_q_heads=32, n_kv_heads=8, head_dim=128, window=32, chunk=10, dtype=pkg.BF16, seqlen=[8192],
             n_keep=[816], kv_base=[0], kv_stride_head=8192 * 128, kv_stride_tok=128)
    d.update(kw)
    return pkg.Problem(**d)


FAKE = C.c_void_p(0x1000)  # never dereferenced: every call below fails its argument check first


def score_rc(lib, prob, q=FAKE, k=FAKE, out=FAKE, ws=FAKE, ws_bytes=1 << 40):
    return lib.chunkkv_score(C.byref(prob.as_c()), q, k, out, None, ws, ws_bytes, None)


def test_workspace_size_is_positive_and_grows_with_layers(lib):
    p = good()
    a = pkg.chunkkv_workspace_bytes(p, 1, 1)
    b = pkg.chunkkv_workspace_bytes(p, 32, 1)
    c = pkg.chunkkv_workspace_bytes(p, 32, 2)
    assert 0 < a < c < b


def test_every_storage_type_is_accepted(lib):
    """fp32, bf16 and fp16 caches pass validation; the 16-bit types need the same workspace."""
    sizes = {dt: pkg.chunkkv_workspace_bytes(good(dtype=dt), 4, 2) for dt in (pkg.F32, pkg.BF16, pkg.F16)}
    assert all(v > 0 for v in sizes.values()) and sizes[pkg.BF16] == sizes[pkg.F16]
    assert (pkg.F32, pkg.BF16, pkg.F16) == (0, 1, 2)          # the enum of the header
    assert score_rc(lib, good(dtype=pkg.F16), ws=None) == 4   # argument checks reach the workspace check


@pytest.mark.parametrize("kw,status", [
    (dict(n_q_heads=30), 2),                       # Hq % Hkv != 0
    (dict(window=0), 2),
    (dict(chunk=0), 2),
    (dict(seqlen=[16]), 2),                        # w > L
    (dict(n_keep=[8161]), 2),                      # n_keep > P
    (dict(n_keep=[-1]), 2),
    (dict(sel_cap=5), 2),                          # needs ceil(816/10)+1 = 83
    (dict(score_cap=10), 2),                       # needs 816
    (dict(kv_stride_tok=100), 2),                  # < head_dim
    (dict(kv_stride_tok=132), 2),                  # rows not 16-byte aligned
    (dict(kv_base=[3]), 2),
    (dict(softmax_scale=-1.0), 2),
    (dict(head_dim=96), 3),
    (dict(dtype=7), 3),
    (dict(flags=4), 3),                            # unknown flag bit
    (dict(flags=0x80000000), 3),
    (dict(window=64, n_q_heads=128, n_keep=[100]), 3),   # g*w = 1024 rows > 512
    # K rows of one (sequence, kv-head) must span < 2 GiB: 1.1 M tokens of a packed 8-head bf16 cache do not
    (dict(seqlen=[1_100_000], n_keep=[1000], kv_stride_head=128, kv_stride_tok=8 * 128), 3),
])
def test_problem_validation(lib, kw, status):
    p = good(**kw)
    assert score_rc(lib, p) == status
    assert pkg.chunkkv_workspace_bytes(p) == 0


def test_flags_travel_per_call(lib):
    """Selection mode and scoring path are bits of chunkkv_problem.flags: every combination of the known bits
    passes validation, the flags change no workspace requirement's validity, and the library exports no
    process-wide switch for them."""
    assert (pkg.FLAG_WHOLE_CHUNKS, pkg.FLAG_TWO_PASS) == (1, 2)       # the values of the header
    for flags in (0, pkg.FLAG_WHOLE_CHUNKS, pkg.FLAG_TWO_PASS, pkg.FLAG_WHOLE_CHUNKS | pkg.FLAG_TWO_PASS):
        p = good(flags=flags)
        assert pkg.chunkkv_workspace_bytes(p, 4, 2) > 0
        assert score_rc(lib, p, ws=None) == 4                           # reaches the workspace check
    header = open(os.path.join(ROOT, "include", "chunkkv.h")).read()
    assert "CHUNKKV_FLAG_WHOLE_CHUNKS 1u" in header and "CHUNKKV_FLAG_TWO_PASS 2u" in header
    assert not [n for n in header_functions() if "_set_" in n]
    for name in ("chunkkv_set_whole_chunks", "chunkkv_set_single_pass", "chunkkv_set_overlap"):
        assert not hasattr(lib, name) or pytest.fail(f"{name} is still exported")


def test_null_pointers_and_workspace(lib):
    p = good()
    assert lib.chunkkv_score(None, FAKE, FAKE, FAKE, None, FAKE, 1 << 40, None) == 1
    assert score_rc(lib, p, q=None) == 1
    assert score_rc(lib, p, k=None) == 1
    assert score_rc(lib, p, out=None) == 1
    assert score_rc(lib, p, q=C.c_void_p(0x1004)) == 2             # misaligned device pointer
    assert score_rc(lib, p, ws=None) == 4
    assert score_rc(lib, p, ws_bytes=pkg.chunkkv_workspace_bytes(p) - 1) == 4
    cp = p.as_c()
    assert lib.chunkkv_chunk_topk(C.byref(cp), None, FAKE, FAKE, FAKE, None, 0, None) == 1
    assert lib.chunkkv_compact(C.byref(cp), FAKE, None, FAKE, FAKE, FAKE, FAKE, FAKE, None) == 1
    bad_out = good(out_base=[0], out_stride_head=848 * 128, out_stride_tok=100)
    assert lib.chunkkv_compact(C.byref(bad_out.as_c()), FAKE, FAKE, FAKE, FAKE, FAKE, FAKE, FAKE, None) == 2


def test_stack_argument_checks(lib):
    p = good()
    cp = p.as_c()
    n = 4
    tab = (C.c_void_p * n)(*[0x1000] * n)
    hole = (C.c_void_p * n)(0x1000, None, 0x1000, None)
    ws = pkg.chunkkv_workspace_bytes(p, n, 2)
    call = lambda q, k, reuse, nl=n, wsb=ws: lib.chunkkv_compress_stack(
        C.byref(cp), nl, reuse, q, k, tab, tab, tab, FAKE, FAKE, FAKE, FAKE, wsb, None)
    assert call(tab, tab, 0) == 2                  # R < 1
    assert call(tab, tab, 2, nl=0) == 2
    assert call(hole, hole, 2) == 1                # K of layer 1 missing
    assert call(hole, tab, 1) == 1                 # every layer needs Q when R = 1
    assert call(tab, tab, 2, wsb=ws - 1) == 4
    assert call(None, tab, 2) == 1


def test_lse_argument_checks(lib):
    # the log-sum-exp variants check what the plain calls check, plus the lse pointers (error paths only:
    # every call returns before a launch)
    p = good()
    cp = p.as_c()
    ws = pkg.chunkkv_workspace_bytes(p)
    assert lib.chunkkv_score_lse(C.byref(cp), FAKE, FAKE, None, FAKE, None, FAKE, ws, None) == 1
    assert lib.chunkkv_score_lse(C.byref(cp), FAKE, None, FAKE, FAKE, None, FAKE, ws, None) == 1
    assert lib.chunkkv_score_lse(C.byref(cp), FAKE, FAKE, FAKE, FAKE, None, FAKE, ws - 1, None) == 4
    n = 4
    tab = (C.c_void_p * n)(*[0x1000] * n)
    hole = (C.c_void_p * n)(0x1000, None, 0x1000, None)
    nol = (C.c_void_p * n)(None, None, 0x1000, None)
    ws4 = pkg.chunkkv_workspace_bytes(p, n, 2)
    call = lambda lse, reuse, wsb=ws4: lib.chunkkv_compress_stack_lse(
        C.byref(cp), n, reuse, tab, tab, tab, lse, tab, tab, FAKE, FAKE, FAKE, FAKE, wsb, None)
    assert call(None, 2) == 1
    assert call(nol, 2) == 1                       # leader layer 0 has no lse
    assert call(hole, 1) == 1                      # every layer is a leader when R = 1
    assert call(hole, 2, wsb=ws4 - 1) == 4         # lse of the non-leader layers may be missing


def test_layer_and_jaccard_argument_checks(lib):
    p = good()
    cp = p.as_c()
    ws = pkg.chunkkv_workspace_bytes(p)
    layer = lambda l, R, q, k=FAKE, wsb=ws: lib.chunkkv_compress_layer(
        C.byref(cp), l, R, q, None, k, FAKE, FAKE, FAKE, FAKE, FAKE, FAKE, FAKE, wsb, None)
    assert layer(-1, 2, FAKE) == 2
    assert layer(0, 0, FAKE) == 2
    assert layer(0, 2, None) == 1                  # a leader layer needs its window queries
    assert layer(2, 2, None) == 1
    assert layer(1, 2, None, k=None) == 1
    assert layer(1, 2, None, wsb=ws - 1) == 4      # a follower layer passes the checks up to the workspace
    assert lib.chunkkv_jaccard(C.byref(cp), 1, FAKE, FAKE, FAKE, FAKE, None) == 2
    assert lib.chunkkv_jaccard(C.byref(cp), 3, FAKE, None, FAKE, FAKE, None) == 1
    assert lib.chunkkv_jaccard(C.byref(cp), 3, FAKE, FAKE, FAKE, None, None) == 1


def test_hybrid_stack_argument_checks(lib):
    # chunk size per reuse group: the table is validated entry by entry, capacities against the smallest entry
    n, R = 5, 2
    tab = (C.c_void_p * n)(*[0x1000] * n)
    chunks = lambda *c: (C.c_int32 * len(c))(*c)
    p1 = good(chunk=1)                               # capacities sized for chunk 1 hold for every chunk size
    cp1 = p1.as_c()
    ws = lib.chunkkv_workspace_bytes_hybrid(C.byref(cp1), n, R, chunks(10, 1, 5))
    assert ws >= max(pkg.chunkkv_workspace_bytes(good(chunk=c, sel_cap=p1.sel_cap, score_cap=p1.score_cap), n, R)
                     for c in (10, 1, 5))
    call = lambda cp, table, wsb=ws, q=tab: lib.chunkkv_compress_stack_hybrid(
        C.byref(cp), n, R, table, q, tab, tab, None, tab, tab, FAKE, FAKE, FAKE, FAKE, wsb, None)
    assert call(cp1, None) == 1
    assert call(cp1, chunks(10, 0, 5)) == 2
    assert call(cp1, chunks(10, -3, 5)) == 2
    assert call(cp1, chunks(10, 1, 5), wsb=ws - 1) == 4
    assert call(cp1, chunks(10, 1, 5), q=None) == 1
    assert lib.chunkkv_workspace_bytes_hybrid(C.byref(cp1), n, R, chunks(10, 0, 5)) == 0
    assert lib.chunkkv_workspace_bytes_hybrid(C.byref(cp1), n, R, None) == 0
    # capacities sized for chunk 10 are too small for a group of chunk 1
    cp10 = good().as_c()
    assert call(cp10, chunks(10, 1, 5)) == 2
    assert call(cp10, chunks(10, 20, 10), wsb=1 << 40, q=None) == 1    # ... but fine for chunk sizes >= 10


def test_quality_metrics_argument_checks(lib):
    p = good()
    cp = p.as_c()
    ws = pkg.chunkkv_quality_workspace_bytes(p)
    assert ws >= max(pkg.chunkkv_decode_workspace_bytes(p, True), pkg.chunkkv_decode_workspace_bytes(p, False))
    call = lambda q=FAKE, k=FAKE, ko=FAKE, l1=FAKE, cos=FAKE, wsb=ws: lib.chunkkv_quality_metrics(
        C.byref(cp), None, q, k, FAKE, ko, FAKE, l1, cos, FAKE, wsb, None)
    assert call(q=None) == 1 and call(k=None) == 1 and call(ko=None) == 1 and call(l1=None) == 1 and call(cos=None) == 1
    assert call(k=C.c_void_p(0x1004)) == 2
    assert call(wsb=ws - 1) == 4
    bad = good(out_base=[0], out_stride_head=848 * 128, out_stride_tok=100)
    assert pkg.chunkkv_quality_workspace_bytes(bad) == 0


def contents(cp):
    """Everything the C struct of a Problem tells the library."""
    arrays = ("seqlen", "n_keep", "kv_base", "out_base")
    return {n: getattr(cp, n)[:cp.batch] if n in arrays else getattr(cp, n) for n, _ in cp._fields_}


HOLDERS = {"list": list, "array": np.array, "tensor": torch.tensor, "list of tensors": lambda x: [torch.tensor(i) for i in x]}


@pytest.mark.parametrize("holder", sorted(HOLDERS))
@pytest.mark.parametrize("field", ["seqlen", "n_keep", "kv_base", "out_base"])
def test_kept_struct_follows_changes_in_place(lib, field, holder):
    """A decoding loop that adds to its lengths or moves its offsets: the next call sees the new ones."""
    values = dict(seqlen=[8192, 4096], n_keep=[816, 400], kv_base=[0, 8192 * 1024], out_base=[0, 848 * 1024])
    p = good(**{n: HOLDERS[holder](x) for n, x in values.items()}, out_stride_head=128, out_stride_tok=1024, score_cap=7000)
    before = pkg.chunkkv_workspace_bytes(p, 1, 1)
    assert contents(p._c()._obj) == contents(p.as_c())
    if holder == "list of tensors":
        getattr(p, field)[1] += 8
    else:
        getattr(p, field)[0] += 8
    assert contents(p._c()._obj) == contents(p.as_c())
    assert contents(p._c()._obj)[field] != values[field]
    if field == "seqlen":
        p.seqlen[0] += 60000
        assert pkg.chunkkv_workspace_bytes(p, 1, 1) > before


def test_kept_struct_follows_assignments(lib):
    p = good()
    for name, value in dict(window=16, chunk=5, dtype=pkg.F16, sel_cap=2000, score_cap=3000, softmax_scale=0.25, flags=2, n_q_heads=16,
                            n_kv_heads=4, head_dim=64, kv_stride_head=64, kv_stride_tok=256, out_stride_head=128, out_stride_tok=512,
                            seqlen=[4096], n_keep=[17], kv_base=[64], out_base=[128]).items():
        was = contents(p._c()._obj)[name]
        setattr(p, name, value)
        now = contents(p._c()._obj)
        assert now == contents(p.as_c()) and now[name] == value != was
    vars(p)["window"] = 8
    assert p._c()._obj.window == 8
    p.softmax_scale = torch.tensor(0.5)
    p.window = torch.tensor(4)
    p._c()
    p.window += 1
    p.softmax_scale += 0.25
    assert (p._c()._obj.window, p._c()._obj.softmax_scale) == (5, 0.75)


def test_kept_struct_is_not_a_field(lib):
    p = good()
    p._c()
    assert pkg.Problem(**vars(p)) == p
    for q in (copy.copy(p), copy.deepcopy(p), pickle.loads(pickle.dumps(p))):
        assert q == p and q._c() is not p._c() and contents(q._c()._obj) == contents(p._c()._obj)
        q.window = 16
        assert p._c()._obj.window == 32 and q._c()._obj.window == 16


def test_missing_library_fails_loudly(tmp_path):
    with pytest.raises(RuntimeError, match="no CPU fallback"):
        pkg.load_library(str(tmp_path / "nope.so"))


def test_static_decode_takes_what_the_even_cut_fits():
    """One long sequence among short ones: cutting it finer must not push the partial results past the static scratch."""
    lens = [30848] + [33] * 15
    p = pkg.Problem(8, 1, 128, 16, 10, pkg.BF16, lens, [1] * 16, [0] * 16, 128 * 40000, 128)
    even = 16 * 8 * ((30848 + 255) // 256) * (128 * 4 + 8)
    assert even < 8 << 20
    assert even <= pkg.chunkkv_decode_workspace_bytes(p, False) <= 8 << 20


@pytest.mark.parametrize("pitch", [1 << 17, 1 << 19, 1 << 21, 1 << 23, 1 << 25])
def test_static_decode_does_not_depend_on_the_row_pitch(pitch):
    """Rows 256 KB to 64 MB apart, as in a cache that holds the layers and sequences of a token together: the ranges, and
    with them the room the partial results need, are those of rows that lie together."""
    keep = [10000] + [4000] * 39
    p = pkg.Problem(32, 8, 64, 8, 10, pkg.BF16, [10008] * 40, keep, [0] * 40, 64, 512, [0] * 40, 64, 512)
    packed = pkg.chunkkv_decode_workspace_bytes(p, True)
    p.out_stride_tok = pitch
    assert 0 < packed == pkg.chunkkv_decode_workspace_bytes(p, True) <= 8 << 20


def test_decode_argument_checks(lib):
    p = good(out_base=[0], out_stride_head=848 * 128, out_stride_tok=128)
    cp = p.as_c()
    full, comp = pkg.chunkkv_decode_workspace_bytes(p, False), pkg.chunkkv_decode_workspace_bytes(p, True)
    assert 0 < comp < full                       # fewer key ranges over the 10 % cache
    f = lib.chunkkv_decode_attention
    assert f(None, 0, None, FAKE, FAKE, FAKE, FAKE, None, FAKE, full, None) == 1
    assert f(C.byref(cp), 0, None, None, FAKE, FAKE, FAKE, None, FAKE, full, None) == 1
    assert f(C.byref(cp), 0, None, FAKE, None, FAKE, FAKE, None, FAKE, full, None) == 1
    assert f(C.byref(cp), 0, None, FAKE, FAKE, None, FAKE, None, FAKE, full, None) == 1
    assert f(C.byref(cp), 0, None, FAKE, FAKE, FAKE, None, None, FAKE, full, None) == 1
    assert f(C.byref(cp), 0, None, C.c_void_p(0x1008), FAKE, FAKE, FAKE, None, FAKE, full, None) == 2
    assert f(C.byref(cp), 0, None, FAKE, FAKE, FAKE, FAKE, None, None, full, None) == 4
    assert f(C.byref(cp), 0, None, FAKE, FAKE, FAKE, FAKE, None, FAKE, full - 1, None) == 4
    assert f(C.byref(cp), 1, None, FAKE, FAKE, FAKE, FAKE, None, FAKE, comp - 1, None) == 4
    # the compressed layout needs the output geometry of the problem
    bad_out = good(out_base=[0], out_stride_head=848 * 128, out_stride_tok=100)
    assert pkg.chunkkv_decode_workspace_bytes(bad_out, True) == 0
    assert pkg.chunkkv_decode_workspace_bytes(bad_out, False) == full
    assert f(C.byref(bad_out.as_c()), 1, None, FAKE, FAKE, FAKE, FAKE, None, FAKE, full, None) == 2
    assert pkg.chunkkv_decode_workspace_bytes(good(head_dim=96), False) == 0
