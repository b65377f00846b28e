"""How decode attention cuts a batch into key ranges (csrc/decode_plan.h), on the host: every row is in one range, the
partial results fit the workspace, whose size is that of an even cut."""
import os
import random
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
F32, BF16, F16 = 0, 1, 2


@pytest.fixture(scope="module")
def cut(tmp_path_factory):
    """cut(problems) -> [(workspace bytes, [(n_split, [(rows, ranges, first range), ...]) per launch])]"""
    exe = str(tmp_path_factory.mktemp("plan") / "decode_plan")
    subprocess.run(["g++", "-std=c++17", "-O1", "-Wall", "-Werror", "-I", os.path.join(ROOT, "include"), "-I",
                    os.path.join(ROOT, "paper_2502_00299_amd", "csrc"), "-o", exe, os.path.join(ROOT, "tests", "decode_plan_main.cpp")], check=True)

    def ask(problems, *mode):
        text = "".join(f"{dt} {hq} {hkv} {d} {pitch} {len(n)} {' '.join(map(str, n))}\n" for dt, hq, hkv, d, pitch, n in problems)
        out = subprocess.run([exe, *mode], input=text, capture_output=True, text=True, check=True, timeout=120).stdout.splitlines()
        if mode:
            return [list(map(int, line.split())) for line in out]
        answers = []
        for line in out:
            total, *launches = line.split(" | ")
            answers.append((int(total), [(int(x.split()[0]), [tuple(map(int, y.split(":"))) for y in x.split()[1:]]) for x in launches]))
        assert len(answers) == len(problems)
        return answers
    return ask


def align(x):
    return (x + 255) // 256 * 256


def workgroups_per_range(dt, hq, hkv):
    """kv-heads times the batches of query heads that one workgroup serves, as the size of the workspace counts them"""
    g = hq // hkv
    G = 8 if dt != F32 and g > 4 else 4 if g > 2 else g
    return hkv * -(-g // G)


def even_results(dt, hq, hkv, d, pitch, n):
    """Partial results of about 1024 ranges of one length, at least 256 rows: what the workspace has always held."""
    launches = -(-len(n) // 16)
    rows = -(-(sum(n) * workgroups_per_range(dt, hq, hkv) // launches) // 1024)
    rows = 256 if rows < 256 else -(-rows // 128) * 128
    return len(n) * hq * -(-max(n) // rows)


def drawn(rng):
    hkv, g, d = rng.choice([1, 2, 4, 8, 16, 32, 64]), rng.choice([1, 2, 3, 4, 7, 8, 9]), rng.choice([64, 128])
    top = int(10 ** rng.uniform(0, 5.1)) + 1
    batch = rng.choice([1, 1, 2, 5, 8, 16, 17, 40])
    n = [max(1, int(top * rng.uniform(0.05, 1))) if rng.random() < 0.7 else rng.randint(1, 300) for _ in range(batch)]
    return rng.choice([F32, BF16, F16]), hkv * g, hkv, d, max(hkv * d, rng.choice([64, 32768, 1 << 21, 1 << 25, 1 << 26])), n


def test_every_row_is_in_one_range_and_the_results_fit(cut):
    rng = random.Random(5)
    problems = [(BF16, 32, 8, 128, 1024, [848]), (BF16, 32, 8, 128, 1024, [512]), (BF16, 32, 8, 128, 1024, [513]),
                (F16, 8, 1, 128, 1024, [30848] + [33] * 15)] + [drawn(rng) for _ in range(3000)]
    for prob, (total, launches) in zip(problems, cut(problems)):
        dt, hq, hkv, d, pitch, n = prob
        results = even_results(*prob)
        assert total == align(results * 8) + align(results * d * 4), prob
        b = 0
        for n_split, seqs in launches:
            places = 0
            for rows, ranges, first in seqs:
                assert rows > 0 and (ranges - 1) * rows < n[b] <= ranges * rows, prob
                assert first == places, prob
                places += ranges
                b += 1
            assert n_split == max(x[1] for x in seqs)
            assert places * hq <= results, prob
        assert b == len(n)


@pytest.mark.parametrize("hkv,n,least", [(32, [4096] + [64] * 15, 6), (16, [4096] + [128] * 15, 8), (15, [4096] + [64] * 15, 8),
                                         (64, [131072] + [300] * 15, 12), (16, [8111] * 3 + [400] * 13, 4)])
def test_short_sequences_do_not_keep_long_ones_from_being_cut(cut, hkv, n, least):
    (_, [(_, seqs)]), = cut([(BF16, hkv, hkv, 128, hkv * 128, n)])
    assert seqs[0][1] >= least


def test_no_range_is_far_longer_than_a_cu_s_share(cut):
    """Twice the rows of the whole launch over 256 CUs at most, however uneven the batch, or the few hundred rows a range has anyway."""
    rng = random.Random(6)
    problems = [p for p in (drawn(rng) for _ in range(4000)) if p[0] != F32 and p[4] < 1 << 25 and len(p[5]) <= 16]
    for prob, (_, [(_, seqs)]) in zip(problems, cut(problems)):
        dt, hq, hkv, d, pitch, n = prob
        share = -(-sum(n) * workgroups_per_range(dt, hq, hkv) // 256)
        assert max(rows for rows, _, _ in seqs) <= max(2 * share + 31, 512), prob


def test_fp32_wavefronts_count_workgroups_that_have_rows(cut):
    """16, 8 or 4 wavefronts by the workgroups with rows: a long sequence among short ones does not count for all of them."""
    rng = random.Random(8)
    problems = [(F32, 16, 4, 64, 256, [8000] + [300] * 7), (F32, 8, 4, 128, 512, [8000] + [300] * 7), (F32, 16, 4, 128, 512, [8000] + [300] * 7)]
    problems += [(F32, *p[1:]) for p in (drawn(rng) for _ in range(2000)) if p[4] < 1 << 25]
    answers = cut(problems, "waves")
    assert answers[:3] == [[16], [16], [8]]
    seen = set()
    for prob, launches, (_, cuts) in zip(problems, answers, cut(problems)):
        dt, hq, hkv, d, pitch, n = prob
        for waves, (_, seqs) in zip(launches, cuts):
            wgs = sum(ranges for _, ranges, _ in seqs) * workgroups_per_range(dt, hq, hkv)
            four_heads = hq // hkv > 2
            want = 16 if wgs <= 256 and not (d == 128 and four_heads) else 8 if d == 128 and wgs <= 512 else 4
            assert waves == want, prob
            seen.add((d, waves))
    assert seen == {(64, 16), (64, 4), (128, 16), (128, 8), (128, 4)}
