"""Arithmetic of the scoring kernels (csrc/score_plan.h), on the host."""
import os
import random
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


@pytest.fixture(scope="module")
def ask(tmp_path_factory):
    exe = str(tmp_path_factory.mktemp("plan") / "score_plan")
    subprocess.run(["g++", "-std=c++17", "-O1", "-Wall", "-Werror", "-I", os.path.join(ROOT, "paper_2502_00299_amd", "csrc"),
                    "-o", exe, os.path.join(ROOT, "tests", "score_plan_main.cpp")], check=True)
    return lambda lines, *mode: subprocess.run([exe, *mode], input="\n".join(lines), capture_output=True, text=True, check=True, timeout=120).stdout.splitlines()


def test_ring_loads_read_prefix_rows_only(ask):
    """Rows next to each other and interleaved, one row, period edges, and the longest heads 32-bit offsets reach."""
    cases = [(p, pitch) for p in (0, 1, 31, 159, 160, 161, 640, 1281, 20011) for pitch in (256, 512, 2048, 2064)]
    cases += [(8388351, 256), (2047744, 1024), (255, 1 << 22), (161, 1 << 22)]
    lines = [f"{p} {pitch} 256" for p, pitch in cases]
    assert dict(zip(lines, ask(lines))) == {line: "ok" for line in lines}


def test_super_tiles_do_not_grow_as_they_are_cut(ask):
    """A short launch halves the keys of its super-tiles to get more of them: whole chunks, of at most that many keys or one."""
    lines = [f"{keys} {chunk}" for chunk in range(1, 257) for keys in (256, 128, 64)]
    got = list(map(int, ask(lines, "stride")))
    for chunk in range(1, 257):
        strides = got[3 * chunk - 3:3 * chunk]
        assert strides == sorted(strides, reverse=True), chunk
        for keys, n in zip((256, 128, 64), strides):
            assert n % chunk == 0 and (n == chunk or keys - chunk < n <= keys), (keys, chunk)


def test_workgroups_fill_whole_rounds(ask):
    """Units per workgroup: within the limits, the least ones for launches of many rounds, and never a longer launch by the rule's own
    measure than one unit or one round would be."""
    rng = random.Random(7)
    cases = [(1, 1, [1]), (1, 0, [0, 0]), (3, 10, [10]), (1, 500, [500]), (4, 4096, [4096] * 16), (1, 513, [513]), (1, 257, [257, 1])]
    cases += [(rng.choice([1, 2, 9]), None, [rng.randrange(0, 2000) for _ in range(rng.randrange(1, 17))]) for _ in range(200)]
    lines, want = [], []
    for lo, hi, units in cases:
        hi, slots, least, rounds, half, start = max(units) if hi is None else hi, rng.choice([256, 512]), rng.choice([-3, 2]), rng.choice([4, 8]), 0.7, rng.choice([0.5, 2.0, 6.0])
        lines.append(f"{lo} {hi} {slots} {least} {rounds} {half} {start} {len(units)} " + " ".join(map(str, units)))
        want.append((lo, hi, slots, least, rounds, half, start, units))
    for line, (lo, hi, slots, least, rounds, half, start, units) in zip(ask(lines, "units"), want):
        def wgs(t):
            return sum(-(-u // t) for u in units)

        def cost(t):
            full, rest = divmod(wgs(t), slots)
            return t * (full + (0 if rest == 0 else half if 2 * rest <= slots else 1)) + start * (full + (rest != 0)) + 0.1 * t
        t, n = map(int, line.split())
        assert lo <= t <= max(lo, hi) and n == wgs(t)
        if lo >= hi or wgs(lo) > rounds * slots:
            assert t == lo
        else:
            for r in range(max(1, least), rounds + 1):
                fits = next((x for x in range(lo, hi + 1) if wgs(x) <= r * slots), hi)
                assert cost(t) <= cost(fits) * (1 + 1e-9)
