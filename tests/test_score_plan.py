"""Arithmetic of the scoring kernels (csrc/score_plan.h), on the host."""
import os
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
