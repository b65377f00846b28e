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
    return lambda lines: subprocess.run([exe], input="\n".join(lines), capture_output=True, text=True, check=True, timeout=120).stdout.splitlines()


def test_ring_loads_read_prefix_rows_only(ask):
    """Rows next to each other and interleaved, one row, period edges, and the longest heads 32-bit offsets reach."""
    cases = [(p, pitch) for p in (0, 1, 31, 159, 160, 161, 640, 1281, 20011) for pitch in (256, 512, 2048, 2064)]
    cases += [(8388351, 256), (2047744, 1024), (255, 1 << 22), (161, 1 << 22)]
    lines = [f"{p} {pitch} 256" for p, pitch in cases]
    assert dict(zip(lines, ask(lines))) == {line: "ok" for line in lines}
