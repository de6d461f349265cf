"""Host-only checks of how the passes are divided and what their workspaces
hold: C++ programs that include the plan headers, compiled here."""
import os
import subprocess

import pytest

from paper_2609_00865_amd import build

HERE = os.path.dirname(os.path.abspath(__file__))


def _run(tmp_path, name, args=(), sources=()):
    exe = str(tmp_path / name)
    subprocess.run([build.HIPCC, "-O2", "-std=c++17", "-I" + os.path.join(build.ROOT, "include"),
                    "-I" + build.CSRC, os.path.join(HERE, name + ".cpp"),
                    *(os.path.join(build.CSRC, s) for s in sources), "-o", exe], check=True)
    r = subprocess.run([exe, *map(str, args)], capture_output=True, text=True)
    assert r.returncode == 0, r.stdout + r.stderr
    return [tuple(map(int, line.split())) for line in r.stdout.splitlines()]


def test_dkdv_shares_cover_every_step_once(tmp_path):
    """Random masks and head counts: every step in one run, partial tiles
    numbered in order and summed once, workspaces as large as what is written
    and within the static scratch where the work items' are."""
    long_ones = [(8192, 1, 16, 4, 128), (3000, 4, 32, 8, 128), (2048, 1, 32, 8, 128)]
    got = _run(tmp_path, "bwd_plan_check", [x for s in long_ones for x in s], ["mask.cpp"])
    # the partial tiles of 256 shares fit the static scratch (8192 tokens: of
    # two for every share, 251 would)
    assert [g[0] for g in got] == [256] * 3
    assert all(g[1] < 2 * 256 for g in got)
