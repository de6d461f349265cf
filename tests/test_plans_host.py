"""Host-only checks of how the passes are divided and what their workspaces
hold: C++ programs that include the plan headers, compiled here."""
import ctypes
import os
import subprocess

import pytest

from paper_2609_00865_amd import build, mv, synth

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


def _attn_ws(trajs, hq, hkv, d):
    m = mv.ViewMask(trajs)
    shape = mv.AttnShape(m.total_tokens, hq, hkv, d, 0.0)
    return m, int(mv.mv_attn_bwd_workspace_bytes(m.handle, ctypes.byref(shape)))


def test_short_rollouts_keep_the_work_items():
    """Batches whose items fill the CUs evenly: no partial tiles, so the
    workspace is the rows' statistics alone (dK/dV in shares: 1142 against 991
    us at the first)."""
    for n, length, hq, hkv in ((16, 2048, 28, 4), (32, 1024, 28, 4), (8, 1024, 32, 8)):
        T = n * length
        trajs = [synth.Trajectory(i * length, (i + 1) * length, ()) for i in range(n)]
        m, ws = _attn_ws(trajs, hq, hkv, 128)
        assert m.stats()["bwd_partial_slots"] == 0
        assert ws == 2 * hq * T * 4 + 256, (n, length, hq, hkv)
    # one such rollout leaves CUs idle
    assert _attn_ws([synth.Trajectory(0, 2048, ())], 32, 8, 128)[1] > 2 * 32 * 2048 * 4 + 256
