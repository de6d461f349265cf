"""Host-only checks of how the passes are divided and what their workspaces
hold: C++ programs that include the plan headers, compiled here."""
import ctypes
import os
import subprocess

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


def test_lm_head_partials_fit_their_room(tmp_path):
    """For every token count the dH partials fit what the workspace has for
    them, and that never shrinks as tokens grow."""
    _run(tmp_path, "lm_plan_check")


LM_SHAPES = [(1024, 32000), (3584, 152064), (4096, 128256), (64, 1000)]


def _lm_sizes(n, H, V, n_traj=8):
    s = mv.LogprobShape(n, H, V, 0.2, 0.2)
    g = mv.GrpoShape(n, n_traj, 8, 0.2, 0.2, 0.0, 1e-6)
    k = mv.KLShape(n, H, V, 16384, 16384)
    ref = ctypes.byref
    return (mv.mv_token_logprob_workspace_bytes(ref(s)),
            mv.mv_token_logprob_grpo_workspace_bytes(ref(s), ref(g)),
            mv.mv_token_logprob_bwd_workspace_bytes(ref(s)),
            mv.mv_sdcc_kl_workspace_bytes(ref(k)), mv.mv_sdcc_kl_bwd_workspace_bytes(ref(k)))


def test_lm_head_workspaces_never_shrink():
    for H, V in LM_SHAPES:
        before = (0,) * 5
        for n in sorted({*range(1, 3400, 3), *range(3071, 3075), *range(256, 33000, 256),
                         *range(257, 33000, 256)}):
            now = _lm_sizes(n, H, V)
            assert all(a >= b for a, b in zip(now, before)), (n, H, V, now, before)
            before = now


def test_lm_head_backward_reserves_what_it_uses():
    """Where dH is not split there is no room for partials: G and W^T alone
    (with room for 32 splits whatever the count, 512 MiB more)."""
    vp = 152064 // 256 * 256
    both = 2 * vp * (32768 + 3584)
    assert _lm_sizes(32768, 3584, 152064)[2] <= both + 4096
    # three fp32 partials of the 1384 leaves' dh, beside G
    assert _lm_sizes(1384, 3584, 152064)[4] <= 2 * vp * 1536 + 3 * 4 * 1384 * 3584 + 65536
