"""The calls this library is used for, as cases that can be timed and checked.

Attention layers under view masks (one short rollout up to a 131072-token
trajectory, forward and backward), an exact packed layer, the LM head's
log-prob forward, backward and weight gradient, the SDCC junction KL, and the
GRPO loss.  Every case goes through the public binding
``paper_2609_00865_amd.mv`` and returns whole outputs; ``exact`` computes the
same results in 64 bits with plain torch."""
from __future__ import annotations

import math

import numpy as np
import torch

DEV = "cuda"
CLIP_LO, CLIP_HI, BETA, ADV_EPS = 0.2, 0.28, 0.04, 1e-6
THETA = 1e6


# --------------------------------------------------------------------------
# the cases
# --------------------------------------------------------------------------
def listed():
    return [
        # One rollout of a few hundred tokens on one small head: the smallest
        # attention call, where launches and latency count.
        {"name": "attn_tiny", "kind": "attn", "workload": "tiny", "n_traj": 1, "length": 512,
         "hq": 1, "hkv": 1, "d": 64, "edits": 2, "restore": False, "backward": True},
        # A handful of short rollouts of uneven length with a memory that
        # offloads and retrieves (keys leave a view and come back), head size 64.
        {"name": "attn_ragged_restore", "kind": "attn", "n_traj": 3, "length": 1451, "hq": 8,
         "hkv": 2, "d": 64, "edits": 4, "restore": True, "backward": True},
        # One ordinary 8192-token trajectory, one layer's forward and backward.
        {"name": "attn_medium", "kind": "attn", "workload": "medium", "n_traj": 1,
         "length": 8192, "hq": 16, "hkv": 4, "d": 128, "edits": 6, "restore": False,
         "backward": True},
        # The training batch: 4 x 32768 tokens, one layer's forward and backward.
        {"name": "attn_batch", "kind": "attn", "workload": "b4x32k", "n_traj": 4,
         "length": 32768, "hq": 28, "hkv": 4, "d": 128, "edits": 16, "restore": False,
         "backward": True},
        # Scoring (forward only) of one very long trajectory, 64/8 heads.
        {"name": "attn_long_score", "kind": "attn", "workload": "long128k", "n_traj": 1,
         "length": 131072, "hq": 64, "hkv": 8, "d": 128, "edits": 40, "restore": False,
         "backward": False},
        # Multi-layer exact scoring of one trajectory: Q, K gathered into the
        # shared-trunk stream and rotated, attention both ways, the gradients
        # rotated back and summed over the copies.
        {"name": "exact_layer", "kind": "layer", "length": 8192, "hq": 28, "hkv": 4, "d": 128,
         "edits": 6, "shared": True, "fused": True},
        # Log-probs and ratios of one assistant turn (a short, odd number of tokens).
        {"name": "score_turn", "kind": "head", "tokens": 201, "hidden": 3584, "vocab": 152064,
         "mode": "score"},
        # One trajectory's log-probs and their gradient into the hidden states
        # (the LM head itself is not trained).
        {"name": "head_trajectory", "kind": "head", "tokens": 4001, "hidden": 3584,
         "vocab": 152064, "mode": "frozen"},
        # A training step of the head of a small model on a few rollouts: the
        # fused GRPO forward, both gradients.
        {"name": "head_train_small", "kind": "head", "tokens": 777, "hidden": 1024,
         "vocab": 32000, "mode": "train"},
        # The training step at full size: 64 rollouts of 512 tokens.
        {"name": "head_train_batch", "kind": "head", "tokens": 32768, "hidden": 3584,
         "vocab": 152064, "mode": "train"},
        # The junction KL of a batch's diverging leaves and its gradient.
        {"name": "sdcc", "kind": "sdcc", "leaves": 1384, "rows": 8192, "hidden": 3584,
         "vocab": 152064},
        # The loss alone, where log-probs come from elsewhere: 64 rollouts.
        {"name": "grpo_loss", "kind": "grpo", "n_traj": 64, "length": 512},
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["attn", "attn", "attn", "layer", "head", "head", "head", "sdcc", "grpo"])
    if kind == "attn":
        n, length = rng.choice([1, 2, 3, 4]), _log(rng, 257, 32768)
        hq, hkv = rng.choice([(1, 1), (8, 2), (16, 4), (28, 4), (32, 8), (12, 12)])
        return {"kind": "attn", "n_traj": n, "length": length, "hq": hq, "hkv": hkv,
                "d": rng.choice([64, 128]), "edits": max(1, length // rng.choice([512, 1024, 2048])),
                "restore": rng.random() < 0.3, "backward": rng.random() < 0.75}
    if kind == "layer":
        hq, hkv = rng.choice([(8, 2), (16, 4), (28, 4)])
        length = _log(rng, 512, 8192)
        return {"kind": "layer", "length": length, "hq": hq, "hkv": hkv,
                "d": rng.choice([64, 128]), "edits": rng.randint(1, 6),
                "shared": rng.random() < 0.5, "fused": rng.random() < 0.6}
    if kind == "head":
        hidden, vocab = rng.choice([(1024, 32000), (2048, 50257), (3584, 152064),
                                    (4096, 128256)])
        return {"kind": "head", "tokens": _log(rng, 48, 8192), "hidden": hidden, "vocab": vocab,
                "mode": rng.choice(["score", "frozen", "train"])}
    if kind == "sdcc":
        hidden, vocab = rng.choice([(1024, 32000), (2048, 50257), (3584, 152064)])
        return {"kind": "sdcc", "leaves": _log(rng, 24, 2048), "rows": _log(rng, 2048, 16384),
                "hidden": hidden, "vocab": vocab}
    return {"kind": "grpo", "n_traj": rng.choice([8, 16, 48, 64, 128]),
            "length": _log(rng, 96, 2048)}


# --------------------------------------------------------------------------
# inputs
# --------------------------------------------------------------------------
def _lib():
    from paper_2609_00865_amd import mv, synth
    return mv, synth


def _gen(seed, salt):
    g = torch.Generator(device=DEV)
    g.manual_seed(1_000_003 * salt + int(seed))
    return g


def _normal(g, *shape):
    return torch.randn(shape, generator=g, device=DEV).to(torch.bfloat16)


def _runs(pos):
    """Sorted positions as half-open spans."""
    pos = np.asarray(pos)
    if not len(pos):
        return ()
    cut = np.flatnonzero(np.diff(pos) != 1) + 1
    return tuple((int(r[0]), int(r[-1]) + 1) for r in np.split(pos, cut))


def _record(rng, synth, begin, length, edits, restore):
    """A rollout's record: each edit evicts a run of the live tokens after the
    prompt (the first sixteenth); a retrieving memory brings some back."""
    lo, alive = max(2, length // 16), np.ones(length, dtype=bool)
    room = np.arange(lo + 1, length)
    junctions = np.sort(rng.choice(room, size=min(edits, len(room)), replace=False))
    out = []
    for J in junctions.tolist():
        live = np.flatnonzero(alive[:J])
        cand, dead = live[live >= lo], np.flatnonzero(~alive[:J])
        n = int(round(rng.uniform(0.1, 0.6) * len(cand)))
        s = int(rng.integers(0, len(cand) - n + 1))
        evict = cand[s:s + n]
        back = ()
        if restore and len(dead) and rng.random() < 0.7:
            m = int(rng.integers(1, min(len(dead), 96) + 1))
            b = int(rng.integers(0, len(dead) - m + 1))
            back = dead[b:b + m]
            alive[back] = True
        alive[evict] = False
        out.append(synth.Edit(begin + J, _runs(evict + begin), (begin + J, begin + J),
                              _runs(np.asarray(back, dtype=int) + begin)))
    return synth.Trajectory(begin, begin + length, tuple(out))


def _trajectories(case, seed):
    _, synth = _lib()
    if case.get("workload"):
        return synth.make_trajectories(case["workload"], int(seed))
    # the lengths are the case's (and a packed layer's whole record, which the
    # length of its stream depends on); the edits are the seed's
    n_traj = case.get("n_traj", 1)
    frac = np.random.default_rng([11, case["length"]]).uniform(0.4, 1.0, size=n_traj)
    rng = np.random.default_rng([17, 0 if case["kind"] == "layer" else int(seed), case["length"]])
    out, b = [], 0
    for t in range(n_traj):
        n = case["length"] if t == 0 else max(8, int(case["length"] * frac[t]))
        out.append(_record(rng, synth, b, n, case["edits"], case.get("restore", False)))
        b += n
    return out


def _attn_inputs(case, seed):
    trajs = _trajectories(case, seed)
    T, g = trajs[-1].end, _gen(seed, 1)
    q = _normal(g, T, case["hq"], case["d"])
    k, v = (_normal(g, T, case["hkv"], case["d"]) for _ in range(2))
    do = _normal(g, T, case["hq"], case["d"])
    return trajs, q, k, v, do


def _layer_inputs(case, seed):
    trajs = _trajectories(case, seed)
    T, g = trajs[-1].end, _gen(seed, 2)
    q = _normal(g, T, case["hq"], case["d"])
    k, v = (_normal(g, T, case["hkv"], case["d"]) for _ in range(2))
    src, _, _ = _stream(trajs, case["shared"])
    do = _normal(g, len(src), case["hq"], case["d"])
    return trajs, q, k, v, do


def _rollouts(T, seed):
    """Offsets of the rollouts that T packed tokens come from (uneven
    lengths), with an exact-match reward and a format bonus."""
    n = max(8, T // 512 // 8 * 8)
    rng = np.random.default_rng([23, int(seed), T])
    ptr = np.concatenate(([0], np.sort(rng.integers(0, T + 1, size=n - 1)), [T]))
    reward = np.array([0.0, 0.2, 1.0])[rng.integers(0, 3, size=n)]
    return (torch.tensor(ptr, dtype=torch.int32, device=DEV),
            torch.tensor(reward, dtype=torch.float32, device=DEV))


def _drift(g, n):
    """log(ratio) of rollout tokens: small, some of them past the clip.  None
    lies within 2e-3 of a clip edge, where one rounding would decide a token."""
    x = 0.1 * torch.randn(n, generator=g, device=DEV)
    for edge in (math.log(1 - CLIP_LO), math.log(1 + CLIP_HI)):
        x = torch.where((x - edge).abs() < 2e-3, torch.zeros_like(x), x)
    return x


def _head_inputs(case, seed):
    g = _gen(seed, 3)
    T, H, V = case["tokens"], case["hidden"], case["vocab"]
    h, w = _normal(g, T, H), torch.empty((V, H), dtype=torch.bfloat16, device=DEV)
    for b in range(0, V, 16384):
        n = min(16384, V - b)
        w[b:b + n] = (0.02 * torch.randn((n, H), generator=g, device=DEV)).to(torch.bfloat16)
    y = torch.randint(0, V, (T,), generator=g, device=DEV)
    # the policy's log-prob now, and the rollout's and the reference's near it
    logp = torch.empty(T, device=DEV)
    for b in range(0, T, 4096):
        e = min(T, b + 4096)
        z = h[b:e] @ w.t()
        m = z.max(1).values.float()
        s = torch.zeros(e - b, device=DEV)
        for c in range(0, V, 16384):
            s += (z[:, c:c + 16384].float() - m[:, None]).exp().sum(1)
        logp[b:e] = (h[b:e].float() * w[y[b:e]].float()).sum(1) - m - s.log()
    off = torch.rand(T, generator=g, device=DEV) < 0.02   # tool output: no target
    old = logp - _drift(g, T)
    ref = logp + 0.05 * torch.randn(T, generator=g, device=DEV)
    mask = ((torch.rand(T, generator=g, device=DEV) < 0.8) & ~off).to(torch.uint8)
    y = torch.where(off, torch.full_like(y, -1), y).to(torch.int32)
    up = torch.randn(T, generator=g, device=DEV)
    ptr, reward = _rollouts(T, seed)
    return {"h": h, "w": w, "y": y, "old": old, "ref": ref, "mask": mask, "up": up, "ptr": ptr,
            "reward": reward}


def _sdcc_inputs(case, seed):
    g = _gen(seed, 4)
    n, R, H, V = case["leaves"], case["rows"], case["hidden"], case["vocab"]
    w = torch.empty((V, H), dtype=torch.bfloat16, device=DEV)
    for b in range(0, V, 16384):
        m = min(16384, V - b)
        w[b:b + m] = (0.02 * torch.randn((m, H), generator=g, device=DEV)).to(torch.bfloat16)
    ht = _normal(g, R, H)
    # the student saw less of the context: a related hidden state
    hs = (0.9 * ht.float() + 0.436 * torch.randn((R, H), generator=g, device=DEV)).to(torch.bfloat16)
    rt = torch.randint(0, R, (n,), generator=g, device=DEV).sort().values.to(torch.int32)
    rs = rt.clone()
    dkl = torch.rand(n, generator=g, device=DEV) * (0.1 / n)
    return {"ht": ht, "hs": hs, "w": w, "rt": rt, "rs": rs, "dkl": dkl}


def _grpo_inputs(case, seed):
    g = _gen(seed, 5)
    T = case["n_traj"] * case["length"]
    rng = np.random.default_rng([29, int(seed), T])
    ptr = np.concatenate(([0], np.sort(rng.integers(0, T + 1, size=case["n_traj"] - 1)), [T]))
    reward = np.array([0.0, 0.2, 1.0])[rng.integers(0, 3, size=case["n_traj"])]
    logp = -2.0 + torch.randn(T, generator=g, device=DEV)
    return {"ptr": torch.tensor(ptr, dtype=torch.int32, device=DEV),
            "reward": torch.tensor(reward, dtype=torch.float32, device=DEV), "logp": logp,
            "old": logp - _drift(g, T),
            "ref": logp + 0.05 * torch.randn(T, generator=g, device=DEV),
            "mask": (torch.rand(T, generator=g, device=DEV) < 0.8).to(torch.uint8)}


def prepare(case, seed):
    mv, _ = _lib()
    kind = case["kind"]
    if kind == "attn":
        trajs, q, k, v, do = _attn_inputs(case, seed)
        mask = mv.ViewMask(trajs).upload()
        s = {"mask": mask, "q": q, "k": k, "v": v, "do": do}
        if case["backward"]:
            s["ws"] = mv.attn_bwd_workspace(mask, q, k)
    elif kind == "layer":
        trajs, q, k, v, do = _layer_inputs(case, seed)
        pack = mv.BranchPack(trajs, shared_trunk=case["shared"]).upload()
        ws = mv.attn_bwd_workspace(pack.mask, do, do[:, :case["hkv"]].contiguous())
        s = {"pack": pack, "q": q, "k": k, "v": v, "do": do, "ws": ws}
    elif kind == "head":
        s = _head_inputs(case, seed)
        if case["mode"] == "train":
            s["ws"] = mv.token_logprob_grpo_workspace(s["h"], s["w"], s["reward"].numel(), 8)
        else:
            s["ws"] = mv.token_logprob_workspace(s["h"], s["w"])
        if case["mode"] != "score":
            s["wsb"] = mv.token_logprob_bwd_workspace(s["h"], s["w"])
    elif kind == "sdcc":
        s = _sdcc_inputs(case, seed)
    else:
        s = _grpo_inputs(case, seed)
    s["case"] = dict(case)
    return s


# --------------------------------------------------------------------------
# one pass
# --------------------------------------------------------------------------
def run(s):
    mv, _ = _lib()
    c = s["case"]
    kind = c["kind"]
    if kind == "attn":
        o, lse = mv.attn_fwd(s["mask"], s["q"], s["k"], s["v"])
        if not c["backward"]:
            return o, lse
        dq, dk, dv = mv.attn_bwd(s["mask"], s["q"], s["k"], s["v"], o, s["do"], lse,
                                 workspace=s["ws"])
        return o, lse, dq, dk, dv
    if kind == "layer":
        p = s["pack"]
        if c["fused"]:
            q, k = mv.pack_rows_rope(p, s["q"], THETA), mv.pack_rows_rope(p, s["k"], THETA)
        else:
            q = mv.pack_rows(p, s["q"])
            k = mv.pack_rows(p, s["k"])
            mv.rope(p, q, THETA, out=q)
            mv.rope(p, k, THETA, out=k)
        v = mv.pack_rows(p, s["v"])
        o, lse = mv.attn_fwd(p.mask, q, k, v)
        dq, dk, dv = mv.attn_bwd(p.mask, q, k, v, o, s["do"], lse, workspace=s["ws"])
        if c["fused"]:
            dq = mv.unpack_rows_sum_rope(p, dq, THETA)
            dk = mv.unpack_rows_sum_rope(p, dk, THETA)
        else:
            mv.rope(p, dq, THETA, inverse=True, out=dq)
            mv.rope(p, dk, THETA, inverse=True, out=dk)
            dq, dk = mv.unpack_rows_sum(p, dq), mv.unpack_rows_sum(p, dk)
        return o, lse, dq, dk, mv.unpack_rows_sum(p, dv)
    if kind == "head":
        if c["mode"] == "train":
            logp, ratio, clipped, lse, adv, dlogp, stats = mv.token_logprob_grpo(
                s["h"], s["w"], s["y"], s["old"], s["ptr"], s["reward"], logp_ref=s["ref"],
                loss_mask=s["mask"], group_size=8, eps_low=CLIP_LO, eps_high=CLIP_HI, beta=BETA,
                adv_eps=ADV_EPS, workspace=s["ws"])
            dh = mv.token_logprob_bwd(s["h"], s["w"], s["y"], lse, dlogp, workspace=s["wsb"])
            dw = mv.token_logprob_dweight(s["h"], s["w"], s["wsb"])
            return logp, ratio, clipped, lse, adv, dlogp, stats, dh, dw
        logp, ratio, clipped, lse = mv.token_logprob(s["h"], s["w"], s["y"], s["old"], CLIP_LO,
                                                     CLIP_HI, workspace=s["ws"])
        if c["mode"] == "score":
            return logp, ratio, clipped, lse
        dh = mv.token_logprob_bwd(s["h"], s["w"], s["y"], lse, s["up"], workspace=s["wsb"])
        return logp, ratio, clipped, lse, dh
    if kind == "sdcc":
        kl, lt, ls = mv.sdcc_kl(s["ht"], s["rt"], s["hs"], s["rs"], s["w"])
        dh = mv.sdcc_kl_bwd(s["ht"], s["rt"], s["hs"], s["rs"], s["w"], lt, ls, s["dkl"])
        return kl, lt, ls, dh
    return mv.grpo_loss(s["ptr"], s["reward"], s["logp"], s["old"], s["ref"], s["mask"],
                        group_size=8, eps_low=CLIP_LO, eps_high=CLIP_HI, beta=BETA,
                        adv_eps=ADV_EPS)


# --------------------------------------------------------------------------
# what a pass cannot do without
# --------------------------------------------------------------------------
def _pairs(trajs):
    """Visible (row, key) pairs: per stretch of rows between two edits, the
    keys alive at its start and the stretch's own rows."""
    return sum(sum(len(keys) * (e - s) + (e - s) * (e - s + 1) // 2 for s, e, keys in _stretches(t))
               for t in trajs)


def work(case):
    kind = case["kind"]
    if kind in ("attn", "layer"):
        trajs = _trajectories(case, 1)
        hq, hkv, d = case["hq"], case["hkv"], case["d"]
        T = trajs[-1].end
        if kind == "layer":
            src, _, segs = _stream(trajs, case["shared"])
            N = len(src)
            pairs = sum(sum(range(len(m) - n + 1, len(m) + 1)) for m, n in segs)
            phys = 2 * T * (hq + 2 * hkv) * d * 2
            return {"bytes": phys + 2 * N * hq * d * 2 + 4 * hq * N, "flops": 14 * d * pairs * hq}
        pairs = _pairs(trajs)
        fwd = (T * (2 * hq + 2 * hkv) * d) * 2 + 4 * hq * T
        if not case["backward"]:
            return {"bytes": fwd, "flops": 4 * d * pairs * hq}
        return {"bytes": fwd + T * (2 * hq + 2 * hkv) * d * 2, "flops": 14 * d * pairs * hq}
    if kind == "head":
        T, H, V = case["tokens"], case["hidden"], case["vocab"]
        gemm = 2 * T * H * V
        n = {"score": 1, "frozen": 3, "train": 4}[case["mode"]]
        nbytes = (T * H + V * H) * 2 + 6 * 4 * T
        if case["mode"] != "score":
            nbytes += T * H * 2
        if case["mode"] == "train":
            nbytes += V * H * 4
        return {"bytes": nbytes, "flops": n * gemm}
    if kind == "sdcc":
        n, H, V = case["leaves"], case["hidden"], case["vocab"]
        return {"bytes": V * H * 2 + 3 * n * H * 2, "flops": 2 * n * H * V * 5}
    T = case["n_traj"] * case["length"]
    return {"bytes": T * (3 * 4 + 1 + 4), "flops": 40 * T}


def tolerance(case):
    # bf16 outputs: one rounding of each (2^-9 at most) on top of bf16
    # operands (probabilities, dS, G) in the products; the loss and the
    # log-probs alone are fp32 sums.
    if case["kind"] == "grpo":
        return {"rel": 1e-5, "max": 1e-3}
    if case["kind"] == "head" and case["mode"] == "score":
        return {"rel": 1e-5, "max": 1e-3}
    return {"rel": 1e-2, "max": 0.4}


# --------------------------------------------------------------------------
# the same results in 64 bits
# --------------------------------------------------------------------------
F64 = torch.float64


def _stretches(traj):
    """(first row, end row, physical keys alive before the first row) of every
    stretch of rows between two edits."""
    alive = np.zeros(traj.end - traj.begin, dtype=bool)
    out, s = [], traj.begin
    for ed in list(traj.edits) + [None]:
        e = traj.end if ed is None else ed.junction
        out.append((s, e, np.flatnonzero(alive) + traj.begin))
        alive[s - traj.begin:e - traj.begin] = True
        if ed is not None:
            for b, x in ed.evict:
                alive[b - traj.begin:x - traj.begin] = False
            for b, x in getattr(ed, "restore", ()):
                alive[b - traj.begin:x - traj.begin] = True
        s = e
    return out


def _stream(trajs, shared):
    """The packed stream of the branch layers: the token and the position of
    every slot, and per layer (slot of each of its tokens, how many of them,
    the last ones, are rows of this layer)."""
    src, pos, segs, n = [], [], [], 0
    for t in trajs:
        prev_tok = prev_slot = None
        for s, e, keys in _stretches(t):
            tok = np.concatenate((keys, np.arange(s, e)))
            same = 0
            if shared and prev_tok is not None:
                m = min(len(tok), len(prev_tok))
                diff = np.flatnonzero(tok[:m] != prev_tok[:m])
                same = int(diff[0]) if len(diff) else m
            new = len(tok) - same
            slot = np.arange(n, n + new)
            if same:
                slot = np.concatenate((prev_slot[:same], slot))
            src.append(tok[same:])
            pos.append(np.arange(same, len(tok)))
            segs.append((slot, new))
            n += new
            prev_tok, prev_slot = tok, slot
    return np.concatenate(src), np.concatenate(pos), segs


def _attend(parts, q, k, v, do, scale):
    """Attention over `parts`, each (rows, keys) index arrays where row i of n
    sees all keys but the last n - 1 - i; gradients when do is given."""
    N, hq, d = q.shape
    hkv = k.shape[1]
    G = hq // hkv
    o, lse = torch.empty((N, hq, d), dtype=F64, device=DEV), torch.empty((hq, N), dtype=F64, device=DEV)
    grads = None
    if do is not None:
        grads = [torch.zeros(x.shape, dtype=F64, device=DEV) for x in (q, k, v)]
    for rows, keys in parts:
        rows, keys = (torch.as_tensor(x, device=DEV) for x in (rows, keys))
        n = len(rows)
        for b in range(0, n, 1024):
            e = min(n, b + 1024)
            r, kk = rows[b:e], keys[:len(keys) - (n - e)]
            R, K = len(r), len(kk)
            hide = torch.ones((R, K), dtype=torch.bool, device=DEV).triu(K - R + 1)
            for h in range(hkv):
                hs = slice(h * G, (h + 1) * G)
                Q = q[r, hs].to(F64).transpose(0, 1).reshape(G * R, d)
                Kh, Vh = k[kk, h].to(F64), v[kk, h].to(F64)
                S = (Q @ Kh.t()) * scale
                S.view(G, R, K).masked_fill_(hide, -math.inf)
                L = torch.logsumexp(S, 1)
                P = S.sub_(L[:, None]).exp_()
                O = P @ Vh
                o[r, hs] = O.view(G, R, d).transpose(0, 1)
                lse[hs][:, r] = L.view(G, R)
                if grads is None:
                    continue
                dO = do[r, hs].to(F64).transpose(0, 1).reshape(G * R, d)
                grads[2][kk, h] += P.t() @ dO
                dS = (dO @ Vh.t()).sub_((dO * O).sum(1, keepdim=True)).mul_(P).mul_(scale)
                grads[0][r, hs] = (dS @ Kh).view(G, R, d).transpose(0, 1)
                grads[1][kk, h] += dS.t() @ Q
    return (o, lse) if grads is None else (o, lse, *grads)


def _rotate(x, pos, sign):
    d = x.shape[-1]
    i = torch.arange(d // 2, dtype=F64, device=DEV)
    a = torch.as_tensor(pos, device=DEV).to(F64)[:, None] * THETA ** (-2 * i / d)
    c, s = a.cos()[:, None], sign * a.sin()[:, None]
    x0, x1 = x[..., :d // 2], x[..., d // 2:]
    return torch.cat((x0 * c - x1 * s, x1 * c + x0 * s), -1)


def _loss64(ptr, reward, logp, old, ref, mask):
    r = reward.to(F64).view(-1, 8)
    adv = ((r - r.mean(1, keepdim=True)) / (r.std(1, keepdim=True) + ADV_EPS)).reshape(-1)
    T = logp.numel()
    who = torch.searchsorted(ptr.long()[1:], torch.arange(T, device=DEV), right=True)
    A, on = adv[who], mask.bool()
    x = logp - old.to(F64)
    rho = x.exp()
    clip = rho.clamp(1 - CLIP_LO, 1 + CLIP_HI)
    active = clip * A < rho * A
    y = ref.to(F64) - logp
    k3 = torch.expm1(y) - y
    n = on.sum().to(F64)
    dlogp = torch.where(on, (torch.where(active, torch.zeros_like(A), -rho * A)
                             - BETA * torch.expm1(y)) / n, torch.zeros_like(A))
    mean = lambda z: torch.where(on, z.to(F64), torch.zeros_like(A)).sum() / n  # noqa: E731
    stats = torch.stack([mean(-torch.minimum(rho * A, clip * A) + BETA * k3), mean(x.abs()),
                         mean(active & (rho < 1 - CLIP_LO)), mean(active & (rho > 1 + CLIP_HI)),
                         mean(k3), mean(rho), n, adv.abs().mean()])
    return adv, dlogp, stats


def _head64(case, seed):
    s = _head_inputs(case, seed)
    T, V = case["tokens"], case["vocab"]
    w, y = s["w"].to(F64), s["y"].long()
    on = y >= 0
    at = y.clamp(min=0)
    lse, tl = (torch.empty(T, dtype=F64, device=DEV) for _ in range(2))
    step = 2048
    for b in range(0, T, step):
        z = s["h"][b:b + step].to(F64) @ w.t()
        lse[b:b + step] = torch.logsumexp(z, 1)
        tl[b:b + step] = z.gather(1, at[b:b + step, None])[:, 0]
    zero = torch.zeros_like(lse)
    logp = torch.where(on, tl - lse, zero)
    ratio = torch.where(on, (logp - s["old"].to(F64)).exp(), zero + 1)
    out = [logp, ratio, ratio.clamp(1 - CLIP_LO, 1 + CLIP_HI), lse]
    if case["mode"] == "score":
        return tuple(out)
    up = s["up"].to(F64)
    if case["mode"] == "train":
        adv, up, stats = _loss64(s["ptr"], s["reward"], logp, s["old"], s["ref"], s["mask"])
        out += [adv, up, stats]
    up = torch.where(on, up, zero)
    dh = torch.empty((T, w.shape[1]), dtype=F64, device=DEV)
    dw = torch.zeros_like(w) if case["mode"] == "train" else None
    for b in range(0, T, step):
        h = s["h"][b:b + step].to(F64)
        z = (h @ w.t()).sub_(lse[b:b + step, None]).exp_().mul_(-up[b:b + step, None])
        z.scatter_add_(1, at[b:b + step, None], up[b:b + step, None])
        dh[b:b + step] = z @ w
        if dw is not None:
            dw.addmm_(z.t(), h)
    return tuple(out + [dh] + ([dw] if dw is not None else []))


def exact(case, seed):
    kind = case["kind"]
    scale = 1.0 / math.sqrt(case["d"]) if "d" in case else None
    if kind == "attn":
        trajs, q, k, v, do = _attn_inputs(case, seed)
        parts = [(np.arange(s, e), np.concatenate((keys, np.arange(s, e))))
                 for t in trajs for s, e, keys in _stretches(t)]
        return _attend(parts, q, k, v, do if case["backward"] else None, scale)
    if kind == "layer":
        trajs, q, k, v, do = _layer_inputs(case, seed)
        src, pos, segs = _stream(trajs, case["shared"])
        at = torch.as_tensor(src, device=DEV)
        parts = [(m[len(m) - n:], m) for m, n in segs]
        Q, K = (_rotate(x[at].to(F64), pos, 1.0) for x in (q, k))
        o, lse, dq, dk, dv = _attend(parts, Q, K, v[at], do, scale)
        back = []
        for g, rotated in ((dq, True), (dk, True), (dv, False)):
            g = _rotate(g, pos, -1.0) if rotated else g
            back.append(torch.zeros((q.shape[0],) + g.shape[1:], dtype=F64,
                                    device=DEV).index_add_(0, at, g))
        return (o, lse, *back)
    if kind == "head":
        return _head64(case, seed)
    if kind == "sdcc":
        s = _sdcc_inputs(case, seed)
        w = s["w"].to(F64)
        out = [[], [], [], []]
        for b in range(0, case["leaves"], 512):
            zt = s["ht"][s["rt"][b:b + 512].long()].to(F64) @ w.t()
            zs = s["hs"][s["rs"][b:b + 512].long()].to(F64) @ w.t()
            lt, ls = torch.logsumexp(zt, 1), torch.logsumexp(zs, 1)
            p, q = (zt - lt[:, None]).exp(), (zs - ls[:, None]).exp()
            kl = (p * (zt - zs)).sum(1) - lt + ls
            dh = ((q - p) * s["dkl"][b:b + 512, None].to(F64)) @ w
            for x, y in zip(out, (kl, lt, ls, dh)):
                x.append(y)
        return tuple(torch.cat(x) for x in out)
    s = _grpo_inputs(case, seed)
    return _loss64(s["ptr"], s["reward"], s["logp"].to(F64), s["old"], s["ref"], s["mask"])
