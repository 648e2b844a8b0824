"""Performance cases: the calls a serving engine makes, over their real ranges.

A case is one pass through a public entry point of ``paper_2608_07855_amd``
(or through the chain of them that one commit makes) on seeded inputs held in
GPU memory.  Keys, values and queries are N(0, 1) bf16 with 1% heavy-hitter
keys scaled by 4, the distribution of the repository's synthetic workloads;
events alternate reasoning, tool call and observation, and the tool-call and
observation events are cut into pages.

Kinds:

  measure     ckv_measure_page_effects, one layer and one window: what every
              commit runs before the tool call ("pre": the cache prefix, R
              only) and after the observation ("post": R, o, lse), with the
              token mass where the next checkpoint scores tokens with it;
              without pages it is the checkpoint's base score alone
  recorded    ckv_measure_recorded: engines that keep the window's outputs
  batch       ckv_measure_page_effects_batch: the commit of every layer of a
              short-budget cache in one call
  joint       ckv_joint_test: the greedy retirement test of one commit
  checkpoint  ckv_select_and_compact: the compression checkpoint of a stack
  commit      pre and post measurement, classification, joint test and the
              layer's checkpoint, in the order an engine calls them
"""
import math

import numpy as np
import torch

import paper_2608_07855_amd as P

DEV = "cuda"
OBS = 128          # tokens of the last observation
_CTX = []          # one context per process, as a serving worker holds it


def _context():
    if not _CTX:
        _CTX.append(P.Context(0))
    return _CTX[0]


def _case(name, kind, hq, hkv, d, S, W, G, **more):
    c = dict(name=name, kind=kind, hq=hq, hkv=hkv, d=d, S=S, W=W, G=G)
    c.update(more)
    return c


def listed():
    return [
        # the smallest call: a 2K cache of a small model, everything asked for
        _case("measure_tiny", "measure", 4, 1, 64, 2048, 32, 16, phase="post", scan=0, head=False, mass=True,
              paged=False),
        # the paper's operating point: budget 4096 plus a checkpoint interval, W 8, G 16, the
        # 64 newest pages of one layer at a commit
        _case("measure_paper", "measure", 40, 8, 128, 4224, 8, 16, phase="pre", scan=64, head=False, mass=False,
              paged=False),
        # the pre-commit window of a 32K layer (a ragged prefix of the cache)
        _case("measure_q8b_pre", "measure", 32, 8, 128, 32768, 64, 32, phase="pre", scan=0, head=False, mass=False,
              paged=False),
        # the post-commit window of the same layer kept as a paged pool, with every output
        _case("measure_q8b_paged", "measure", 32, 8, 128, 32768, 64, 32, phase="post", scan=0, head=True, mass=True,
              paged=True),
        # a long context: 128K tokens, 64 query heads, 128-row windows, 64-token pages
        _case("measure_q32b", "measure", 64, 8, 128, 131072, 128, 64, phase="post", scan=0, head=False, mass=False,
              paged=False),
        # page effects and token mass from the outputs an engine recorded
        _case("recorded_q8b", "recorded", 32, 8, 128, 32768, 64, 32, scan=0, mass=True),
        # the commit of 40 layers at the paper's operating point in one call
        _case("batch_paper", "batch", 40, 8, 128, 4224, 8, 16, scan=64, layers=40),
        # the base score of an agent's checkpoint: token mass of one layer, no pages
        _case("score_agent", "measure", 32, 8, 128, 16512, 64, 32, phase="post", scan=-1, head=False, mass=True,
              paged=False),
        # the joint test of a commit that retires many pages
        _case("joint_stress", "joint", 32, 8, 128, 32768, 64, 32, scan=0, forced=0.30),
        # an agent's periodic checkpoint: 36 layers, 128 tokens over the budget
        _case("checkpoint_agent", "checkpoint", 32, 8, 128, 16512, 64, 32, layers=36, seqs=1, budget=16384),
        # a batched checkpoint of two long sequences
        _case("checkpoint_stack", "checkpoint", 32, 8, 128, 65536, 64, 32, layers=36, seqs=2, budget=16384),
        # one commit of a 32K layer from end to end
        _case("commit_q8b", "commit", 32, 8, 128, 32768, 64, 32, scan=0, forced=0.05, budget=8192),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["measure", "measure", "measure", "recorded", "batch", "joint", "checkpoint", "commit"])
    hq, hkv, d = rng.choice([(4, 1, 64), (32, 8, 128), (40, 8, 128), (64, 8, 128), (16, 4, 64)])
    W = _log_int(rng, 8, 128)
    G = rng.choice([16, 32, 64, rng.randint(9, 63)])
    top = {"measure": 131072, "recorded": 65536, "batch": 8192, "joint": 40000, "checkpoint": 65536,
           "commit": 65536}[kind]
    low = {"measure": 600, "recorded": 2048, "batch": 1024, "joint": 4096, "checkpoint": 2048, "commit": 4096}[kind]
    S = _log_int(rng, low, top)
    c = dict(kind=kind, hq=hq, hkv=hkv, d=d, S=S, W=W, G=G)
    if kind == "measure":
        c.update(phase=rng.choice(["pre", "post"]), scan=rng.choice([0, 0, 64, -1]), head=rng.random() < 0.3,
                 mass=rng.random() < 0.4, paged=rng.random() < 0.3)
        c["mass"] = c["mass"] or c["scan"] < 0
    elif kind == "recorded":
        c.update(scan=rng.choice([0, 64]), mass=rng.random() < 0.6)
    elif kind == "batch":
        c.update(scan=rng.choice([0, 64]), layers=rng.randint(2, 48))
        c["W"] = min(W, 64)
    elif kind == "joint":
        c.update(scan=0, forced=round(rng.uniform(0.02, 0.3), 3))
        c["W"], c["G"] = min(W, 64), max(G, 24)
    elif kind == "checkpoint":
        c.update(layers=_log_int(rng, 1, 40), seqs=rng.randint(1, 2))
        c["budget"] = max(256, int(S * rng.uniform(0.2, 0.98)))
    else:
        c.update(scan=0, forced=round(rng.uniform(0.02, 0.1), 3))
        c["W"], c["G"] = min(W, 64), max(G, 24)
        c["budget"] = max(512, int(S * rng.uniform(0.2, 0.6)))
    return c


# ------------------------------------------------------------------ inputs

def _layout(c, rng):
    """Pages of the tool-call and observation events before the post window,
    the committed call's own pages, and the length of the pre-commit prefix."""
    S, W, G = c["S"], c["W"], c["G"]
    lo, hi = (32, 256) if S <= 6000 else (64, 2048)
    # the events' lengths belong to the sizes, their order to the seed, so that every
    # seed has as many pages
    size_rng = np.random.default_rng([S, W, G])
    head = S - W - OBS - max(int(size_rng.integers(lo, min(hi, 256) + 1)), W)
    lens = []
    while sum(lens) < head:
        lens.append(min(int(size_rng.integers(lo, hi + 1)), head - sum(lens)))
    events = [(n, k % 3 != 0) for k, n in enumerate(lens)]
    start, length, t = [], [], 0
    for i in rng.permutation(len(events)):
        n, paged = events[i]
        if paged:
            for off in range(0, n, G):
                start.append(t + off)
                length.append(min(G, n - off))
        t += n
    n_before = len(start)
    s_pre = S - W - OBS
    for off in range(0, s_pre - head, G):
        start.append(head + off)
        length.append(min(G, s_pre - head - off))
    pend = len(start) - n_before
    scan = c.get("scan", 0)
    if scan > 0:
        start, length = start[-scan:], length[-scan:]
    elif scan < 0:
        start, length = [], []
    return np.array(start, np.int32), np.array(length, np.int32), min(pend, len(start)), s_pre


def _normal(gen, shape):
    return torch.randn(shape, generator=gen, device=DEV, dtype=torch.bfloat16)


def _layer(c, gen, heavy):
    k, v = _normal(gen, (c["hkv"], c["S"], c["d"])), _normal(gen, (c["hkv"], c["S"], c["d"]))
    k[:, heavy] *= 4
    return k, v


def _inputs(c, seed):
    """Everything the call reads, from the seed alone, in plain torch."""
    rng = np.random.default_rng([260807855, seed])
    gen = torch.Generator(device=DEV)
    gen.manual_seed(seed)
    S, W, d = c["S"], c["W"], c["d"]
    x = dict(rng=rng, gen=gen)
    x["start"], x["len"], x["pend"], x["s_pre"] = _layout(c, rng)
    heavy = torch.from_numpy(rng.choice(S, max(1, S // 100), replace=False)).to(DEV)
    pos = torch.arange(S, dtype=torch.int32, device=DEV)
    x["pos"] = pos
    x["qpos_pre"] = pos[x["s_pre"] - W:x["s_pre"]].clone()
    x["qpos_post"] = pos[S - W:].clone()
    if c["kind"] == "checkpoint":
        L, n = c["layers"], c["seqs"]
        shape = (n, L, c["hkv"], S, d)
        x["k"], x["v"] = torch.empty(shape, dtype=torch.bfloat16, device=DEV), torch.empty(shape, dtype=torch.bfloat16, device=DEV)
        for t in (x["k"], x["v"]):
            for s in range(n):
                for i in range(L):
                    t[s, i] = _normal(gen, shape[2:])
        # window masses: most tokens near 1/S, some far above
        x["score"] = torch.exp(torch.randn((n, S), generator=gen, device=DEV) * 1.5) / S
        x["pos2"] = pos[None].repeat(n, 1).contiguous()
        x["r_pre"] = torch.rand((n, max(1, x["pend"])), generator=gen, device=DEV)
        return x
    if c["kind"] == "batch":
        x["layers"] = [(*_layer(c, gen, heavy), _normal(gen, (c["hq"], W, d))) for _ in range(c["layers"])]
        return x
    x["k"], x["v"] = _layer(c, gen, heavy)
    x["q_pre"], x["q_post"] = _normal(gen, (c["hq"], W, d)), _normal(gen, (c["hq"], W, d))
    if c["kind"] in ("joint", "commit"):
        # a share of the pages loses its attention mass between the two windows: their
        # logits carry +ln 3 in the pre window and ln 0.2 in the post window
        n = len(x["start"])
        forced = np.sort(rng.choice(n, max(1, round(c["forced"] * n)), replace=False))
        tok = torch.from_numpy(np.concatenate([np.arange(x["start"][j], x["start"][j] + x["len"][j]) for j in forced])).to(DEV)
        x["k"][:, :, 0] = 0
        x["k"][:, tok, 0] = math.sqrt(d)
        x["q_pre"][:, :, 0], x["q_post"][:, :, 0] = math.log(3.0), math.log(0.2)
        x["forced"] = forced
    if c["kind"] == "commit":
        x["score"] = torch.exp(torch.randn((1, S), generator=gen, device=DEV) * 1.5) / S
    return x


# -------------------------------------------------- the same in plain torch

def _attend(k, v, q, pos, qpos, start, length, dtype, mass=True, residual_of=None):
    """Window outputs, log-sum-exp, page effects per head and token mass of one
    layer, by the definition; with ``residual_of`` (page indices) the pages'
    residuals u - A o, masses A and the output norms per row instead of the effects."""
    hkv, S, d = k.shape
    hq, W, _ = q.shape
    grp, n = hq // hkv, len(start)
    sc = 1.0 / math.sqrt(d)
    lens = torch.from_numpy(length.astype(np.int64)).to(k.device)
    G = int(length.max()) if n else 1
    idx = torch.from_numpy(start.astype(np.int64)).to(k.device)[:, None] + torch.arange(G, device=k.device)
    ok = torch.arange(G, device=k.device)[None] < lens[:, None]
    idx = torch.where(ok, idx, 0)
    hide = pos[None].long() > qpos[:, None].long()                 # [W, S]
    o, lse = torch.empty((hq, W, d), dtype=dtype, device=k.device), torch.empty((hq, W), dtype=dtype, device=k.device)
    m = torch.zeros(S, dtype=dtype, device=k.device)
    R = torch.empty((n, hq), dtype=dtype, device=k.device)
    res = []
    for g in range(hkv):
        kg, vg, qg = k[g].to(dtype), v[g].to(dtype), q[g * grp:(g + 1) * grp].to(dtype).reshape(grp * W, d)
        a = ((qg @ kg.T) * sc).masked_fill_(hide.repeat(grp, 1), -math.inf)
        l = torch.logsumexp(a, 1)
        a = a.sub_(l[:, None]).exp_()
        og = a @ vg
        o[g * grp:(g + 1) * grp], lse[g * grp:(g + 1) * grp] = og.view(grp, W, d), l.view(grp, W)
        if mass:
            m = torch.maximum(m, a.view(grp, W, S).sum(1).amax(0))
        pick = range(0, n, 256) if residual_of is None else [None]
        for b in pick:
            sel = slice(b, b + 256) if residual_of is None else residual_of
            ii, kk = idx[sel], ok[sel]
            ap = a[:, ii].masked_fill_(~kk[None], 0.0).transpose(0, 1).contiguous()        # [m, rows, G]
            A = ap.sum(2)
            r = torch.matmul(ap, vg[ii].contiguous()) - A[:, :, None] * og[None]
            if residual_of is None:
                t = r.norm(dim=2) / ((1 - A) * og.norm(dim=1)[None])
                R[sel, g * grp:(g + 1) * grp] = t.view(-1, grp, W).amax(2)
            else:
                res.append((r, A, og.norm(dim=1)))
            del ap, r
        del a
    return dict(o=o, lse=lse, mass=m, R_head=R, residuals=res)


def _effects(c, x, phase, dtype, **kw):
    S = x["s_pre"] if phase == "pre" else c["S"]
    q, qp = (x["q_pre"], x["qpos_pre"]) if phase == "pre" else (x["q_post"], x["qpos_post"])
    return _attend(x["k"][:, :S], x["v"][:, :S], q, x["pos"][:S], qp, x["start"], x["len"], dtype, **kw)


# ------------------------------------------------------------------ prepare

def _view(c, x, phase, paged=False):
    S = x["s_pre"] if phase == "pre" else c["S"]
    if not paged:
        return P.kv_view(x["k"], x["v"], x["pos"], S)
    rows = c["S"] + c["S"] // 2
    slot = torch.randperm(rows, generator=x["gen"], device=DEV)[:c["S"]]
    kp = torch.zeros((c["hkv"], rows, c["d"]), dtype=torch.bfloat16, device=DEV)
    vp = torch.zeros_like(kp)
    kp[:, slot], vp[:, slot] = x["k"], x["v"]
    return P.kv_view(kp, vp, x["pos"], S, slot=slot.to(torch.int32))


def prepare(case, seed):
    c = case
    x = _inputs(c, seed)
    s = dict(c=c, ctx=_context(), pages=P.Pages(x["start"], x["len"]))
    kind = c["kind"]
    if kind == "checkpoint":
        n, L, B = c["seqs"], c["layers"], c["budget"]
        out = (n, L, c["hkv"], B, c["d"])
        no, keep = P.Pages([], []), slice(len(x["start"]) - x["pend"], None)
        s.update(k=x["k"], v=x["v"], pos=x["pos2"], score=x["score"], n_tokens=[c["S"]] * n, retired=[no] * n,
                 pending=[P.Pages(x["start"][keep], x["len"][keep])] * n, r_pre=[x["r_pre"][i] for i in range(n)],
                 k_out=torch.zeros(out, dtype=torch.bfloat16, device=DEV),
                 v_out=torch.zeros(out, dtype=torch.bfloat16, device=DEV),
                 pos_out=torch.zeros((n, B), dtype=torch.int32, device=DEV))
        return s
    if kind == "batch":
        s["kv"] = [P.kv_view(k, v, x["pos"], x["s_pre"]) for k, v, _ in x["layers"]]
        s["win"] = [P.window_view(q, x["qpos_pre"]) for _, _, q in x["layers"]]
        s["all_pages"] = [s["pages"]] * c["layers"]
        return s
    if kind == "measure":
        ph = c["phase"]
        s["kv"] = _view(c, x, ph, c["paged"])
        s["win"] = P.window_view(x["q_" + ph], x["qpos_" + ph])
        s["want"] = ["R"] + ["R_head"] * c["head"] + ["o", "lse"] * (ph == "post" and c["scan"] >= 0) + ["token_mass"] * c["mass"]
        return s
    s["kv"] = _view(c, x, "post")
    s["win"] = P.window_view(x["q_post"], x["qpos_post"])
    if kind in ("recorded", "joint"):
        e = _effects(c, x, "post", torch.float32, mass=False)
        s["o"], s["lse"] = e["o"].contiguous(), e["lse"].contiguous()
        if kind == "joint":
            R = e["R_head"].amax(1).cpu().numpy()[x["forced"]]
            cand = x["forced"][np.argsort(R, kind="stable")].astype(np.int32)
            s["cand"], s["n_cand"] = torch.from_numpy(cand).to(DEV), torch.tensor([len(cand)], dtype=torch.int32, device=DEV)
        return s
    # commit
    s["kv_pre"] = _view(c, x, "pre")
    s["win_pre"] = P.window_view(x["q_pre"], x["qpos_pre"])
    force = np.zeros(len(x["start"]), np.uint8)
    force[x["forced"]] = 1
    s["force"] = torch.from_numpy(force).to(DEV)
    s["keep"] = slice(len(x["start"]) - x["pend"], len(x["start"]))
    B, shape = c["budget"], (1, 1, c["hkv"], c["budget"], c["d"])
    s.update(k=x["k"][None, None], v=x["v"][None, None], pos=x["pos"][None], score=x["score"], no_pages=P.Pages([], []),
             pending=P.Pages(x["start"][s["keep"]], x["len"][s["keep"]]),
             k_out=torch.zeros(shape, dtype=torch.bfloat16, device=DEV),
             v_out=torch.zeros(shape, dtype=torch.bfloat16, device=DEV),
             pos_out=torch.zeros((1, B), dtype=torch.int32, device=DEV))
    return s


# ---------------------------------------------------------------------- run

MAX_CAND = 256


def run(s):
    c, ctx, kind = s["c"], s["ctx"], s["c"]["kind"]
    if kind == "measure":
        return P.ckv_measure_page_effects(ctx, s["kv"], s["win"], s["pages"], want=s["want"])
    if kind == "recorded":
        return P.ckv_measure_recorded(ctx, s["kv"], s["win"], s["pages"], s["o"], s["lse"],
                                      want=("R", "token_mass") if c["mass"] else ("R",))
    if kind == "batch":
        return [r["R"] for r in P.ckv_measure_page_effects_batch(ctx, s["kv"], s["win"], s["all_pages"])]
    if kind == "joint":
        return P.ckv_joint_test(ctx, s["kv"], s["win"], s["o"], s["lse"], s["pages"], s["cand"], s["n_cand"],
                                s["cand"].numel())
    if kind == "checkpoint":
        return P.ckv_select_and_compact(ctx, s["k"], s["v"], s["pos"], s["n_tokens"], s["score"], s["retired"],
                                        s["pending"], s["r_pre"], budget=c["budget"], keep_recent=min(c["W"], 64),
                                        k_out=s["k_out"], v_out=s["v_out"], pos_out=s["pos_out"])
    pre = P.ckv_measure_page_effects(ctx, s["kv_pre"], s["win_pre"], s["pages"])
    post = P.ckv_measure_page_effects(ctx, s["kv"], s["win"], s["pages"], want=("R", "o", "lse", "token_mass"))
    cl = P.ckv_classify_pages(ctx, pre["R"], post["R"], force=s["force"], max_cand=MAX_CAND)
    jt = P.ckv_joint_test(ctx, s["kv"], s["win"], post["o"], post["lse"], s["pages"], cl["cand"], cl["n_cand"], MAX_CAND)
    sel = P.ckv_select_and_compact(ctx, s["k"], s["v"], s["pos"], [c["S"]], s["score"], [s["no_pages"]], [s["pending"]],
                                   [pre["R"][s["keep"]]], budget=c["budget"], keep_recent=c["W"], k_out=s["k_out"],
                                   v_out=s["v_out"], pos_out=s["pos_out"],
                                   accepted=[(s["pages"], cl["cand"], cl["n_cand"], jt["accepted"], MAX_CAND)])
    return dict(R_pre=pre["R"], R_post=post["R"], o=post["o"], lse=post["lse"], token_mass=post["token_mass"],
                classes=cl, joint=jt, checkpoint=sel)


# --------------------------------------------------------- work, tolerance

def work(case):
    c = case
    hq, hkv, d, S, W, kind = c["hq"], c["hkv"], c["d"], c["S"], c["W"], c["kind"]
    rows = hq * W
    kv, q, out = S * hkv * d * 4 + 4 * S, rows * d * 2, rows * (d + 1) * 4
    flops = 4.0 * rows * S * d                       # q.k and the weighted values, once per token
    if kind == "measure":
        o = (out if c["phase"] == "post" and c["scan"] >= 0 else 0) + (4 * S if c["mass"] else 0)
        return {"bytes": kv + q + o, "flops": flops}
    if kind == "recorded":
        return {"bytes": kv + q + out + (4 * S if c["mass"] else 0), "flops": flops}
    if kind == "batch":
        return {"bytes": c["layers"] * (kv + q), "flops": c["layers"] * flops}
    if kind == "joint":
        tok = 0.65 * c["forced"] * S                 # tokens of the candidate pages
        return {"bytes": tok * hkv * d * 4 + q + out, "flops": 4.0 * rows * tok * d}
    moved = c["budget"] * (2.0 * hkv * d * 4) + 8 * c["budget"]
    if kind == "checkpoint":
        return {"bytes": c["seqs"] * (c["layers"] * moved + 4 * S), "flops": 0.0}
    return {"bytes": 2 * (kv + q) + out + 8 * S + moved, "flops": 2 * flops}


def tolerance(case):
    if case["kind"] == "checkpoint":
        return "exact"
    # float16 weights: 5e-5 off 64 bits on the longest case; a near tie may swap two candidates
    return {"rel": 2e-4, "max": 4e-3, "differ": 0.01}


# -------------------------------------------------------------------- exact

def exact(case, seed):
    c = case
    x = _inputs(c, seed)
    f8, kind = torch.float64, c["kind"]

    def amax(e):
        return e["R_head"].amax(1)

    if kind == "measure":
        e = _effects(c, x, c["phase"], f8, mass=c["mass"])
        post = c["phase"] == "post" and c["scan"] >= 0
        return dict(R=amax(e) if len(x["start"]) else None, R_head=e["R_head"] if c["head"] else None,
                    o=e["o"] if post else None, lse=e["lse"] if post else None,
                    token_mass=e["mass"] if c["mass"] else None)
    if kind == "recorded":
        e = _effects(c, x, "post", f8, mass=c["mass"])
        return dict(R=amax(e), R_head=None, token_mass=e["mass"] if c["mass"] else None)
    if kind == "batch":
        n = x["s_pre"]
        return [amax(_attend(k[:, :n], v[:, :n], q, x["pos"][:n], x["qpos_pre"], x["start"], x["len"], f8, mass=False))
                for k, v, q in x["layers"]]
    if kind == "joint":
        e = _effects(c, x, "post", torch.float32, mass=False)
        R = e["R_head"].amax(1).cpu().numpy()[x["forced"]]
        cand = x["forced"][np.argsort(R, kind="stable")]
        e = _effects(c, x, "post", f8, mass=False, residual_of=torch.from_numpy(cand).to(DEV))
        n, union, acc = len(cand), [], []
        D = [torch.zeros_like(r[0]) for r, _, _ in e["residuals"]]
        A = [torch.zeros_like(a[0]) for _, a, _ in e["residuals"]]
        for t in range(n):
            u = max(float(((D[g] + r[t]).norm(dim=1) / ((1 - A[g] - a[t]) * on)).max())
                    for g, (r, a, on) in enumerate(e["residuals"]))
            union.append(u)
            acc.append(u <= np.float32(0.01))
            if acc[-1]:
                for g, (r, a, on) in enumerate(e["residuals"]):
                    D[g] += r[t]
                    A[g] += a[t]
        return dict(accepted=torch.tensor(acc, dtype=torch.uint8), union_R=torch.tensor(union, dtype=f8),
                    n_accepted=torch.tensor([sum(acc)], dtype=torch.int32))
    if kind == "checkpoint":
        return None                                  # bytes copied: nothing is computed
    pre, post = _effects(c, x, "pre", f8, mass=False), _effects(c, x, "post", f8)
    return dict(R_pre=amax(pre), R_post=amax(post), o=post["o"], lse=post["lse"], token_mass=post["mass"],
                classes=None, joint=None, checkpoint=None)
