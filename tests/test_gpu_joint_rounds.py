"""The joint test's rounds at their edges: candidate counts around the round's
window, decision sequences that mix both outcomes, rows whose state lives in
global memory, a fix-up list that fills up, and a caller that does not read
the union effects.

Reference: float64 torch, the union of each step deleted by its definition,
decisions replayed.  Tolerance 2e-3 relative as for every score (float16
weights round to 2^-11, and up to a union mass of 0.8 the effect carries at
most A / (1 - A) = 4 of them; above it the library recomputes by definition).
"""
import ctypes

import numpy as np
import pytest
import torch

from tests.gpu_util import REL_TOL, assert_scores_close

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def ckv():
    import paper_2608_07855_amd as P
    ctx = P.Context(0)
    yield P, ctx
    ctx.close()


def _replay64(k, v, q, pos, qpos, pages, cand, acc):
    """max over heads and rows of ||o - o^{\\X}|| / ||o|| for X = accepted before t, and t."""
    hq, W, d = q.shape
    grp = hq // k.shape[0]
    start, length = pages
    S = k.shape[1]
    out = np.zeros(len(cand))
    hide = pos[None].long() > qpos[:, None].long()
    for h in range(hq):
        kh, vh = k[h // grp].double(), v[h // grp].double()
        a = ((q[h].double() @ kh.T) / d ** 0.5).masked_fill(hide, -torch.inf).softmax(1)
        o = a @ vh
        keep = torch.ones(S, dtype=torch.bool, device=k.device)
        for t, j in enumerate(cand):
            kt = keep.clone()
            kt[start[j]:start[j] + length[j]] = False
            m = (a * kt).sum(1, keepdim=True)
            od = ((a * kt) @ vh) / m
            out[t] = max(out[t], float(((o - od).norm(dim=1) / o.norm(dim=1)).max()))
            if acc[t]:
                keep = kt
    return out


def _layer(hq, hkv, d, S, W, G, seed, heavy_first=False):
    g = torch.Generator(device="cuda")
    g.manual_seed(seed)
    k = torch.randn((hkv, S, d), generator=g, device="cuda", dtype=torch.bfloat16)
    v = torch.randn((hkv, S, d), generator=g, device="cuda", dtype=torch.bfloat16)
    q = torch.randn((hq, W, d), generator=g, device="cuda", dtype=torch.bfloat16)
    pos = torch.arange(S, dtype=torch.int32, device="cuda")
    qpos = pos[S - W:].clone()
    start = np.arange(0, S - W - G + 1, G, dtype=np.int32)
    length = np.full(len(start), G, np.int32)
    if heavy_first:   # page 0 carries about 0.9 of every row's mass
        q[:, :, 0] = 1
        k[:, :, 0] = 0
        k[:, :G, 0] = d ** 0.5 * float(np.log(9.0 * (S - G) / G))
    return k, v, q, pos, qpos, start, length


def _run(P, ctx, layer, cand, tau):
    k, v, q, pos, qpos, start, length = layer
    kv, win, pages = P.kv_view(k, v, pos), P.window_view(q, qpos), P.Pages(start, length)
    m = P.ckv_measure_page_effects(ctx, kv, win, pages, want=("R", "o", "lse"))
    dc = torch.tensor(cand, dtype=torch.int32, device="cuda")
    nc = torch.tensor([len(cand)], dtype=torch.int32, device="cuda")
    if callable(tau):
        tau = tau(m["R"].cpu().numpy()[cand])
    out = P.ckv_joint_test(ctx, kv, win, m["o"], m["lse"], pages, dc, nc, len(cand) + 2, tau)
    torch.cuda.synchronize()
    ctx.sync()
    acc, u = out["accepted"].cpu().numpy(), out["union_R"].cpu().numpy()
    n = len(cand)
    assert not acc[n:].any() and np.isnan(u[n:]).all()
    assert int(out["n_accepted"].item()) == int(acc.sum())
    return acc[:n], u[:n], tau, (kv, win, pages, m, dc, nc)


def _check(layer, cand, acc, u, tau, gate=True):
    k, v, q, pos, qpos, start, length = layer
    ref = _replay64(k, v, q, pos, qpos, (start, length), cand, acc)
    assert_scores_close(u, ref, "union_R")
    for t, (a, r) in enumerate(zip(acc, ref)):
        if gate and abs(r - tau) > REL_TOL * tau:
            assert bool(a) == (r <= tau), f"step {t}: decision {a}, R_ref {r}, tau {tau}"


@pytest.mark.parametrize("d,W", [(64, 5), (128, 33)])
@pytest.mark.parametrize("n", [1, 16, 31, 32, 33, 64, 65, 97])
def test_window_edges(ckv, d, W, n):
    """Candidates in a random order: accepted and rejected ones alternate."""
    P, ctx = ckv
    layer = _layer(4, 2, d, 900, W, 8, seed=n)
    cand = np.random.default_rng(n).permutation(len(layer[5]))[:n]
    print(f"[joint rounds] d={d} W={W} n={n}", flush=True)
    acc, u, tau, _ = _run(P, ctx, layer, cand, lambda R: float(np.median(R) * 1.3))
    print("".join(map(str, acc)))
    _check(layer, cand, acc, u, tau)


def test_state_in_global_memory(ckv):
    """16640 window rows: more than 64 per workgroup."""
    P, ctx = ckv
    layer = _layer(64, 2, 64, 700, 260, 16, seed=7)
    cand = np.random.default_rng(7).permutation(len(layer[5]))[:20]
    acc, u, tau, _ = _run(P, ctx, layer, cand, lambda R: float(np.median(R) * 1.1))
    assert 0 < acc.sum() < len(cand)
    _check(layer, cand, acc, u, tau)


@pytest.mark.parametrize("gate", [False, True])
def test_union_above_the_closed_form(ckv, gate):
    """The first candidate carries about 0.9 of every row: without the gate all
    are accepted and every later pair is recomputed by definition, more than
    the list holds at once; with a gate that passes everything each candidate
    is decided by such pairs alone."""
    P, ctx = ckv
    layer = _layer(4, 2, 64, 1300, 32, 16, seed=11, heavy_first=True)
    cand = np.arange(77 if not gate else 6)
    if not gate:
        ctx.set_policy("no_joint")
    try:
        acc, u, tau, _ = _run(P, ctx, layer, cand, 1e30)
    finally:
        ctx.set_policy()
    assert acc.all()
    _check(layer, cand, acc, u, tau)


@pytest.mark.parametrize("again", [2, 5, 40])
def test_page_listed_twice(ckv, again):
    """The heavy page is candidate 0 and candidate `again` (of the same round, or
    of the next): candidates in between, which are recomputed by definition,
    miss its tokens all the same."""
    P, ctx = ckv
    layer = _layer(4, 2, 64, 1300, 32, 16, seed=14, heavy_first=True)
    cand = np.insert(np.arange(45), again, 0)
    ctx.set_policy("no_joint")
    try:
        acc, u, tau, _ = _run(P, ctx, layer, cand, 1e30)
    finally:
        ctx.set_policy()
    assert acc.all()
    _check(layer, cand, acc, u, tau)


def test_union_not_read(ckv):
    """union_R NULL: the same decisions."""
    P, ctx = ckv
    layer = _layer(4, 2, 64, 1300, 32, 16, seed=12, heavy_first=True)
    cand = np.array([3, 0, 5, 1, 2, 9])
    acc, u, tau, (kv, win, pages, m, dc, nc) = _run(P, ctx, layer, cand, 0.05)
    acc2 = torch.full((8,), 7, dtype=torch.uint8, device="cuda")
    na = torch.full((1,), -5, dtype=torch.int32, device="cuda")
    pl = pages.view()
    ctx.check(P.lib().ckv_joint_test(ctx.handle, ctypes.byref(kv), ctypes.byref(win), m["o"].data_ptr(),
                                     m["lse"].data_ptr(), ctypes.byref(pl), dc.data_ptr(), nc.data_ptr(), 8, tau,
                                     acc2.data_ptr(), None, na.data_ptr()))
    torch.cuda.synchronize()
    np.testing.assert_array_equal(acc2.cpu().numpy()[:6], acc)
    assert int(na.item()) == int(acc.sum())


def test_more_segments_than_fixup_items(ckv):
    """A paged cache of 31.6 million tokens over a pool of 4096 rows: one row of
    a pair alone has more 1024-token segments (30860) than the fix-up aims at
    (30720).  Page 0 carries about 0.9 of every row's mass, so both candidates
    are decided by such pairs.  Reference: float64 over the pool's rows, each
    weighted by the tokens that map to it."""
    P, ctx = ckv
    S, rows, W, d, G = 31_600_000, 4096, 2, 64, 16
    g = torch.Generator(device="cuda")
    g.manual_seed(13)
    k = torch.randn((1, rows, d), generator=g, device="cuda", dtype=torch.bfloat16)
    v = torch.randn((1, rows, d), generator=g, device="cuda", dtype=torch.bfloat16)
    q = torch.randn((1, W, d), generator=g, device="cuda", dtype=torch.bfloat16)
    q[:, :, 0] = 1
    k[:, :, 0] = 0
    k[:, :G, 0] = d ** 0.5 * float(np.log(20.0 * (S - G) / G))
    slot = torch.randint(G, rows, (S,), generator=g, device="cuda", dtype=torch.int32)
    slot[:G] = torch.arange(G, dtype=torch.int32, device="cuda")
    pos = torch.arange(S, dtype=torch.int32, device="cuda")
    kv, win = P.kv_view(k, v, pos, S, slot=slot), P.window_view(q, pos[S - W:].clone())
    pages = P.Pages([0, 1000], [G, G])
    print("[joint rounds] 31.6M tokens", flush=True)
    m = P.ckv_measure_page_effects(ctx, kv, win, pages, want=("R", "o", "lse"))
    out = P.ckv_joint_test(ctx, kv, win, m["o"], m["lse"], pages, torch.tensor([0, 1], dtype=torch.int32, device="cuda"),
                           torch.tensor([2], dtype=torch.int32, device="cuda"), 2, 1e30)
    torch.cuda.synchronize()
    ctx.sync()

    def output(p, gone):
        count = torch.bincount(slot[:S - W + p + 1].long(), minlength=rows).double()
        for s in gone:
            count -= torch.bincount(slot[s:s + G].long(), minlength=rows).double()
        x = (k[0].double() @ q[0, p].double()) / d ** 0.5
        w = count * torch.exp(x - x.max())
        return (w / w.sum()) @ v[0].double()

    ref = np.zeros(2)
    for t, gone in enumerate(([0], [0, 1000])):
        for p in range(W):
            o = output(p, [])
            ref[t] = max(ref[t], float((o - output(p, gone)).norm() / o.norm()))
    assert out["accepted"].cpu().tolist() == [1, 1] and int(out["n_accepted"].item()) == 2
    assert_scores_close(out["union_R"].cpu().numpy(), ref, "union_R")
