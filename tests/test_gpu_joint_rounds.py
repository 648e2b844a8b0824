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
