"""ckv_measure_page_effects_batch over runs of problems that share their
kernels (one launch each over the whole run): every output bit-identical to
the single calls, whose results the oracle tests pin.

The problems of a run differ in length (ragged last splits and tiles) and
page lists; one has no pages, and a heavy key puts pairs on the fix-up list.
The shapes are the edges of the batch's kernels: up to 64 rows per KV head
(two page groups per workgroup), up to 128, above (8 waves), several row
blocks; pages of at most 32 tokens and longer; contiguous and paged caches;
the token mass in its fast and general forms.  Twelve problems of 32 splits
and 8 KV heads give a workgroup several splits.
"""
import ctypes

import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu

WANT = ("R", "R_head", "o", "lse", "token_mass")


@pytest.fixture(scope="module")
def ckv():
    import paper_2608_07855_amd as P
    ctx = P.Context(0)
    yield P, ctx
    ctx.close()


def _problem(P, hq, hkv, d, S, W, G, paged, seed, pages=True):
    g = torch.Generator(device="cuda")
    g.manual_seed(seed)
    rows = S + 300 if paged else S
    k = torch.randn((hkv, rows, d), generator=g, device="cuda", dtype=torch.bfloat16)
    v = torch.randn((hkv, rows, d), generator=g, device="cuda", dtype=torch.bfloat16)
    q = torch.randn((hq, W, d), generator=g, device="cuda", dtype=torch.bfloat16)
    slot = torch.randperm(rows, generator=g, device="cuda")[:S].to(torch.int32) if paged else None
    for t in range(5, S, S // 7):     # keys that dominate some rows
        k[:, int(slot[t]) if paged else t] *= 5
    pos = torch.arange(S, dtype=torch.int32, device="cuda")
    kv = P.kv_view(k, v, pos, S, slot=slot) if paged else P.kv_view(k, v, pos, S)
    start = np.arange(3, S - W - G, G + 5, dtype=np.int32) if pages else np.zeros(0, np.int32)
    rng = np.random.default_rng(seed)
    length = rng.integers(max(1, G - 7), G + 1, len(start)).astype(np.int32)
    return kv, P.window_view(q, pos[S - W:].clone()), P.Pages(start, length), (k, v, q, pos, slot)


def _same(got, ref, what):
    for i, (b, s) in enumerate(zip(got, ref)):
        for key in WANT:
            if b[key] is None:
                assert s[key] is None or s[key].numel() == 0
                continue
            x, y = b[key].cpu().numpy().view(np.uint32), s[key].cpu().numpy().view(np.uint32)
            assert np.array_equal(x, y), f"{what}: problem {i} {key}"


@pytest.mark.parametrize("mass", [False, True])
@pytest.mark.parametrize("paged", [False, True])
@pytest.mark.parametrize("hq,hkv,d,W,G", [(5, 1, 128, 8, 16), (4, 2, 64, 32, 48), (8, 2, 128, 32, 32),
                                          (8, 2, 128, 29, 64), (8, 2, 64, 64, 24), (6, 2, 128, 100, 40),
                                          (2, 1, 64, 80, 30)])
def test_batch_is_the_single_calls(ckv, hq, hkv, d, W, G, paged, mass):
    P, ctx = ckv
    print(f"[batch] hq={hq} hkv={hkv} d={d} W={W} G={G} paged={paged} mass={mass}", flush=True)
    want = WANT if mass else WANT[:-1]
    pr = [_problem(P, hq, hkv, d, S, W, G, paged, seed=100 + i, pages=i != 2)
          for i, S in enumerate((700, 1234, 900, 641, 2049))]
    got = P.ckv_measure_page_effects_batch(ctx, [p[0] for p in pr], [p[1] for p in pr], [p[2] for p in pr], want=want)
    ref = [P.ckv_measure_page_effects(ctx, p[0], p[1], p[2], want=want) for p in pr]
    torch.cuda.synchronize()
    ctx.sync()
    _same(got, ref, "batch")


def test_several_splits_per_workgroup_and_workspace_limit(ckv):
    """Twelve problems in one launch; then with a workspace that holds one
    problem only, where they go out one by one; then one that holds a run of
    one beside it, and one that holds a run of two."""
    P, ctx0 = ckv
    pr = [_problem(P, 16, 8, 64, 4096 - 60 * i, 8, 16, False, seed=i) for i in range(12)]
    args = [[p[j] for p in pr] for j in range(3)]
    ref = [P.ckv_measure_page_effects(ctx0, *p[:3], want=WANT) for p in pr]
    _same(P.ckv_measure_page_effects_batch(ctx0, *args, want=WANT), ref, "no limit")
    one = P.Context(0)
    P.ckv_measure_page_effects(one, *pr[0][:3], want=WANT)
    need = one.workspace_bytes()
    one.close()
    for limit in (need, 2 * need + 65536, 3 * need + 131072):
        ctx = P.Context(0)
        ctx.set_workspace_limit(limit)
        got = P.ckv_measure_page_effects_batch(ctx, *args, want=WANT)
        torch.cuda.synchronize()
        assert ctx.workspace_bytes() <= limit
        _same(got, ref, f"limit {limit}")
        ctx.close()


def test_problem_that_goes_out_alone(ckv):
    """25000 tokens and 1024 window rows per KV head (391 x 8 x 4 window tiles,
    more than 48 per compute unit) between problems that share a launch."""
    P, ctx = ckv
    pr = [_problem(P, 64, 8, 64, S, 128, 64, False, seed=70 + i) for i, S in enumerate((700, 1100, 25000, 900, 641, 25000))]
    got = P.ckv_measure_page_effects_batch(ctx, *[[p[j] for p in pr] for j in range(3)], want=WANT)
    _same(got, [P.ckv_measure_page_effects(ctx, *p[:3], want=WANT) for p in pr], "alone")


@pytest.mark.parametrize("shared", ["o", "lse", "R", "R_head", "token_mass"])
def test_problems_that_share_an_output(ckv, shared):
    """One buffer for the same output of every problem: the other outputs are
    those of single calls (R comes from the problem's own o), and the buffer
    holds the last problem's."""
    P, ctx = ckv
    print(f"[batch] shared {shared}", flush=True)
    hq, d, W = 8, 64, 8
    pr = [_problem(P, hq, 2, d, S, W, 16, False, seed=50 + i) for i, S in enumerate((900, 700, 820, 641))]
    ref = [P.ckv_measure_page_effects(ctx, *p[:3], want=WANT) for p in pr]
    size = lambda key, p: {"R": p[2].n, "R_head": p[2].n * hq, "o": hq * W * d, "lse": hq * W,
                           "token_mass": p[0].n_tokens}[key]
    outs = {key: [torch.full((size(key, p),), -3.0, device="cuda") for p in pr] for key in WANT}
    outs[shared] = [torch.full((max(size(shared, p) for p in pr),), -3.0, device="cuda")] * len(pr)
    n = len(pr)
    arrs = [(ctypes.c_void_p * n)(*[t.data_ptr() for t in outs[key]]) for key in WANT]
    ctx.check(P.lib().ckv_measure_page_effects_batch(
        ctx.handle, n, (type(pr[0][0]) * n)(*[p[0] for p in pr]), (type(pr[0][1]) * n)(*[p[1] for p in pr]),
        (type(pr[0][2].view()) * n)(*[p[2].view() for p in pr]), *arrs))
    torch.cuda.synchronize()
    for i, (p, s) in enumerate(zip(pr, ref)):
        for key in WANT:
            if key == shared and i < n - 1:
                continue
            got = outs[key][i][:size(key, p)]
            assert torch.equal(got.view(torch.int32), s[key].reshape(-1).view(torch.int32)), f"problem {i} {key}"


def test_single_calls_keep_their_memory(ckv):
    """A graph of a single call stays valid when a batch of such problems grows
    the context's memory, and gives the single call's results."""
    P, _ = ckv
    stream = torch.cuda.Stream()
    pr = [_problem(P, 8, 2, 64, 3000 + 50 * i, 8, 16, False, seed=80 + i) for i in range(8)]
    torch.cuda.synchronize()
    ctx = P.Context(0, stream)
    with torch.cuda.stream(stream):
        ref = [P.ckv_measure_page_effects(ctx, *p[:3], want=WANT) for p in pr]
        held = ctx.workspace_bytes()
        R = torch.empty(pr[0][2].n, device="cuda")
        graph = torch.cuda.CUDAGraph()
        with torch.cuda.graph(graph, stream=stream):
            P.ckv_measure_page_effects(ctx, *pr[0][:3], R=R)
        for _ in range(3):
            got = P.ckv_measure_page_effects_batch(ctx, *[[p[j] for p in pr] for j in range(3)], want=WANT)
            _same(got, ref, "batch")
            # what the memory that the batch took in place of the calls' would hold by now
            junk = torch.full((held // 4,), float("nan"), device="cuda")
            R.fill_(-1)
            graph.replay()
            stream.synchronize()
            assert torch.equal(R.view(torch.int32), ref[0]["R"].view(torch.int32))
            del junk
    assert ctx.workspace_bytes() > 2 * held
    del graph
    ctx.close()


def test_batch_under_capture(ckv):
    """A batch call recorded in a graph after an equal one: every replay, with
    other inputs and with eager batches of other problems in between (which
    reuse the pinned memory that eager batches pass their arguments through),
    gives the single calls' results."""
    P, _ = ckv
    stream = torch.cuda.Stream()
    pr = [_problem(P, 8, 2, 64, S, 8, 16, False, seed=90 + i, pages=i != 1) for i, S in enumerate((900, 700, 820))]
    other = [_problem(P, 8, 2, 64, 2000 + 60 * i, 8, 24, False, seed=95 + i) for i in range(5)]
    torch.cuda.synchronize()
    ctx = P.Context(0, stream)
    with torch.cuda.stream(stream):
        args = [[p[j] for p in pr] for j in range(3)]
        P.ckv_measure_page_effects_batch(ctx, *args, want=WANT)
        R = [torch.empty(max(p[2].n, 1), device="cuda") for p in pr]
        graph = torch.cuda.CUDAGraph()
        with torch.cuda.graph(graph, stream=stream):
            got = P.ckv_measure_page_effects_batch(ctx, *args, R=R, want=WANT)
        for rep in range(4):
            for _ in range(5):
                P.ckv_measure_page_effects_batch(ctx, *[[p[j] for p in other] for j in range(3)], want=WANT)
            for p in pr:
                p[3][2].mul_(-1 if rep % 2 else 0.5)   # the queries
            for x in got:
                for key in WANT:
                    x[key].fill_(-1)
            graph.replay()
            stream.synchronize()
            _same(got, [P.ckv_measure_page_effects(ctx, *p[:3], want=WANT) for p in pr], f"replay {rep}")
    del graph
    ctx.sync()
    ctx.close()


def test_memory_grows_ahead(ckv):
    """A batch that grows by a problem per call does not move its memory at
    every call."""
    P, _ = ckv
    pr = [_problem(P, 8, 2, 64, 700, 8, 16, False, seed=i) for i in range(12)]
    ctx = P.Context(0)
    held = []
    for n in range(8, 12):    # 12 problems would just miss one and a half times 8
        P.ckv_measure_page_effects_batch(ctx, *[[p[j] for p in pr[:n]] for j in range(3)])
        held.append(ctx.workspace_bytes())
    torch.cuda.synchronize()
    assert held[0] < held[1] == held[2] == held[3]
    ctx.close()
