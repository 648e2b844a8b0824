"""Edges of the token mass's pair slices, of the complement pass of recorded
outputs and of the compaction's row batches, against plain torch in float64
(the compaction: bytes).

* Token mass: a workgroup's 8 waves take a (query head, 32-row block) pair
  each; more pairs go to further slices (the last one partly filled), heads of
  16 row blocks take two pairs a wave, and heads that do not fill a workgroup
  the general form, which holds every pair (more than rows / 32 where heads
  round up).  Tolerance: weights come from float32 scores of
  exact bf16 products (1e-4 in the exponent at these sizes) and a log-sum-exp
  whose sum holds float16 weights (2^-11 relative at most): 1e-3.
* Complement pass: pairs with A > 0.99 are spread over parts of their row, at
  most 32 while the pairs are few, in a launch of its own, with and without a
  token mass after it.  2e-3, the score tolerance.
"""
import math

import pytest
import torch

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def ckv():
    import paper_2608_07855_amd as P
    ctx = P.Context(0)
    yield P, ctx
    ctx.close()


def _layer(hkv, group, d, S, W, seed):
    g = torch.Generator(device="cuda")
    g.manual_seed(seed)

    def normal(*shape):
        return torch.randn(shape, generator=g, device="cuda", dtype=torch.bfloat16)

    pos = torch.arange(S, dtype=torch.int32, device="cuda")
    return normal(hkv, S, d), normal(hkv, S, d), normal(hkv * group, W, d), pos, pos[S - W:].clone()


def _attend(k, v, q, pos, qpos):
    """Weights [Hq, W, S], outputs and log-sum-exp in float64."""
    group = q.shape[0] // k.shape[0]
    kk, vv = (t.double().repeat_interleave(group, 0).contiguous() for t in (k, v))
    x = torch.matmul(q.double(), kk.transpose(1, 2).contiguous()) / math.sqrt(q.shape[2])
    x = x.masked_fill(pos[None, None, :] > qpos[None, :, None], -math.inf)
    lse = torch.logsumexp(x, 2)
    a = torch.exp(x - lse[..., None])
    return a, torch.matmul(a, vv), lse, vv


@pytest.mark.parametrize("group,W,d,S", [(1, 8, 64, 65), (5, 8, 128, 700), (8, 32, 128, 1025), (3, 96, 64, 513),
                                         (5, 64, 128, 900), (3, 128, 64, 1200), (8, 128, 128, 2049), (2, 512, 64, 1100),
                                         # the general form with more pairs than rows / 32: 72, 93, 70
                                         (24, 65, 64, 200), (31, 66, 128, 200), (14, 146, 64, 300)])
def test_token_mass_slices(ckv, group, W, d, S):
    P, ctx = ckv
    print(f"[mass] group={group} W={W} d={d} S={S}", flush=True)
    k, v, q, pos, qpos = _layer(2, group, d, S, W, seed=11)
    a, o, lse, _ = _attend(k, v, q, pos, qpos)
    want = a.sum(1).amax(0)
    kv, win = P.kv_view(k, v, pos), P.window_view(q, qpos)
    pages = P.Pages([1, 40], [20, 16])
    fused = P.ckv_measure_page_effects(ctx, kv, win, pages, want=("R", "token_mass"))
    alone = P.ckv_measure_page_effects(ctx, kv, win, P.Pages([], []), want=("R", "token_mass"))
    rec = P.ckv_measure_recorded(ctx, kv, win, pages, o.float().contiguous(), lse.float().contiguous(),
                                 want=("R", "token_mass"))
    two = P.ckv_measure_page_effects_batch(ctx, [kv] * 2, [win] * 2, [pages] * 2, want=("R", "token_mass"))
    for got in (fused, alone, rec, *two):
        torch.testing.assert_close(got["token_mass"].double(), want, rtol=1e-3, atol=1e-9)


@pytest.mark.parametrize("mass", [False, True])
@pytest.mark.parametrize("S,d", [(150, 128), (1000, 64), (5000, 128), (20000, 128), (17000, 64)])
def test_recorded_complement_parts(ckv, S, d, mass):
    P, ctx = ckv
    print(f"[complement] S={S} d={d} mass={mass}", flush=True)
    W, page = 16, (33, 30)
    k, v, q, pos, qpos = _layer(1, 2, d, S, W, seed=12)
    # one key of the page along a few rows' queries: A of 0.99 and more there
    for r in (2, 5, 11):
        q[1, r] = q[0, 2]
    k[0, page[0] + 7] = q[0, 2] * ((math.log(S) + 6.5) * math.sqrt(d) / float(q[0, 2].double().square().sum()))
    a, o, lse, vv = _attend(k, v, q, pos, qpos)
    sel = slice(page[0], page[0] + page[1])
    A = a[..., sel].sum(2)
    assert int((A > 0.992).sum()) >= 3
    rest = a.clone()
    rest[..., sel] = 0
    o2 = torch.matmul(rest, vv) / rest.sum(2, keepdim=True)
    want = ((o - o2).norm(dim=2) / o.norm(dim=2)).amax()
    got = P.ckv_measure_recorded(ctx, P.kv_view(k, v, pos), P.window_view(q, qpos), P.Pages([page[0]], [page[1]]),
                                 o.float().contiguous(), lse.float().contiguous(),
                                 want=("R", "token_mass") if mass else ("R",))
    assert abs(float(got["R"][0]) - float(want)) <= 2e-3 * float(want)
    if mass:
        torch.testing.assert_close(got["token_mass"].double(), a.sum(1).amax(0), rtol=1e-3, atol=1e-9)


@pytest.mark.parametrize("d", [64, 128])
@pytest.mark.parametrize("budget", [9, 127, 128, 129, 255, 257, 400])
def test_compaction_batches(ckv, d, budget):
    P, ctx = ckv
    S, L, H = 600, 2, 3
    g = torch.Generator(device="cuda")
    g.manual_seed(budget)
    k = torch.randn((1, L, H, S, d), generator=g, device="cuda", dtype=torch.bfloat16)
    v = torch.randn((1, L, H, S, d), generator=g, device="cuda", dtype=torch.bfloat16)
    pos = torch.arange(S, dtype=torch.int32, device="cuda")[None] * 2
    score = torch.rand((1, S), generator=g, device="cuda")
    # outputs a few rows longer than the budget: the rows past it stay as they are
    ko, vo = (torch.zeros((1, L, H, budget + 3, d), device="cuda", dtype=torch.bfloat16) for _ in range(2))
    po = torch.zeros((1, budget + 3), dtype=torch.int32, device="cuda")
    no = P.Pages([], [])
    P.ckv_select_and_compact(ctx, k, v, pos, [S], score, [no], [no], [torch.zeros(1, device="cuda")], budget=budget,
                             keep_recent=4, k_out=ko, v_out=vo, pos_out=po)
    s = score[0].clone()
    s[S - 4:] = 2
    kept = torch.sort(torch.topk(s, budget).indices).values
    assert torch.equal(ko[:, :, :, :budget], k[:, :, :, kept]) and torch.equal(vo[:, :, :, :budget], v[:, :, :, kept])
    assert torch.equal(po[:, :budget], pos[:, kept])
    assert not ko[:, :, :, budget:].any() and not vo[:, :, :, budget:].any() and not po[:, budget:].any()
