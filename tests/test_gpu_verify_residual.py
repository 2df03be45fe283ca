"""dyspec_verify on the residual updates: many rejected siblings under one node (past the 64 whose keys are made
together), vocabularies around a thread's share (4), a segment (2048) and the largest, both table types, and rows in which
R - D leaves no mass (R is kept).  Compared with the oracle by the helpers' rules and tolerances."""
import numpy as np
import pytest

import oracle
from helpers import f32, verify_in_full

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


def star(dy, tokens):
    """The root with one child per token, in this order."""
    n = len(tokens) + 1
    parent = np.array([-1] + [0] * (n - 1), np.int32)
    fc, ns, dep = oracle.links_from_parent(parent)
    token = np.array([-1] + list(tokens), np.int32)
    rank = np.array([0] + list(range(n - 1)), np.int32)
    mk = lambda a: torch.from_numpy(np.ascontiguousarray(a, dtype=np.int32)).cuda()
    return dy.Tree(mk(parent), mk(token), mk(rank), mk(fc), mk(ns), mk(dep)), (token, fc, ns)


def compare(dy, tokens, d, t, td, tt, seed, bf16):
    dd, tg = torch.from_numpy(d), torch.from_numpy(t)
    if bf16:
        dd, tg = dd.to(torch.bfloat16), tg.to(torch.bfloat16)
    batch = dy.Batch.from_sizes([len(tokens) + 1])
    tree, otree = star(dy, tokens)
    gd, gt = dd.cuda(), tg.cuda()
    return verify_in_full(lambda sd: dy.verify(gd, gt, batch, tree, (td,), (tt,), sd), batch, [otree],
                          dd.float().numpy(), tg.float().numpy(), (td,), (tt,), seed)


@pytest.fixture(scope="module")
def dy():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2410_11744_amd as m
    m.load_library()
    return m


@pytest.mark.parametrize("bf16", [False, True])
@pytest.mark.parametrize("kids,V,tt", [(1, 4, 1.0), (3, 5, 0.7), (30, 1000, 1.0), (63, 2047, 0.6), (64, 2048, 0.6), (65, 2049, 1.0), (66, 2052, 0.0),
                                       (130, 4100, 0.6), (200, 32000, 1.0), (200, 32768, 0.0), (70, 32765, 0.6)])
def test_many_rejections(dy, kids, V, tt, bf16):
    print(f"children {kids} V={V} target temperature {tt} bf16={bf16}", flush=True)
    rng = np.random.default_rng(kids * 70000 + V)
    n = kids + 1
    d = (rng.standard_normal((n, V)) * 2.0).astype(np.float32)
    t = (rng.standard_normal((n, V)) * 2.0).astype(np.float32)          # unrelated to the draft: most children are rejected
    tokens = np.argsort(-(d[0] / f32(0.9) + rng.gumbel(size=V)))[:kids]  # a sample without replacement
    compare(dy, tokens, d, t, 0.9, tt, 5 + kids, bf16)


@pytest.mark.parametrize("bf16", [False, True])
@pytest.mark.parametrize("kids,late,V,tt", [(65, 63, 2048, 0.6), (65, 64, 2049, 1.0), (130, 127, 4100, 0.6), (130, 129, 1000, 1.0), (200, 128, 32000, 1.0),
                                            (200, 199, 32765, 0.6), (200, 65, 32768, 0.0)])
def test_child_far_down_the_scan_is_accepted(dy, kids, late, V, tt, bf16):
    """The children before number `late` are impossible for the target, which puts most of its weight on that one: all of
    them are tested, rejected, and it is accepted, whatever the draws."""
    rng = np.random.default_rng(kids * 1000 + late)
    d = (rng.standard_normal((kids + 1, V)) * 2.0).astype(np.float32)
    t = (rng.standard_normal((kids + 1, V)) * 2.0).astype(np.float32)
    tokens = np.argsort(-(d[0] / f32(0.9) + rng.gumbel(size=V)))[:kids]
    t[0, tokens[:late]] = -np.inf
    t[0, tokens[late]] = 20.0
    out, _ = compare(dy, tokens, d, t, 0.9, tt, 5 + kids, bf16)
    assert out.n_accepted.item() == 1 and out.accepted_nodes[0].item() == late + 1
    ratio = out.accept_ratio.cpu().numpy()
    assert (ratio[1:late + 1] == 0.0).all() and ratio[late + 1] >= 1.0 and (ratio[late + 2:] == -2.0).all()


@pytest.mark.parametrize("V,tt", [(6, 1.0), (6, 0.0), (2100, 1.0), (2100, 0.0), (32000, 0.7)])
def test_rows_that_leave_no_mass(dy, V, tt):
    """Draft and target alike, children on tokens neither can emit: every one is rejected, R == D stays, and the last
    token comes from it; then a child on a possible token, whose ratio is 1."""
    live = [V // 2, V - 1]
    row = np.full(V, -np.inf, np.float32)
    row[live] = [0.5, 0.5] if tt > 0 else [0.5, -np.inf]                 # temperature 0: one token in both
    d = np.repeat(row[None], 6, axis=0)
    dead = [x for x in range(V) if x not in live][:4]
    for tokens in ([dead[0]], dead[:3], [dead[0], live[0]], [dead[0], dead[1], live[0], dead[2]]):
        n = len(tokens) + 1
        h = np.ascontiguousarray(d[:n])
        tree, (token, fc, ns) = star(dy, tokens)
        g = torch.from_numpy(h).cuda()
        for seed in range(4):
            out = dy.verify(g, g, dy.Batch.from_sizes([n]), tree, (1.0,), (tt,), seed)
            want = oracle.verify(h, h, token, fc, ns, 1.0, f32(tt), seed, seq=0, emit_bonus=True)
            # (an impossible token's ratio is 0 / 0 in the oracle: the path and the last token are compared; no draw
            #  comes near an acceptance ratio of 0 or 1, and the two tokens split the last draw in the middle)
            k = int(out.n_accepted.item())
            assert k == want.n_accepted and out.accepted_nodes.cpu().numpy()[:k].tolist() == want.accepted_nodes.tolist()
            assert want.resid_margin < 1e-5 or out.final_token.item() == want.final_token


@pytest.mark.parametrize("bf16", [False, True])
@pytest.mark.parametrize("V,rest", [(40, 1e-3), (40, 1e-5), (3000, 1e-4), (3001, 1e-6), (32000, 1e-5), (32765, 1e-6)])
def test_ratio_behind_a_sibling_that_outweighs_the_rest(dy, V, rest, bf16):
    """The first child's token holds all but `rest` of the draft row and is impossible for the target: rejected. The
    second child's ratio divides by what is left of the draft row, against 64 bits.  Bound: weights exp(x) with
    |x| <= 27 carry 2^-24 (3 |x| + 2) = 5e-6 each, in the row sums as well; sums of at most 64 terms in a row
    another 4e-6 each, for draft and target: 3e-5 in all."""
    rng = np.random.default_rng(V + int(1 / rest))
    d = rng.standard_normal((3, V)).astype(np.float32)
    t = rng.standard_normal((3, V)).astype(np.float32)
    y1, y2 = V // 3, V - 2
    d[0, y1] = np.log(np.exp(np.delete(d[0], y1).astype(np.float64)).sum() / rest)
    t[0, y1] = -60.0
    t[0, y2] = 8.0                                                      # R - D keeps it nearly whole
    gd, gt = torch.from_numpy(d), torch.from_numpy(t)
    if bf16:
        gd, gt = gd.to(torch.bfloat16), gt.to(torch.bfloat16)
    tree, _ = star(dy, [y1, y2])
    out = dy.verify(gd.cuda(), gt.cuda(), dy.Batch.from_sizes([3]), tree, (1.0,), (1.0,), 11)
    p, q = (np.exp(x.double().numpy()[0]) for x in (gd, gt))
    p, q = p / p.sum(), q / q.sum()
    r = np.maximum(q - p, 0.0)
    left = np.delete(p, y1).sum()
    np.testing.assert_allclose(out.accept_ratio.cpu().numpy()[2], r[y2] / r.sum() / (p[y2] / left), rtol=3e-5)


@pytest.mark.parametrize("kids,V,tt", [(20, 50, 1.0), (300, 1000, 1.0), (300, 1000, 0.0), (700, 32000, 0.8)])
def test_mass_that_shrinks_with_every_rejection(dy, kids, V, tt):
    """What is left of the target lies on one token, which holds most of the draft row and is no child: each rejection
    takes more than half of its weight (2^-700 in all), and the last token is still that one."""
    rng = np.random.default_rng(kids + V)
    d = (rng.standard_normal((kids + 1, V)) * 0.5).astype(np.float32)
    t = d.copy()
    top = V // 2
    d[0, top] = np.log(2.0 * np.exp(np.delete(d[0], top).astype(np.float64)).sum())
    t[0] = d[0]
    t[0, top] += 3.0
    tokens = np.array([x for x in rng.permutation(V) if x != top][:kids])
    out, _ = compare(dy, tokens, d, t, 1.0, tt, 3, False)
    assert out.n_accepted.item() == 0 and out.final_token.item() == top


@pytest.mark.parametrize("low", [-40.0, -60.0, -86.0])
def test_what_is_left_weighs_next_to_nothing(dy, low):
    """Draft and target alike but for one token of weight exp(low) that only the target has: after a rejected child it is
    all that is left, however small."""
    V, a, b = 2100, 7, 2099
    d = np.full((4, V), -np.inf, np.float32)
    d[:, a] = 0.0
    t = d.copy()
    t[:, b] = low
    for tokens in ([3], [3, 2051], [3, 2051, 4]):
        n = len(tokens) + 1
        tree, _ = star(dy, tokens)
        out = dy.verify(torch.from_numpy(d[:n].copy()).cuda(), torch.from_numpy(t[:n].copy()).cuda(), dy.Batch.from_sizes([n]), tree, (1.0,), (1.0,), 1)
        assert out.n_accepted.item() == 0 and out.final_token.item() == b


@pytest.mark.parametrize("bf16", [False, True])
@pytest.mark.parametrize("V", [2100, 2101, 32000, 32768])
def test_draft_rest_far_below_the_first_child(dy, V, bf16):
    """The draft row lies on a few tokens, 84 nats and more apart, all of them children; the target is flat: all children
    are rejected and the last token is one of the others.  (A factor that turns the draft's weights into shares of a
    target row of weight V is past the range of fp32 here.)"""
    tokens = [V // 3, 5, V - 1]
    d, t = np.full((4, V), -np.inf, np.float32), np.zeros((4, V), np.float32)
    d[:, tokens[0]], d[:, tokens[1]], d[:, tokens[2]] = 0.0, -84.0, -87.0
    tree, (token, fc, ns) = star(dy, tokens)
    gd, gt = torch.from_numpy(d), torch.from_numpy(t)
    if bf16:
        gd, gt = gd.to(torch.bfloat16), gt.to(torch.bfloat16)
    gd, gt = gd.cuda(), gt.cuda()
    want = oracle.accept_ratio_all(d, t, token, fc, ns, 1.0, 1.0)
    last = set()
    for seed in range(16):
        out = dy.verify(gd, gt, dy.Batch.from_sizes([4]), tree, (1.0,), (1.0,), seed)
        # weights exp(x) with |x| <= 87 carry 2^-24 (3 |x| + 2) = 1.6e-5, twice in a ratio
        np.testing.assert_allclose(out.accept_ratio.cpu().numpy(), want, rtol=5e-5, atol=1e-12)
        assert out.n_accepted.item() == 0
        last.add(out.final_token.item())
    assert not last & set(tokens) and len(last) > 8


def spoilt(kind, rows, V, at, rng):
    x = (rng.standard_normal((rows, V)) * 2.0).astype(np.float32)
    if kind == "all -inf":
        x[:] = -np.inf
    elif kind == "one nan":
        x[:, at] = np.nan
    elif kind == "all nan":
        x[:] = np.nan
    elif kind == "one inf":
        x[:, at] = np.inf
    return x


@pytest.mark.parametrize("bf16", [False, True])
@pytest.mark.parametrize("draft,target,tt", [("fine", "all -inf", 1.0), ("fine", "one nan", 1.0), ("fine", "all nan", 1.0), ("fine", "one inf", 1.0),
                                             ("all -inf", "fine", 1.0), ("one nan", "fine", 1.0), ("all nan", "fine", 1.0), ("one inf", "fine", 1.0),
                                             ("one nan", "one nan", 1.0), ("all -inf", "all -inf", 1.0),
                                             ("all -inf", "fine", 0.0), ("one nan", "fine", 0.0), ("one inf", "fine", 0.0)])
def test_rows_that_are_no_distribution(dy, draft, target, tt, bf16):
    """Against the oracle: under such a target row no child is accepted and there is no last token; after a draft row like
    that the first child's rejection ends the scan, and the last token comes from the target row as it is.  (The
    children are impossible for the target, so the first one is rejected.)"""
    rng = np.random.default_rng(len(draft) * 100 + len(target))
    last_tokens = 0
    for V in (5, 2101, 4096):
        for tokens in ([V // 2], [0, V - 1, 1, V // 2], [V // 2, V // 2 - 1, 0]):
            n = len(tokens) + 1
            d, t = spoilt(draft, n, V, V // 2, rng), spoilt(target, n, V, V // 2 + 1, rng)
            if target != "all nan":
                t[:, tokens] = -np.inf
            dd, tg = torch.from_numpy(d), torch.from_numpy(t)
            if bf16:
                dd, tg = dd.to(torch.bfloat16), tg.to(torch.bfloat16)
            tree, (token, fc, ns) = star(dy, tokens)
            for seed in range(4):
                out = dy.verify(dd.cuda(), tg.cuda(), dy.Batch.from_sizes([n]), tree, (1.0,), (tt,), seed)
                want = oracle.verify(dd.float().numpy(), tg.float().numpy(), token, fc, ns, 1.0, tt, seed, seq=0, emit_bonus=True)
                assert out.n_accepted.item() == want.n_accepted == 0
                if want.final_token < 0 or want.resid_margin >= 1e-5:
                    assert out.final_token.item() == want.final_token
                    last_tokens += 1
    assert last_tokens >= 24
