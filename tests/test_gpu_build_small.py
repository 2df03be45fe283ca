"""dyspec_build_tree with a workspace on many small trees.  The draw waves keep copies of row totals (csrc/row_copies.h);
a node's second draw must start from its row as the first one left it, whoever was served in between.  That order is
rare in one tree, so sixty-four sequences are built per call, of tables in which nodes are drawn from again
and again, and compared with the oracle and with the form without a workspace."""
import numpy as np
import pytest

import oracle
from helpers import BUILD_MARGIN, compare_trees, f32, oracle_trees

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

DRAW_WAVES = 14


@pytest.fixture(scope="module")
def dy():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2410_11744_amd as m
    m.load_library()
    return m


def table(kind, rows, V, rng):
    x = (rng.standard_normal((rows, V)) * 3.0).astype(np.float32)
    if kind.startswith("top"):                          # the rest impossible: rows run empty after a few draws
        k = int(kind[3:])
        keep = np.argpartition(-x, k, axis=1)[:, :k]
        y = np.full_like(x, -np.inf)
        np.put_along_axis(y, keep, np.take_along_axis(x, keep, axis=1), axis=1)
        x = y
    elif kind == "sharp":
        x *= 4.0
    elif kind == "flat":
        x *= 0.1
    elif kind == "lone":                                # a run of 128 tokens that one draw empties (V = 1 mod 128)
        x[:, V - 1] = 6.0 + rng.standard_normal(rows).astype(np.float32)
    return x


def second_draws_after_another_node(parent, n_built, N):
    """Rows of a tree that were drawn from one of a wave's last nodes, again, after the wave had served another node:
    the draws for which a copy fetched before the node's first draw would be outdated."""
    waves = range(DRAW_WAVES)
    held, ahead, next_new = [-1 for _ in waves], [-1 for _ in waves], list(waves)
    held_draws = [0 for _ in waves]
    draws, outdated, hits = {}, {}, 0

    def serve(i):
        w = i % DRAW_WAVES
        if ahead[w] < next_new[w] < N:
            ahead[w] = next_new[w]
        if held[w] != i:
            held_draws[w] = 0 if ahead[w] == i else draws.get(i, 0)
            held[w] = i
        next_new[w] = max(next_new[w], i + DRAW_WAVES)
        outdated[i] = held_draws[w] != draws.get(i, 0)
        draws[i] = draws.get(i, 0) + 1
        held_draws[w] += 1

    for n in range(1, n_built):
        p = int(parent[n])
        hits += p != 0 and outdated[p]
        serve(n)
        if p != 0:                                      # the root's draws are another wave's
            serve(p)
    return hits


def test_a_row_that_an_outdated_copy_would_change(dy):
    """Node 18 draws, node 4 of the same wave draws, node 18 draws again (row 28)."""
    d = (np.random.default_rng(134).normal(size=(32, 1000)) * 3).astype(np.float32)
    want = oracle.build_tree(d, 32, f32(0.6), 134)
    assert second_draws_after_another_node(want.parent, want.n_built, 32) > 0 and want.parent[28] == 18
    batch = dy.Batch.from_sizes([32])
    assert compare_trees(dy.build_tree(torch.from_numpy(d).cuda(), batch, (0.6,), 134), batch, [want]) == 1


@pytest.mark.parametrize("kind", ["normal", "top3", "top5", "sharp", "flat", "lone"])
@pytest.mark.parametrize("N,V", [(15, 1000), (16, 129), (28, 1000), (29, 1025), (32, 1000), (43, 4001), (64, 513)])
def test_small_trees(dy, kind, N, V):
    n_seq, calls, reached = 64, 4, 0
    print(f"{kind} N={N} V={V}", flush=True)
    batch = dy.Batch.from_sizes([N] * n_seq)
    temps = [0.6 if s % 4 else 1.0 for s in range(n_seq)]
    for seed in range(calls):
        d = table(kind, N * n_seq, V, np.random.default_rng([seed, N, V, len(kind)]))
        dd = torch.from_numpy(d).cuda()
        a = dy.build_tree(dd, batch, temps, seed)
        b = dy.build_tree(dd, batch, temps, seed, use_workspace=False)
        trees = oracle_trees(d, [N] * n_seq, temps, seed)
        # (decisions closer than BUILD_MARGIN end a sequence's comparison: hardly any)
        assert compare_trees(a, batch, trees) >= n_seq - 2
        for name in ("parent", "token", "sib_rank", "first_child", "next_sibling", "depth"):
            assert torch.equal(getattr(a.tree, name), getattr(b.tree, name)), name
        assert torch.equal(a.n_built, b.n_built) and torch.equal(a.anc_mask, b.anc_mask) and torch.equal(a.est_value, b.est_value)
        token, parent = a.tree.token.cpu().numpy().reshape(n_seq, N), a.tree.parent.cpu().numpy().reshape(n_seq, N)
        for s, t in enumerate(trees):
            n = t.n_built
            assert ((token[s, 1:n] >= 0) & (token[s, 1:n] < V)).all()
            assert len(set(zip(parent[s, 1:n].tolist(), token[s, 1:n].tolist()))) == n - 1, "siblings' tokens are distinct"
            reached += second_draws_after_another_node(t.parent, n, N)
    if N >= 2 * DRAW_WAVES and kind != "flat":          # two nodes to a wave; in flat rows the root is drawn from all the time
        assert reached > 0
