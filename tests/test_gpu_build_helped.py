"""dyspec_build_tree where nodes that are drawn from again and again get a workgroup of their own (batches whose widest tree has 64 rows
or more, up to 28 sequences): one hot node or more of them than there are helpers, rows that run empty in a helper, tree sizes
and batch sizes on both sides of every line, repeated calls.  Against the oracle, decision for decision."""
import numpy as np
import pytest

from helpers import compare_trees, oracle_trees

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


@pytest.fixture(scope="module")
def dy():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2410_11744_amd as m
    m.load_library()
    return m


def check(dy, table, nodes, temps, seed):
    batch = dy.Batch.from_sizes(nodes)
    dev = torch.from_numpy(table).cuda()
    built = dy.build_tree(dev, batch, temps, seed)
    trees = oracle_trees(table, nodes, temps, seed)
    assert compare_trees(built, batch, trees) >= len(nodes) - len(nodes) // 16       # (a decision closer than the margin ends a comparison: hardly any)
    for _ in range(3):
        again = dy.build_tree(dev, batch, temps, seed)
        assert torch.equal(again.est_value, built.est_value) and torch.equal(again.anc_mask, built.anc_mask) and torch.equal(again.n_built, built.n_built)
        for name in ("parent", "token", "sib_rank", "first_child", "next_sibling", "depth"):
            assert torch.equal(getattr(again.tree, name), getattr(built.tree, name)), name
    return built, trees


@pytest.mark.parametrize("N", [63, 64, 65, 129, 300])
@pytest.mark.parametrize("V", [301, 4000, 32000])
@pytest.mark.parametrize("hot", [0, 1, 3, 11])
def test_hot_nodes(dy, N, V, hot):
    """`hot` nodes under the root share all draws (0: the root has them)."""
    rng = np.random.default_rng([N, V, hot])
    x = rng.standard_normal((N, V)).astype(np.float32)
    if hot:
        x[0] = -np.inf
        x[0, rng.permutation(V)[:hot]] = 3.0 + 0.1 * rng.standard_normal(hot).astype(np.float32)
    _, trees = check(dy, x, [N], [1.0], N + V)
    draws = np.bincount(trees[0].parent[1:trees[0].n_built], minlength=N)
    assert draws[1:].max() >= (N - 12) // hot // 2 if hot else draws[0] >= N // 2


@pytest.mark.parametrize("left", [9, 12, 13, 40, 77])
def test_rows_that_run_empty(dy, left):
    """The hot node's row has `left` tokens: it runs empty before, at or after the draws that its helper makes."""
    rng = np.random.default_rng(left)
    N, V = 200, 1000
    x = np.full((N, V), -np.inf, np.float32)
    for i in range(N):
        x[i, rng.permutation(V)[:left if i == 1 else 1 if i == 0 else 3]] = rng.standard_normal(left if i == 1 else 1 if i == 0 else 3).astype(np.float32)
    check(dy, x, [N], [1.0], left)


@pytest.mark.parametrize("n_seq", [2, 28, 29])
def test_ragged_batches(dy, n_seq):
    sizes = [64, 15, 16, 17, 1, 2, 63, 100, 8, 33]
    nodes = [sizes[s % len(sizes)] for s in range(n_seq)]
    temps = [0.6 if s % 3 else 1.0 for s in range(n_seq)]
    x = (np.random.default_rng(n_seq).standard_normal((sum(nodes), 2001)) * 3.0).astype(np.float32)
    check(dy, x, nodes, temps, n_seq)


@pytest.mark.parametrize("N,V", [(600, 32000), (1024, 32768), (1024, 1000)])
def test_wide_trees(dy, N, V):
    x = (np.random.default_rng(N + V).standard_normal((N, V)) * 3.0).astype(np.float32)
    check(dy, x, [N], [0.6], V)
