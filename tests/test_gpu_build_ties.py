"""The builder with a workspace keeps the 64 best open slots of a tree in order and makes that list again when it runs short.
Here it runs short: many slots of equal value (the one opened first is popped first), more than 64 of them open at a time, against
the form without a workspace, which compares all slots at every pop."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


# equal tokens: a value is a quotient of small integers, exact or rounded alike in both forms, so whole numbers must be equal
@pytest.mark.parametrize("V,live", [(2, 2), (3, 3), (8, 8), (64, 16), (129, 64), (1000, 4), (1000, 256)])
@pytest.mark.parametrize("nodes", [(64, 65, 66), (127, 128, 129, 130), (700,), (1024, 300)])
def test_more_equal_slots_than_the_list_holds(nodes, V, live):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2410_11744_amd as dy
    print(f"nodes={nodes} V={V} live={live}", flush=True)
    rng = np.random.default_rng(V + live + nodes[0])
    x = np.full((sum(nodes), V), -np.inf, np.float32)
    for row in x:
        row[rng.choice(V, live, replace=False)] = 0.25
    check_against_no_workspace(dy, x, nodes)


def check_against_no_workspace(dy, x, nodes):
    batch = dy.Batch.from_sizes(nodes)
    dd = torch.from_numpy(x).cuda()
    a = dy.build_tree(dd, batch, 1.0, 5)
    b = dy.build_tree(dd, batch, 1.0, 5, use_workspace=False)
    torch.cuda.synchronize()
    assert torch.equal(a.n_built, b.n_built)
    for name in ("parent", "token", "sib_rank", "first_child", "next_sibling", "depth"):
        assert torch.equal(getattr(a.tree, name), getattr(b.tree, name)), name
    assert torch.equal(a.anc_mask, b.anc_mask) and torch.equal(a.est_value, b.est_value)


# Many different slots of like size: the list is made again from those above a line.  With equal tokens, some rows of few and
# some of many, the line meets groups of equal values, of fewer than it can list and of more.
@pytest.mark.parametrize("V,live", [(1000, None), (4099, None), (1000, (2, 3, 5, 16, 40)), (300, (1, 2, 7)), (64, (2, 2, 2, 3, 64))])
@pytest.mark.parametrize("nodes", [(330, 400, 65), (960,), (1024, 1023)])
def test_more_slots_of_like_size_than_the_list_holds(nodes, V, live):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2410_11744_amd as dy
    print(f"nodes={nodes} V={V} live={live}", flush=True)
    rng = np.random.default_rng(V + nodes[0])
    if live is None:
        x = (10.0 * rng.standard_normal((sum(nodes), V))).astype(np.float32)
    else:
        x = np.full((sum(nodes), V), -np.inf, np.float32)
        for row in x:
            row[rng.choice(V, rng.choice(live), replace=False)] = 0.25
    check_against_no_workspace(dy, x, nodes)


# Nodes that are drawn from again and again, their slots equal or nearly so: the draws of several of them are popped together, up to the
# tree's last row, with the root's among them or with slots of single draws between them.
@pytest.mark.parametrize("hot", [1, 2, 5, 8, 13])
@pytest.mark.parametrize("live", [(40, 40), (300, 300), (300, 299), (299, 40)])
@pytest.mark.parametrize("nodes", [(64, 65), (71, 72, 73, 200), (333,), (1024,)])
def test_equal_slots_of_nodes_drawn_from_again_and_again(nodes, live, hot):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2410_11744_amd as dy
    print(f"nodes={nodes} live={live} hot={hot}", flush=True)
    V = 300
    rng = np.random.default_rng(hot + live[0] + nodes[0])
    x = np.full((sum(nodes), V), -np.inf, np.float32)
    base = 0
    for n in nodes:
        for i in range(n):
            x[base + i, rng.choice(V, hot if i == 0 else live[i % 2] if i <= 2 * hot else 2 + i % 3, replace=False)] = 0.25
        base += n
    check_against_no_workspace(dy, x, nodes)
