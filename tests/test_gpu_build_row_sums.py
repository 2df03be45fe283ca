"""The pass over the rows that the builder with a workspace starts with is built for rows of up to 4096, 16384 and 32768 tokens:
trees on both sides of those lines, and of the segments of 2048 tokens it skips, against the oracle (bit-exact topology) and the form
without a workspace (equal throughout)."""
import numpy as np
import pytest

from helpers import compare_trees, oracle_trees

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


@pytest.mark.parametrize("V", [7, 2048, 2049, 4092, 4095, 4096, 4097, 4100, 6145, 16380, 16383, 16384, 16385, 16388, 30720, 30721])
def test_rows_at_the_edges_of_the_segments(V):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2410_11744_amd as dy
    print(f"V={V}", flush=True)
    nodes, temps = (60, 9, 24), (0.6, 1.0, 0.8)
    rng = np.random.default_rng(V)
    d = (rng.standard_normal((sum(nodes), V)) * 2.5).astype(np.float32)
    # the ends of the row and of its segments hold much of the weight
    for t in {0, 2047, 2048, 4095, 4096, 16383, 16384, V - 1}:
        if t < V:
            d[:, t] += 7.0
    batch = dy.Batch.from_sizes(nodes)
    dd = torch.from_numpy(d).cuda()
    a = dy.build_tree(dd, batch, temps, 11)
    b = dy.build_tree(dd, batch, temps, 11, use_workspace=False)
    torch.cuda.synchronize()
    compare_trees(a, batch, oracle_trees(d, nodes, temps, 11))
    assert torch.equal(a.n_built, b.n_built)
    for name in ("parent", "token", "sib_rank", "first_child", "next_sibling", "depth"):
        assert torch.equal(getattr(a.tree, name), getattr(b.tree, name)), name
    assert torch.equal(a.anc_mask, b.anc_mask) and torch.equal(a.est_value, b.est_value)
