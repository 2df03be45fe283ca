"""A node's draws have the same bits whoever makes them: a tree must not depend on when its helpers (csrc/build_tree.hip) came.

Tables rounded to bf16 are full of children of one node with equal logits, whose slots are equal but for the roundings of the sums
behind them.  The same sequence in a batch of 29 has no helpers; where the root's row does not fit beside the tree's state in LDS
(499 rows of 32768 tokens and more), all its draws are made from memory, by the sums that helpers have to make as well."""
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

ARRAYS = ("parent", "token", "sib_rank", "first_child", "next_sibling", "depth")


@pytest.mark.parametrize("V", [32768, 32765])
@pytest.mark.parametrize("nodes", [500, 512, 1024])
@pytest.mark.parametrize("seed", [0, 1, 2, 3])
def test_with_helpers_as_without(V, nodes, seed):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2410_11744_amd as dy
    print(f"V={V} nodes={nodes} seed={seed}", flush=True)
    x = (torch.randn(nodes, V, generator=torch.Generator().manual_seed(seed)) * 3.0).bfloat16().float().cuda()
    alone, batch = dy.Batch.from_sizes([nodes]), dy.Batch.from_sizes([nodes] + [1] * 28)
    want = dy.build_tree(torch.cat([x, torch.zeros(28, V, device=x.device)]), batch, 0.6, seed)
    for _ in range(5):
        got = dy.build_tree(x, alone, 0.6, seed)
        for name in ARRAYS:
            assert torch.equal(getattr(got.tree, name), getattr(want.tree, name)[:nodes]), name
        assert torch.equal(got.est_value, want.est_value[:nodes]) and torch.equal(got.anc_mask, want.anc_mask[:nodes])
