"""dyspec_build_tree with a workspace and without helpers: batches of more than 28 sequences, whose trees are the size of those that have
helpers in smaller batches.  Against the form without a workspace, as in test_gpu_build_forms.py: both sides of the line where the
root's row fits into LDS beside the tree's state (32000 tokens: 564 rows, 32768: 498), nodes drawn from again and again by their own waves."""
import numpy as np
import pytest

from test_gpu_build_forms import table

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


@pytest.mark.parametrize("kind", ["normal", "child", "equal", "few", "peaked", "chain"])
@pytest.mark.parametrize("N,V", [(564, 32000), (565, 32000), (498, 32768), (499, 32768), (64, 32000), (200, 2050), (1024, 1001)])
def test_as_without_a_workspace(N, V, kind):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2410_11744_amd as dy
    print(f"N={N} V={V} kind={kind}", flush=True)
    nodes = [N] + [1] * 20 + [2, 5, 10, 20, 1, 3, 1, 1]
    rng = np.random.default_rng(N + V)
    batch = dy.Batch.from_sizes(nodes)
    dd = torch.from_numpy(table(kind, nodes, V, rng)).cuda()
    # Equal logits, equal slots: at temperature 1 every weight is exactly 1 and a sum of up to 2^53 of them exact in any order, so the forms have
    # the same slots.  At 0.6 a weight is exp(fma(1.5, 1 / 0.6, -m)) = 1 - 2^-53, and each form's own roundings order the slots.
    temp = 1.0 if kind == "equal" else 0.6
    a = dy.build_tree(dd, batch, temp, 17)
    b = dy.build_tree(dd, batch, temp, 17, use_workspace=False)
    torch.cuda.synchronize()
    assert torch.equal(a.n_built, b.n_built)
    for name in ("parent", "token", "sib_rank", "first_child", "next_sibling", "depth"):
        assert torch.equal(getattr(a.tree, name), getattr(b.tree, name)), name
    assert torch.equal(a.anc_mask, b.anc_mask) and torch.equal(a.est_value, b.est_value)
