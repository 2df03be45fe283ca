"""The pointers that the binding takes from a tree it has just made, and a batch whose sizes are changed between calls."""
import pytest

torch = pytest.importorskip("torch")

from paper_2410_11744_amd import binding


@pytest.mark.gpu
@pytest.mark.parametrize("n", [0, 1, 127, 128, 129, 1000])
def test_pointers_of_a_new_tree(n):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    tree, c = binding.Tree._empty_c(n, torch.device("cuda"))
    assert bytes(c) == bytes(tree._c())


def test_a_new_tree_on_the_host_is_refused():
    with pytest.raises(ValueError):
        binding.Tree._empty_c(4, "cpu")


def test_a_batch_is_looked_at_anew():
    batch = binding.Batch.from_sizes([3, 64], [5, 7])
    memo = batch._memo()
    first = batch._c(memo)
    assert batch._mask_words(memo) == batch.mask_words == 1 and batch._c() is first
    batch.node_offset[2] = 3 + 65
    memo = batch._memo()
    assert batch._c(memo) is not first and batch._c(memo).node_offset[2] == 68 and batch._mask_words(memo) == batch.mask_words == 2
