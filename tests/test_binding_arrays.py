"""What the binding hands to the library: temperatures as C arrays, the arrays of an empty tree (CPU)."""
import ctypes

import numpy as np
import pytest

torch = pytest.importorskip("torch")

from paper_2410_11744_amd import binding


@pytest.mark.parametrize("x,n", [(0.6, 1), (0.1, 5), (float("nan"), 2), (float("inf"), 2), (1e-42, 1), (1.0, 0), ([0.6, 1.0 / 3.0], 2), ((0.7,), 1),
                                 ([0.3], 4), ([1, 2.5], 2), (2, 3), (np.float32(0.6), 2), (np.array([0.25, 0.1]), 2), ([np.float64(0.1), 0.2], 2)])
def test_temperatures_as_numpy_makes_them(x, n):
    keep, p = binding._temps(x, n)
    want = np.broadcast_to(np.asarray(x, dtype=np.float32), (n,))
    p = ctypes.cast(p, ctypes.POINTER(ctypes.c_float))
    assert np.array([p[i] for i in range(n)], np.float32).tobytes() == want.tobytes()


@pytest.mark.parametrize("x,n", [([0.5, 0.6], 3), ((0.5, 0.6, 0.7), 2), ("abc", 1)])
def test_temperatures_of_another_length_are_refused(x, n):
    with pytest.raises(ValueError):
        binding._temps(x, n)


@pytest.mark.parametrize("n", [0, 1, 127, 128, 129, 1000])
def test_arrays_of_an_empty_tree(n):
    tree = binding.Tree.empty(n, "cpu")
    arrays = [getattr(tree, k) for k in ("parent", "token", "sib_rank", "first_child", "next_sibling", "depth")]
    for k, t in enumerate(arrays):
        assert t.shape == (n,) and t.dtype == torch.int32 and t.is_contiguous()
        assert (t.data_ptr() - arrays[0].data_ptr()) % 512 == 0
        t.fill_(k)
    for k, t in enumerate(arrays):
        assert bool((t == k).all())
