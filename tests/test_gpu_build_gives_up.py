"""A greedy build that gives up waiting for a draw says so in n_built and leaves a tree of the rows it had; the bound on
the waits is set from the host."""
import ctypes

import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


@pytest.mark.parametrize("nodes,V", [((40, 5, 1, 300), 1000), ((600,), 32000)])
def test_a_build_that_gives_up_is_told_from_one_that_ran_empty(nodes, V):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2410_11744_amd as dy
    from paper_2410_11744_amd import binding
    lib = dy.load_library()
    batch = dy.Batch.from_sizes(nodes)
    n = batch.total_nodes
    logits = torch.randn(n, V, generator=torch.Generator().manual_seed(V)).mul_(3).cuda()
    built = dy.build_tree(logits, batch, [0.6] * len(nodes), 7)
    assert built.n_built.tolist() == list(nodes)

    tree = dy.Tree.empty(n, logits.device)
    est = torch.empty(n, device=logits.device)
    mask = torch.empty((n, batch.mask_words), dtype=torch.int64, device=logits.device)
    nb = torch.empty(len(nodes), dtype=torch.int32, device=logits.device)
    c, ct = batch._c(), tree._c()
    temps = (ctypes.c_float * len(nodes))(*([0.6] * len(nodes)))
    ws = torch.empty(lib.dyspec_workspace_bytes(binding.WS_BUILD_TREE, ctypes.byref(c), V, 0, 0, 0) // 8, dtype=torch.float64, device=logits.device)

    def build(max_polls):
        st = lib.dyspec_build_tree_bounded(ctypes.c_void_p(logits.data_ptr()), V, ctypes.byref(c), temps, ctypes.c_uint64(7), ctypes.byref(ct),
                                           ctypes.c_void_p(est.data_ptr()), ctypes.c_void_p(mask.data_ptr()), ctypes.c_void_p(nb.data_ptr()),
                                           ctypes.c_void_p(ws.data_ptr()), ctypes.c_size_t(ws.numel() * 8), max_polls,
                                           ctypes.c_void_p(torch.cuda.current_stream().cuda_stream))
        assert st == 0

    build(0)                                             # gives up at the first draw
    assert nb.tolist() == [-1 if k > 1 else 1 for k in nodes]
    assert (tree.parent == -1).all() and (tree.token == -1).all() and (tree.first_child == -1).all()
    build(1 << 24)
    assert torch.equal(nb, built.n_built) and torch.equal(est, built.est_value) and torch.equal(mask, built.anc_mask)
    assert torch.equal(tree.parent, built.tree.parent) and torch.equal(tree.token, built.tree.token)
