"""dyspec_build_tree's helpers in use: they do take nodes over (a tree without them would be the same one, only later), beside other calls on
other streams, and recorded in a graph."""
import ctypes

import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

ARRAYS = ("parent", "token", "sib_rank", "first_child", "next_sibling", "depth")


@pytest.fixture(scope="module")
def dy():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2410_11744_amd as m
    m.load_library()
    m.init()
    return m


def arrays(built):
    return [getattr(built.tree, a) for a in ARRAYS] + [built.est_value, built.anc_mask, built.n_built]


def same(a, b):
    return all(torch.equal(x, y) for x, y in zip(arrays(a), arrays(b)))


def table(nodes, V, seed):
    """Rounded to bf16: many slots that are equal but for roundings, so that a tree shows who made its draws if that made a difference."""
    return (torch.randn(sum(nodes), V, generator=torch.Generator().manual_seed(seed)) * 3.0).bfloat16().float().cuda()


@pytest.mark.parametrize("V", [1000, 32000])
def test_the_hot_nodes_draws_are_a_helpers(dy, V):
    from paper_2410_11744_amd import binding
    lib = dy.load_library()
    N, hot = 300, 1
    x = torch.randn(N, V, generator=torch.Generator().manual_seed(V)) * 0.5
    x[0] = float("-inf")
    x[0, 5] = 0.0                                       # the root has one child, which has all the others
    x = x.cuda()
    batch = dy.Batch.from_sizes([N])
    tree, est = dy.Tree.empty(N, x.device), torch.empty(N, device=x.device)
    mask, nb = torch.empty((N, batch.mask_words), dtype=torch.int64, device=x.device), torch.empty(1, dtype=torch.int32, device=x.device)
    c, ct = batch._c(), tree._c()
    ws = torch.full((lib.dyspec_workspace_bytes(binding.WS_BUILD_TREE, ctypes.byref(c), V, 0, 0, 0) // 8,), float("nan"), dtype=torch.float64, device=x.device)
    st = lib.dyspec_build_tree(ctypes.c_void_p(x.data_ptr()), V, ctypes.byref(c), (ctypes.c_float * 1)(1.0), ctypes.c_uint64(7), ctypes.byref(ct),
                               ctypes.c_void_p(est.data_ptr()), ctypes.c_void_p(mask.data_ptr()), ctypes.c_void_p(nb.data_ptr()),
                               ctypes.c_void_p(ws.data_ptr()), ctypes.c_size_t(ws.numel() * 8), ctypes.c_void_p(torch.cuda.current_stream().cuda_stream))
    assert st == 0 and nb.item() == N
    draws = int((tree.parent == hot).sum())
    assert draws > 200
    # the mailboxes of the helpers (csrc/row_workspace.h: kRowSumDoubles, kMailOffset), as words: state, draws taken, key, key, draws told
    rows = ws.view(N, 24 + 32768 // 64).cpu()
    mails = rows[:8, 518:521].contiguous().view(torch.int32).tolist()
    told = [m[4] for m in mails if m[0] == 2 | hot << 2]
    assert len(told) == 1 and told[0] >= draws - 64, mails
    assert all(m[1] == -2 ** 31 for m in mails)         # the end of the tree has been told


def test_beside_calls_on_other_streams(dy):
    jobs = [([200, 64, 100], 8000, 1), ([64] * 28, 2000, 2), ([512], 32000, 3), ([30, 20], 4000, 4)]
    inputs = [(table(n, V, s), dy.Batch.from_sizes(n), s) for n, V, s in jobs]
    want = [dy.build_tree(x, b, 0.6, s) for x, b, s in inputs]
    nodes, V = (300, 90), 32000
    batch, temps = dy.Batch.from_sizes(nodes), (0.6, 1.0)
    draft = table(nodes, V, 5)
    target = draft + table(nodes, V, 6) / 3.0
    tree = dy.build_tree(draft, batch, temps, 5).tree
    want_v = dy.verify(draft, target, batch, tree, temps, temps, 11)
    streams = [torch.cuda.Stream() for _ in range(len(inputs) + 1)]
    torch.cuda.synchronize()
    for rep in range(10):
        got = []
        for (x, b, s), stream in zip(inputs, streams):
            with torch.cuda.stream(stream):
                got.append(dy.build_tree(x, b, 0.6, s))
        with torch.cuda.stream(streams[-1]):
            v = [dy.verify(draft, target, batch, tree, temps, temps, 11) for _ in range(3)]
        torch.cuda.synchronize()
        for k, (a, b) in enumerate(zip(got, want)):
            assert same(a, b), f"round {rep}, job {k}"
        for o in v:
            assert torch.equal(o.n_accepted, want_v.n_accepted) and torch.equal(o.final_token, want_v.final_token)
            assert torch.equal(o.row_stats, want_v.row_stats) and torch.equal(o.accept_ratio, want_v.accept_ratio)


@pytest.mark.parametrize("nodes,V", [([512], 32000), ([64] * 28, 2001), ([100, 17, 1, 64], 1000)])
def test_replays_of_a_recorded_build(dy, nodes, V):
    x, batch = table(nodes, V, V), dy.Batch.from_sizes(nodes)
    want = dy.build_tree(x, batch, 0.6, 9)
    other, small = table([300], 5000, 1), dy.Batch.from_sizes([300])
    side = torch.cuda.Stream()
    side.wait_stream(torch.cuda.current_stream())
    with torch.cuda.stream(side):
        dy.build_tree(x, batch, 0.6, 9)
    side.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph, stream=side):
        built = dy.build_tree(x, batch, 0.6, 9)
    first = None
    for rep in range(4):
        for t in arrays(built):
            t.zero_()
        torch.cuda.synchronize()
        graph.replay()
        torch.cuda.synchronize()
        assert same(built, want), f"replay {rep}"
        eager = dy.build_tree(other, small, 1.0, 3)         # the process's own work between replays
        first = first or eager
        assert same(eager, first) and torch.isfinite(eager.est_value.sum()).item()
