"""dyspec_build_tree with a workspace (draws made ahead by waves of their own) against the form without one, over the
shapes of trees and tables it accepts: whole numbers and fp32 values must be equal.  Both forms sum the same fp64
weights in different orders, so a decision could differ only where its margin is near 1e-13, and a stored
fp32 value only where the fp64 one lies that close to a rounding boundary.  (Many small trees at a time, where the
order in which nodes are served matters most: test_gpu_build_small.py.)"""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


def normal(rng, rows, V, sigma=3.0):
    return (rng.standard_normal((rows, V)) * sigma).astype(np.float32)


def table(kind, nodes, V, rng):
    rows = sum(nodes)
    x = normal(rng, rows, V)
    if kind == "chain":                     # one token holds nearly all: every new node is popped next
        x[np.arange(rows), rng.integers(0, V, rows)] += 40.0
    elif kind == "child":                   # the root has one child worth having, which takes all the draws
        x[0] = -50.0
        x[0, V // 2] = 20.0
    elif kind == "equal":                   # slots of equal value: the one opened first
        x[:] = 1.5
    elif kind == "two":                     # two equal tokens in a row, the rest impossible
        x[:] = -np.inf
        x[:, [V // 3, V - 1]] = 0.25
    elif kind == "few":                     # rows run empty: some tokens possible, rows without any among them
        x[rng.random((rows, V)) < 0.98] = -np.inf
        x[::5] = -np.inf
        x[0] = normal(rng, 1, V)[0]
    elif kind == "peaked":                  # weights over many orders of magnitude
        x = x * 20.0
    elif kind == "odd":                     # values a table can hold
        x[1::3, : V // 2] = np.nan
        x[2::3, 0] = np.float32(3e38)
    return x.astype(np.float32)


CASES = [("normal", n, v) for n, v in (((2,), 1), ((1,), 5), ((3,), 2), ((40,), 31), ((40,), 33), ((64,), 511), ((65,), 512), ((66,), 513),
                                       ((127, 128, 129), 4097), ((130,), 4096), ((511, 512), 2050), ((513,), 1000), ((1024,), 3000),
                                       ((1024, 5), 32000), ((556,), 32000), ((557,), 32000), ((489,), 32768), ((490,), 32768),
                                       ((300,), 32767), ((895, 896, 897, 898), 700))]
CASES += [(k, n, v) for k in ("chain", "child", "equal", "few", "peaked", "odd")
          for n, v in (((60,), 64), ((200, 31), 1000), ((140,), 2047), ((260,), 32000), ((900,), 32768))]
CASES += [(k, n, v) for k in ("normal", "chain", "few", "odd")      # both sides of the size from which the root's row is kept in LDS
          for n, v in (((8, 9), 1000), ((9,), 5), ((9,), 32001), ((10,), 5), ((9, 10), 129), ((10,), 32000), ((11, 2), 2050))]
CASES += [("two", (9,), 40), ("two", (1024,), 600), ("equal", (1024,), 2), ("equal", (600,), 4)]


@pytest.mark.parametrize("kind,nodes,V", CASES)
def test_same_tree_as_without_a_workspace(kind, nodes, V):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2410_11744_amd as dy
    print(f"{kind} nodes={nodes} V={V}", flush=True)
    rng = np.random.default_rng(len(nodes) * 1000 + nodes[0] + V)
    batch = dy.Batch.from_sizes(nodes)
    dd = torch.from_numpy(table(kind, nodes, V, rng)).cuda()
    temps = [0.6 if s % 2 == 0 else 1.0 for s in range(len(nodes))]
    a = dy.build_tree(dd, batch, temps, 17)
    b = dy.build_tree(dd, batch, temps, 17, use_workspace=False)
    torch.cuda.synchronize()
    assert torch.equal(a.n_built, b.n_built)
    for name in ("parent", "token", "sib_rank", "first_child", "next_sibling", "depth"):
        assert torch.equal(getattr(a.tree, name), getattr(b.tree, name)), name
    assert torch.equal(a.anc_mask, b.anc_mask)
    assert torch.equal(a.est_value, b.est_value)


@pytest.mark.parametrize("nodes,V", [((8,), 5), ((40, 20), 1000), ((64,), 2047), ((600,), 32000)])
def test_temperature_so_small_that_the_maximum_over_it_is_rounded(nodes, V):
    """The largest logit is 20 everywhere: 20 / 1e-20 is rounded down by 65536, its weight is infinite, and it is still
    all that there is: one chain of those tokens, as in the oracle, where 20 / 1e-20 less itself is 0."""
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2410_11744_amd as dy
    from helpers import oracle_trees
    rng = np.random.default_rng(V)
    x = normal(rng, sum(nodes), V)
    x = np.minimum(x, 19.0).astype(np.float32)
    x[np.arange(len(x)), rng.integers(0, V, len(x))] = 20.0
    batch = dy.Batch.from_sizes(nodes)
    a = dy.build_tree(torch.from_numpy(x).cuda(), batch, [1e-20] * len(nodes), 3)
    for s, t in enumerate(oracle_trees(x, nodes, [1e-20] * len(nodes), 3)):
        rows = slice(int(batch.node_offset[s]), int(batch.node_offset[s + 1]))
        assert a.n_built[s].item() == t.n_built == nodes[s]
        for name in ("parent", "token", "sib_rank", "first_child", "next_sibling", "depth"):
            np.testing.assert_array_equal(getattr(a.tree, name).cpu().numpy()[rows], getattr(t, name), err_msg=name)
        np.testing.assert_array_equal(a.est_value.cpu().numpy()[rows], t.est_value.astype(np.float32))
