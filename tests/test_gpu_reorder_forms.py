"""GPU parity of dyspec_dfs_reorder over every form of links it accepts: trees (chains, stars, random, shuffled
siblings, rows never attached) and links that are no tree (inconsistent, cyclic, merging, out of range),
against the walk written out step by step.  Whole numbers: equality."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


def literal(parent, first_child, next_sibling):
    """Order and mask as the definition states them, one step after the other."""
    N = len(parent)
    link = lambda a: [int(v) if 0 <= v < N else -1 for v in a]
    par, fc, ns = link(parent), link(first_child), link(next_sibling)
    rank, order, cur, climbs = [-1] * N, [], 0, 0
    while cur >= 0 and len(order) < N and rank[cur] < 0:
        rank[cur] = len(order)
        order.append(cur)
        nxt = fc[cur]
        while nxt < 0 and cur >= 0 and climbs <= 2 * N:
            nxt = ns[cur]
            if nxt < 0:
                cur = par[cur]
                climbs += 1
        cur = nxt
    for i in range(N):
        if rank[i] < 0:
            rank[i] = len(order)
            order.append(i)
    new_parent = [rank[par[o]] if par[o] >= 0 else -1 for o in order]
    mask = np.zeros((N, (N + 63) // 64), np.uint64)
    for j in range(N):
        a, prev = j, N
        while 0 <= a < prev:
            mask[j, a >> 6] |= np.uint64(1) << np.uint64(a & 63)
            a, prev = new_parent[a], a
    named = lambda a: np.array([rank[a[o]] if a[o] >= 0 else -1 for o in order], np.int32)
    return np.array(order, np.int32), np.array(new_parent, np.int32), named(fc), named(ns), mask


def links(parent, rng=None):
    n = len(parent)
    kids = [[] for _ in range(n)]
    for i in range(n):
        if parent[i] >= 0:
            kids[parent[i]].append(i)
    fc, ns = np.full(n, -1, np.int32), np.full(n, -1, np.int32)
    for k in kids:
        if rng is not None:
            rng.shuffle(k)
        for a, b in zip(k, k[1:]):
            ns[a] = b
    for p, k in enumerate(kids):
        if k:
            fc[p] = k[0]
    return np.asarray(parent, np.int32), fc, ns


def random_parents(n, rng):
    return np.array([-1] + [int(rng.integers(0, i)) for i in range(1, n)], np.int32)


def forms(name, rng):
    if name == "trees":
        sizes = [1, 2, 3, 63, 64, 65, 255, 256, 257, 1023, 1025]
        return [links(random_parents(n, rng), rng) for n in sizes]
    if name.startswith("short"):                            # the widest tree on either side of the size from which positions are doubled
        n = 12 if name.startswith("short 12") else 13
        out = [links(random_parents(k, rng), rng) for k in (n, 1, 2, n, n - 1)] + [links(np.arange(-1, n - 1)), links(np.array([-1] + [0] * (n - 1)))]
        if name.endswith("no tree"):
            for par, fc, ns in out:
                for a in (par, fc, ns):
                    a[int(rng.integers(0, len(a)))] = int(rng.integers(-3, n + 3))
        return out
    if name == "largest":
        return [links(random_parents(2048, rng), rng)]
    if name == "chain":
        return [links(np.arange(-1, n - 1)) for n in (2048, 2, 1024, 700)]
    if name == "star":
        return [links(np.array([-1] + [0] * (n - 1))) for n in (2048, 257, 513)]
    if name == "never attached":
        out = []
        for n, live in ((2048, 900), (100, 1), (1030, 1029), (300, 256)):
            par = np.concatenate([random_parents(live, rng), np.full(n - live, -1, np.int32)])
            perm = np.concatenate([[0], 1 + rng.permutation(n - 1)])             # the loose rows lie among the others
            moved = np.empty(n, np.int32)
            moved[perm] = np.where(par >= 0, perm[par], -1)
            out.append(links(moved, rng))
        return out
    out = []
    for n in (1, 2, 5, 8, 64, 300, 1500, 2048):
        par, fc, ns = links(random_parents(n, rng), rng)
        kind = rng.integers(0, 4)
        for _ in range(int(rng.integers(1, 6))):
            a, b = int(rng.integers(0, n)), int(rng.integers(-3, n + 3))
            [par, fc, ns, [par, fc, ns][int(rng.integers(0, 3))]][kind][a] = b
        out.append((par, fc, ns))
    return out


@pytest.mark.parametrize("name,seed", [("trees", 0), ("largest", 1), ("chain", 2), ("star", 3), ("never attached", 4)]
                         + [("no tree", s) for s in range(5, 17)] + [("short 12", 17), ("short 13", 18)]
                         + [("short 12 no tree", s) for s in range(19, 25)] + [("short 13 no tree", s) for s in range(25, 29)])
def test_every_form_of_links(name, seed):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2410_11744_amd as dy
    rng = np.random.default_rng(seed)
    seqs = forms(name, rng)
    batch = dy.Batch.from_sizes([len(s[0]) for s in seqs])
    total = batch.total_nodes
    payload = [rng.integers(-5, 30000, total).astype(np.int32) for _ in range(3)]          # token, sib_rank, depth travel along
    mk = lambda a: torch.from_numpy(np.ascontiguousarray(a, dtype=np.int32)).cuda()
    cat = lambda k: np.concatenate([s[k] for s in seqs])
    re = dy.dfs_reorder(dy.Tree(mk(cat(0)), mk(payload[0]), mk(payload[1]), mk(cat(1)), mk(cat(2)), mk(payload[2])), batch)
    torch.cuda.synchronize()
    got = {k: getattr(re.tree, k).cpu().numpy() for k in ("parent", "token", "sib_rank", "first_child", "next_sibling", "depth")}
    order, mask = re.order.cpu().numpy(), re.anc_mask.cpu().numpy().view(np.uint64)
    for s, (par, fc, ns) in enumerate(seqs):
        a, b = int(batch.node_offset[s]), int(batch.node_offset[s + 1])
        o, p, f, n, m = literal(par, fc, ns)
        what = f"{name} seed {seed} sequence {s} of {b - a} rows"
        assert np.array_equal(order[a:b], o), what
        for key, want in (("parent", p), ("first_child", f), ("next_sibling", n), ("token", payload[0][a:b][o]),
                          ("sib_rank", payload[1][a:b][o]), ("depth", payload[2][a:b][o])):
            assert np.array_equal(got[key][a:b], want), f"{what}: {key}"
        assert np.array_equal(mask[a:b, :m.shape[1]], m) and not mask[a:b, m.shape[1]:].any(), f"{what}: mask"
