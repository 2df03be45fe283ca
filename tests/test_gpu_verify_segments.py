"""GPU parity of the verification walk at the edges of the row sizes it is built for (2, 8 and 16 segments of 2048 tokens):
many rejected siblings, whose tokens lie in all parts of the row, and last tokens drawn from rows that end inside, at and
just past a segment."""
import numpy as np
import pytest

from helpers import verify_in_full

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


@pytest.fixture(scope="module")
def dy():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2410_11744_amd as m
    m.load_library()
    return m


@pytest.mark.parametrize("V", [90, 2047, 2052, 4095, 4096, 4097, 4100, 16383, 16384, 16385, 16388, 30721, 32768])
@pytest.mark.parametrize("bf16", [False, True])
def test_rejections_and_last_tokens(dy, V, bf16):
    rng = np.random.default_rng(V)
    nodes, temps, targets = (81, 40, 24), (1.0, 0.8, 1.0), (1.0, 0.7, 0.0)
    n = sum(nodes)
    draft = (rng.standard_normal((n, V)) * 1.5).astype(np.float32)
    target = (rng.standard_normal((n, V)) * 1.5).astype(np.float32)          # nothing to do with the draft: most children are rejected
    if bf16:
        draft, target = (torch.from_numpy(x).to(torch.bfloat16).float().numpy() for x in (draft, target))
    batch = dy.Batch.from_sizes(nodes)
    # a root whose children's tokens lie all over the row (first, last and segment edges among them); the fourth child has four of its own
    parent, token = [], []
    for c in nodes:
        edges = sorted({t for t in (0, V - 1, 2047, 2048, 4095, 4096, V // 2) if t < V})
        rest = [t for t in rng.permutation(V) if t not in edges]
        toks = (edges + rest)[:c - 5]
        rng.shuffle(toks)
        parent.append([-1] + [0] * (c - 5) + [4] * 4)
        token.append([-1] + [int(t) for t in toks] + [int(t) for t in rng.permutation(V)[:4]])
    first, after, rank, depth = [], [], [], []
    for p in parent:
        f, a, r, d, last = [-1] * len(p), [-1] * len(p), [0] * len(p), [0] * len(p), {}
        for i, q in enumerate(p):
            if q < 0:
                continue
            d[i] = d[q] + 1
            if q in last:
                a[last[q]] = i
                r[i] = r[last[q]] + 1
            else:
                f[q] = i
            last[q] = i
        first.append(f), after.append(a), rank.append(r), depth.append(d)
    whole = lambda xs: torch.tensor([x for y in xs for x in y], dtype=torch.int32, device="cuda")
    tree = dy.Tree(whole(parent), whole(token), whole(rank), whole(first), whole(after), whole(depth))
    trees = [tuple(np.array(x, np.int32) for x in t) for t in zip(token, first, after)]
    dt = torch.bfloat16 if bf16 else torch.float32
    dd, tg = torch.from_numpy(draft).cuda().to(dt), torch.from_numpy(target).cuda().to(dt)
    for seed in range(4):
        verify_in_full(lambda sd: dy.verify(dd, tg, batch, tree, temps, targets, sd), batch, trees, draft, target, temps, targets, seed)
