"""Statistics of rows that are not made of whole 16-byte pieces (they begin at any value, their end is read from their last 16 bytes) and
the walk's loads of such rows: vocabularies on both sides of a piece, of a batch of pieces and of a segment, the largest logit
in the piece that overlaps the one before, rows of -inf and NaN.  Against 64 bits: a row's maximum over T is rounded once (2^-24 of it), and of its
sum, weights of an exponent known to 2^-23 of itself, added up in chains of at most 32."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

SIZES = [4, 5, 7, 8, 9, 12, 15, 17, 1021, 1023, 2047, 2049, 2052, 4095, 4099, 8190, 16379, 16385, 16388, 16391, 32001, 32765, 32767]


def verified(x, y, t, target_t, emit_bonus=True):
    import paper_2410_11744_amd as dy
    n, V = x.shape
    batch = dy.Batch.from_sizes([n])
    i32 = lambda a: torch.tensor(a, dtype=torch.int32, device="cuda")
    tree = dy.Tree(i32([-1] + [0] * (n - 1)), i32([-1] + [i % V for i in range(n - 1)]), i32([0] + list(range(n - 1))), i32([1] + [-1] * (n - 1)),
                   i32([-1] + list(range(2, n)) + [-1]), i32([0] + [1] * (n - 1)))
    out = dy.verify(x, y, batch, tree, [t], [target_t], 7, emit_bonus=emit_bonus)
    torch.cuda.synchronize()
    return out


@pytest.mark.parametrize("V", SIZES)
@pytest.mark.parametrize("dtype", ["float32", "bfloat16"])
@pytest.mark.parametrize("target_t", [0.0, 0.6])
def test_statistics(V, dtype, target_t):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    print(f"V={V} {dtype} {target_t}", flush=True)
    rng = np.random.default_rng(V)
    n, t = 9, 0.6
    x = (3.0 * rng.standard_normal((2, n, V))).astype(np.float32)
    for i in range(n):                          # the largest logit in the last piece, at its start and end, and just before
        x[:, i, max(V - 1 - i, 0)] = 21.0
    x, y = (torch.from_numpy(a).to(getattr(torch, dtype)) for a in x)
    stats = verified(x.cuda(), y.cuda(), t, target_t).row_stats.cpu().double()
    for col, table, temp in ((0, x, t), (2, y, target_t)):
        z = table.double()
        if temp == 0.0:
            assert torch.equal(stats[:, col], z.max(1).values) and torch.equal(stats[:, col + 1].long(), z.argmax(1))
            continue
        z = z / np.float64(np.float32(temp))
        top = z.max(1).values
        assert ((stats[:, col] - top).abs() <= 2.0 ** -22 * top.abs()).all()
        total = torch.exp(z - stats[:, col:col + 1]).sum(1)
        spread = (z.max(1).values - z.min(1).values).clamp(max=20.0)
        assert ((stats[:, col + 1] / total - 1).abs() <= 2.0 ** -22 * (spread + 32)).all()


@pytest.mark.parametrize("V", [5, 9, 1021, 16387, 32767])
@pytest.mark.parametrize("dtype", ["float32", "bfloat16"])
@pytest.mark.parametrize("where", ["first", "last", "overlap"])
def test_one_nan_or_nothing(V, dtype, where):
    """A row of -inf with one NaN has no sum, wherever it lies; a row of -inf with one finite value has that value's."""
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    print(f"V={V} {dtype} {where}", flush=True)
    at = {"first": 0, "last": V - 1, "overlap": V - 4}[where]
    x = torch.full((3, V), -np.inf)
    x[0, at] = np.nan
    x[1, at] = 1.5
    x[2] = 0.25
    x[2, at] = np.nan
    x = x.to(getattr(torch, dtype)).cuda()
    s = verified(x, x.clone(), 1.0, 1.0).row_stats.cpu()
    assert torch.isnan(s[0, 1]) and torch.isnan(s[0, 3]) and torch.isnan(s[2, 1]) and torch.isnan(s[2, 3])
    assert s[1].tolist() == [1.5, 1.0, 1.5, 1.0]


@pytest.mark.parametrize("V", [7, 1023, 4099, 16385, 16390, 32767])
@pytest.mark.parametrize("dtype", ["float32", "bfloat16"])
def test_last_token_from_the_end_of_a_row(V, dtype):
    """All weight of the target on one of the last tokens, none of the draft's there: every child is refused, that token comes out."""
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    for back in range(4):
        x = torch.zeros((4, V))
        y = torch.full((4, V), -np.inf)
        y[:, V - 1 - back] = 0.0
        x[:, V - 1 - back] = -np.inf
        out = verified(x.to(getattr(torch, dtype)).cuda(), y.to(getattr(torch, dtype)).cuda(), 1.0, 1.0)
        assert out.final_token.item() == V - 1 - back and out.n_accepted.item() == 0
