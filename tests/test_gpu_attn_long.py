"""GPU parity of the long-walk attention kernel (csrc/tree_attn_mfma.hip) against the fp64 oracle.  Sizes at its edges mostly choose the
other kernel by themselves, so it is asked for by form; sizes that choose it are checked to do so."""
import math

import numpy as np
import pytest

from helpers import ATTN_TOL, attn_in_form, oracle_attention_rows
from test_gpu_random_shapes import HEADS
from test_gpu_tree_attn import make_case

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


@pytest.fixture(scope="module")
def dy():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2410_11744_amd as m
    m.load_library()
    return m


def check(dy, form, nodes, prefix, Hq, Hkv, d, seed, max_rows=2000, **kw):
    print(f"long attn form={form} nodes={nodes} prefix={prefix} H={Hq}/{Hkv} d={d} seed={seed}", flush=True)
    batch = dy.Batch.from_sizes(nodes, prefix)
    q, kp, vp, kt, vt, mask = make_case(nodes, prefix, Hq, Hkv, d, "bf16", seed, **kw)
    scale = 1.0 / math.sqrt(d)
    dev = [t.cuda() if t.numel() else torch.empty((1,) + tuple(t.shape[1:]), dtype=t.dtype, device="cuda") for t in (q, kp, vp, kt, vt)]
    out = attn_in_form(dy, form, *dev, torch.from_numpy(mask.view(np.int64)).cuda(), batch, scale)
    got = out.float().cpu().numpy()
    assert np.isfinite(got).all()
    host = [t.float().numpy() for t in (q, kp, vp, kt, vt)]
    rng = np.random.default_rng(seed + 1)
    for s, n in enumerate(nodes):
        pick = np.arange(n * Hq) if n * Hq <= max_rows else rng.choice(n * Hq, max_rows, replace=False)
        rj, rh = np.divmod(pick, Hq)
        want = oracle_attention_rows(*host, mask, batch, s, scale, rj, rh)
        assert np.abs(got[int(batch.node_offset[s]) + rj, rh] - want).max() <= ATTN_TOL["bf16"]
    return out, dev, mask, batch, scale


@pytest.mark.parametrize("nodes,prefix,Hq,Hkv,d,kw", [
    ((32,), (128,), 8, 8, 64, {}),
    ((100,), (1000,), 8, 2, 128, {}),                   # ragged prefix tile and ragged tree tile
    ((512,), (333,), 16, 2, 128, {}),
    ((70,), (0,), 4, 2, 128, {}),                       # no prefix
    ((1,), (65,), 8, 8, 128, {}),                       # one row
    ((1, 1, 3), (0, 1, 64), 4, 4, 64, {}),
    ((64, 7, 200, 1), (100, 1, 513, 64), 8, 2, 128, {}),
    ((300,), (64,), 6, 2, 64, {}),                      # three heads to a KV head
    ((259, 10), (130, 31), 9, 3, 128, {}),
    ((768,), (129,), 8, 1, 128, {}),
    ((1024,), (64 * 9 + 5,), 8, 1, 128, {}),
    ((1024, 300), (512, 700), 8, 2, 128, dict(shallow=True)),       # tree tiles left out
    ((1024, 640), (0, 100), 4, 4, 128, dict(shallow=True)),
    ((900,), (130,), 8, 8, 64, dict(shallow=True)),
    ((2048,), (0,), 2, 2, 128, {}),                     # all 32 tree tiles
    ((130,), (70,), 4, 2, 128, dict(chain=True)),
    ((130,), (70,), 4, 2, 64, dict(chain=True)),
    ((96,), (2048,), 8, 2, 128, dict(qscale=3.0, ramp=3.0)),        # the running maximum is raised many times
    ((200,), (640,), 4, 4, 64, dict(qscale=4.0, ramp=2.0)),
])
def test_unsplit_walks_match_the_oracle(dy, nodes, prefix, Hq, Hkv, d, kw):
    check(dy, (0, 1, 0), nodes, prefix, Hq, Hkv, d, 50, **kw)


@pytest.mark.parametrize("parts,tree_part,by_itself,nodes,prefix,Hq,Hkv,d", [
    (8, 0, False, (32,), (4096,), 64, 8, 128),
    (4, 0, False, (128,), (1024 + 37,), 8, 8, 128),     # ragged last prefix tile, the last part holds the tree alone
    (4, 0, False, (40, 9), (64 * 22, 64 * 17 + 1), 4, 2, 128),      # uneven shares
    (5, 1, False, (128,), (1024,), 32, 32, 128),        # a part for the two tree tiles
    (3, 1, False, (128, 64), (1024, 640), 8, 8, 128),
    (8, 1, True, (118,), (5043,), 32, 32, 128),
    (3, 0, True, (256,), (2048,), 40, 40, 128),
    (6, 1, True, (58, 214, 76), (1425, 1802, 2843), 9, 3, 128),
    (8, 0, False, (70,), (2048 + 5,), 8, 8, 64),
    (3, 1, False, (128, 33), (1024, 700), 4, 4, 64),
    (8, 0, True, (43,), (4637,), 64, 8, 64),
    (6, 0, True, (98,), (1939,), 40, 40, 64),
    (6, 1, True, (128,), (2238,), 40, 40, 64),
    (3, 1, True, (16, 117), (3810, 639), 40, 40, 64),
    (5, 1, True, (296, 185, 244), (1653, 1020, 2395), 6, 2, 64),
])
def test_split_walks_match_the_oracle_and_the_unsplit_walk(dy, parts, tree_part, by_itself, nodes, prefix, Hq, Hkv, d):
    from paper_2410_11744_amd import binding
    form = (0, parts, tree_part)
    out, dev, mask, batch, scale = check(dy, form, nodes, prefix, Hq, Hkv, d, 60)
    mask_dev = torch.from_numpy(mask.view(np.int64)).cuda()
    whole = attn_in_form(dy, (0, 1, 0), *dev, mask_dev, batch, scale)
    # the same products; each part's share of a row is rounded to bf16 before the merge
    assert float((out.float() - whole.float()).abs().max()) <= 2.0 ** -6
    for _ in range(3):          # parts are summed in their order whoever merges them
        assert torch.equal(attn_in_form(dy, form, *dev, mask_dev, batch, scale).view(torch.int16), out.view(torch.int16))
    if by_itself:
        assert binding.tree_attn_form(batch, Hq, Hkv, d) == form
        assert torch.equal(dy.tree_attn(*dev, mask_dev, batch, scale).view(torch.int16), out.view(torch.int16))


@pytest.mark.parametrize("seed", range(16))
def test_random_shapes(dy, seed):
    rng = np.random.default_rng(9000 + seed)
    n_seq = int(rng.integers(1, 6))
    nodes = tuple(int(x) for x in rng.integers(1, 260, n_seq))
    prefix = tuple(int(x) for x in rng.choice([0, 1, 17, 64, 65, 127, 128, 300, 513, 700], n_seq))
    Hq, Hkv = HEADS[int(rng.integers(0, len(HEADS)))]
    check(dy, (0, 1, 0), nodes, prefix, Hq, Hkv, int(rng.choice([64, 128])), 9100 + seed, max_rows=1200, shallow=bool(rng.integers(0, 2)))
