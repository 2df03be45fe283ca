"""GPU parity of the short-walk attention kernel against the fp64 oracle: every number of waves and parts it is launched
with, at the edges of its 32-row and 32-key blocks."""
import math

import numpy as np
import pytest

from test_gpu_tree_attn import make_case, run_and_compare

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


@pytest.fixture(scope="module")
def dy():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2410_11744_amd as m
    m.load_library()
    return m


# (waves, parts): the form that these sizes are there for, and take
@pytest.mark.parametrize("waves,parts,nodes,prefix,Hq,Hkv,d,shallow", [
    (8, 1, (1,), (65,), 8, 8, 128, False),              # one row, a block of one key, waves without any
    (8, 1, (1, 1, 3), (0, 1, 64), 4, 4, 128, False),    # a sequence without prefix, one whose blocks are of a key each
    (4, 1, (33,), (31,), 32, 32, 128, False),           # a second block of one row and one key, prefix short of a block
    (4, 1, (95,), (33,), 32, 32, 128, False),
    (4, 1, (768,), (129,), 8, 1, 128, False),           # four nodes to a row block
    (2, 1, (700,), (100,), 32, 32, 128, True),          # tree blocks left out, prefix blocks before them
    (2, 1, (1100,), (0,), 32, 32, 128, False),          # tree only
    (2, 1, (2048,), (0,), 8, 8, 128, False),            # all 64 tree blocks
    (8, 2, (70,), (1500,), 32, 32, 128, False),
    (8, 3, (33,), (4095,), 64, 8, 128, False),          # shares of unequal size
    (8, 7, (9,), (700,), 6, 2, 128, False),             # three heads to a row block's nodes
    (8, 4, (7, 1, 90), (2100, 800, 1500), 10, 2, 128, False),    # sequences of unequal length, five heads to a KV head
    (4, 1, (3, 50, 17), (300, 31, 0), 10, 2, 128, False),
    (4, 1, (5,), (40,), 8, 8, 64, False),
    (8, 1, (5,), (257,), 8, 8, 64, False),              # ten blocks, the last of the prefix a key
    (4, 1, (31, 5), (129, 1), 40, 40, 64, False),
    (8, 1, (65,), (300,), 8, 8, 64, False),
    (4, 1, (600,), (0,), 9, 3, 64, True),
    (4, 1, (2048,), (0,), 64, 64, 64, False),
    (8, 4, (64,), (2000,), 32, 32, 64, False),
    (8, 8, (7,), (2100,), 10, 2, 64, False),
])
def test_short_walks_match_the_oracle(dy, waves, parts, nodes, prefix, Hq, Hkv, d, shallow):
    from paper_2410_11744_amd import binding
    assert binding.tree_attn_form(dy.Batch.from_sizes(nodes, prefix), Hq, Hkv, d) == (waves, parts, 0)
    run_and_compare(dy, nodes, prefix, Hq, Hkv, d, "bf16", 70, shallow=shallow, max_rows=2500)


def test_rising_scores_raise_the_reference(dy):
    # the reference maximum of a wave is raised block after block
    run_and_compare(dy, (60,), (700,), 8, 8, 128, "bf16", 71, qscale=3.0, ramp=3.0)
    run_and_compare(dy, (40,), (200,), 32, 32, 64, "bf16", 72, qscale=4.0, ramp=2.0)


def test_rows_past_the_end_are_not_written(dy):
    """Row blocks reach past the last row of a sequence: the neighbour's rows and what lies behind the output stay."""
    nodes, prefix, Hq, Hkv = (3, 50, 17), (300, 31, 0), 10, 2
    batch = dy.Batch.from_sizes(nodes, prefix)
    q, kp, vp, kt, vt, mask = make_case(nodes, prefix, Hq, Hkv, 128, "bf16", 73)
    room = torch.full((sum(nodes) + 40, Hq, 128), 7.0, dtype=torch.bfloat16, device="cuda")
    out = room[20:20 + sum(nodes)]
    args = [t.cuda() for t in (q, kp, vp, kt, vt)]
    dy.tree_attn(*args, torch.from_numpy(mask.view(np.int64)).cuda(), batch, 1.0 / math.sqrt(128), out=out)
    torch.cuda.synchronize()
    assert (room[:20] == 7.0).all() and (room[20 + sum(nodes):] == 7.0).all()
    assert np.isfinite(out.float().cpu().numpy()).all()
