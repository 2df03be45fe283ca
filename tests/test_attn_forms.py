"""Which matrix-core kernel and which parts a bf16 attention call is launched as (csrc/tree_attn_short.hip, tree_attn_short_plan): the
limits of every form over random shapes, and forms that do not exist refused on the host."""
import ctypes
import math
import random

import pytest

from paper_2410_11744_amd import binding

HEADS = [(32, 32), (40, 40), (64, 8), (8, 8), (8, 1), (9, 3), (6, 2), (1, 1), (2048, 2)]


def shapes(count, seed):
    rng = random.Random(seed)
    size = lambda a, b: int(round(math.exp(rng.uniform(math.log(a), math.log(b)))))
    for _ in range(count):
        seqs = rng.choice([1, 1, 2, 5, 16])
        n = [size(1, 2048) for _ in range(seqs)]
        p = [size(16, 8192) if rng.random() > 0.1 else rng.choice([0, 1, 33]) for _ in range(seqs)]
        yield (binding.Batch.from_sizes(n, p),) + rng.choice(HEADS) + (rng.choice([64, 128]),)


def workspace_bytes(batch, Hq, Hkv, d, layers=1):
    return binding.load_library().dyspec_tree_attn_layers_workspace_bytes(ctypes.byref(batch._c()), layers, Hq, Hkv, d)


def blocks(batch, G, rows):
    return sum(-(-G * int(n) // rows) for n in batch.node_offset[1:] - batch.node_offset[:-1])


def test_forms_stay_within_their_limits():
    seen = set()
    for batch, Hq, Hkv, d in shapes(6000, 1):
        G = Hq // Hkv
        if G > 1024:
            continue
        waves, parts, tree_part = binding.tree_attn_form(batch, Hq, Hkv, d)
        seen.add((d, waves, min(parts, 2), tree_part))
        assert waves in ((0, 2, 4, 8) if d == 128 else (0, 4, 8)) and 1 <= parts <= 8
        room = workspace_bytes(batch, Hq, Hkv, d) - 4096
        if parts > 1:           # parts are resident at once, a counter per group, their rows in the workspace
            groups = blocks(batch, G, 32 if waves else 128) * Hkv
            part = 32 * (d // 4 + 1) * 8 if waves else 4 * 64 * (d // 4 + 2) * 4
            assert groups * parts <= 256 and groups * parts * part <= room
            assert waves in (0, 8)
        assert not (waves and tree_part)
        # without a workspace nothing is split
        assert binding.tree_attn_form(batch, Hq, Hkv, d, use_workspace=False)[1:] == (1, 0)
    assert {f[1:] for f in seen if f[0] == 128} >= {(0, 1, 0), (0, 2, 0), (0, 2, 1), (2, 1, 0), (4, 1, 0), (8, 1, 0), (8, 2, 0)}
    assert {f[1:] for f in seen if f[0] == 64} >= {(0, 1, 0), (0, 2, 0), (4, 1, 0), (8, 1, 0), (8, 2, 0)}


def test_unsplit_calls_choose_alike_for_any_number_of_layers():
    for batch, Hq, Hkv, d in shapes(1500, 2):
        one = binding.tree_attn_form(batch, Hq, Hkv, d, use_workspace=False)
        for layers in (2, 7, 80):
            assert binding.tree_attn_form(batch, Hq, Hkv, d, layers, use_workspace=False) == one


# Measured: the kernel for long walks 40, 21 and 28 us, the one for short walks (8, 4 and 8 waves) 66, 34 and 41: a quarter
# more workgroups than CUs, where the other kernel has at most one to a CU.
@pytest.mark.parametrize("layers,nodes,prefix,Hq,Hkv,d", [(32, 23, 5271, 12, 2, 64), (8, 234, 2360, 5, 5, 64), (8, 45, 3349, 24, 8, 64)])
def test_stacked_calls_count_whole_workgroups(layers, nodes, prefix, Hq, Hkv, d):
    waves, parts, _ = binding.tree_attn_form(binding.Batch.from_sizes([nodes], [prefix]), Hq, Hkv, d, layers)
    assert waves == 0 and parts > 1


@pytest.mark.parametrize("layers", [1, 80])
@pytest.mark.parametrize("nodes,prefix,Hq,Hkv", [((25,), (0,), 64, 8), ((14,), (24,), 64, 8), ((19,), (54,), 16, 1), ((40, 64), (33, 64), 8, 8)])
def test_walks_of_four_blocks_of_keys_take_no_eight_waves(nodes, prefix, Hq, Hkv, layers):
    form = binding.tree_attn_form(binding.Batch.from_sizes(nodes, prefix), Hq, Hkv, 64, layers)
    assert form == (4, 1, 0)


# Measured: the kernel for long walks 73 and 70 us, two waves 91 and 88, four 47 and 45.
@pytest.mark.parametrize("layers,nodes,prefix,Hq,Hkv", [(1, (10, 1005, 32, 55, 29, 184, 153, 5), (437, 22, 6883, 178, 68, 63, 48, 34), 8, 1),
                                                        (2, (7, 314), (6731, 32), 16, 1)])
def test_one_long_walk_among_many_short_ones_takes_four_waves(layers, nodes, prefix, Hq, Hkv):
    assert binding.tree_attn_form(binding.Batch.from_sizes(nodes, prefix), Hq, Hkv, 128, layers) == (4, 1, 0)


def test_more_heads_to_a_kv_head_than_the_short_kernel_divides_by():
    batch = binding.Batch.from_sizes([3], [40])
    assert binding.tree_attn_form(batch, 1024, 1, 64)[0] != 0
    assert binding.tree_attn_form(batch, 1025, 1, 64)[0] == 0


@pytest.mark.parametrize("form,status", [((3, 1, 0), -3), ((1, 1, 0), -3), ((16, 1, 0), -3), ((2, 1, 0), -3),       # (2 waves: head_dim 128 only)
                                         ((4, 2, 0), -3), ((8, 9, 0), -3), ((8, 0, 0), -3), ((8, 2, 1), -3),
                                         ((0, 2, 0), -3), ((0, 0, 0), -3), ((0, 1, 1), -3)])
def test_forms_that_do_not_exist_are_refused(form, status):
    lib = binding.load_library()
    A = 0x7f0000001000
    batch = binding.Batch.from_sizes([40], [100])
    f = (ctypes.c_int32 * 3)(*form)
    p = ctypes.c_void_p
    call = lambda dtype, ws: lib.dyspec_tree_attn_in_form(f, p(A), p(A), p(A), p(A), p(A), p(A), ctypes.byref(batch._c()), 8, 8, 64, dtype,
                                                          ctypes.c_float(0.1), p(A), p(A if ws else None), ctypes.c_size_t(ws), p(None))
    assert call(binding.BF16, 8 << 20) == status
    f = (ctypes.c_int32 * 3)(8, 2, 0)
    assert call(binding.BF16, 0) == -3 and call(binding.BF16, 4096) == -3           # no room for the parts
    f = (ctypes.c_int32 * 3)(8, 1, 0)
    assert call(binding.F32, 0) == -3 and call(binding.BF16_WAVE, 0) == -3
