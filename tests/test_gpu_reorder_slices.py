"""dyspec_dfs_reorder on both sides of the line between workgroups of 64 and of 256 rows (512 workgroups of 64 rows over
the batch, counted with its widest tree): trees, rows never attached and links that are no tree, sizes at the edges of
a slice and of a mask word.  Whole numbers: equality with the walk written out."""
import numpy as np
import pytest

import test_gpu_reorder_forms as every

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n_seq,widest", [(16, 2048), (17, 2048), (64, 512), (64, 513)])
def test_slices(monkeypatch, n_seq, widest):
    def batch(name, rng):
        edges = [widest, widest, 1, 63, 64, 65, 127, 129, 255, 256, 257, 320, 511, 13]
        sizes = edges + [int(rng.integers(1, 300)) for _ in range(n_seq - len(edges))]
        out = []
        for s, n in enumerate(sizes):
            par = every.random_parents(n, rng) if s % 5 else np.arange(-1, n - 1)
            if s % 4 == 1 and n > 40:                       # the last rows are not attached
                par[n - 20:] = -1
            par, fc, ns = every.links(par, rng)
            if s % 4 == 3:
                [par, fc, ns][s % 3][int(rng.integers(0, n))] = int(rng.integers(-3, n + 3))
            out.append((par, fc, ns))
        return out

    monkeypatch.setattr(every, "forms", batch)
    every.test_every_form_of_links(f"{n_seq} sequences, {widest} rows", n_seq + widest)


@pytest.mark.parametrize("widest", [5, 6, 7])
@pytest.mark.parametrize("wrong", [False, True])
def test_smallest_doubled(monkeypatch, widest, wrong):
    """Either side of the size up to which one lane walks the links, every tree of a few shapes, and with one link wrong."""
    def batch(name, rng):
        out = []
        for s in range(24):
            n = widest if s % 3 == 0 else int(rng.integers(1, widest + 1))
            par, fc, ns = every.links([every.random_parents(n, rng), np.arange(-1, n - 1), np.array([-1] + [0] * (n - 1)),
                                       np.where(rng.random(n) < 0.3, -1, every.random_parents(n, rng))][s % 4], rng)
            if wrong:
                [par, fc, ns][int(rng.integers(0, 3))][int(rng.integers(0, n))] = int(rng.integers(-3, n + 3))
            out.append((par, fc, ns))
        return out

    monkeypatch.setattr(every, "forms", batch)
    every.test_every_form_of_links(f"widest {widest}", widest + 100 * wrong)
