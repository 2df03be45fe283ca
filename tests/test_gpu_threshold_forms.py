"""dyspec_build_tree_threshold against the oracle where one wave's draws from a row in LDS can go wrong: vocabularies
around a leaf (32 tokens), a group (512) and a sweep of the workgroup (4096), draws around 64 (written out
64 at a time), rows that run empty, weights over many orders of magnitude.

Values: a value is a product of factors 1 - R, each computed with an absolute error of 2^-53 (rounding of R and of the
difference).  No factor is below the value, so with values >= t the relative error is below 100 x 2^-52 / t where R comes
close to 1: 2e-7 for the peaked table at t = 1e-7, inside the comparison's 1e-6 (at t = 1e-12 it would not be)."""
import numpy as np
import pytest

from helpers import next_seed
from test_gpu_threshold import compare_threshold_trees

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

CASES = [(kind, cap, V, t) for kind, cap, V, t in
         [("flat", c, 300, 1e-6) for c in (63, 64, 65, 66, 128, 129, 130)] +
         [("normal", 40, V, 0.01) for V in (1, 2, 31, 32, 33, 63, 511, 512, 513, 2047, 4095, 4096, 4097, 8191, 32764, 32767, 32768)] +
         [("few", 200, 700, 1e-9), ("few", 60, 4097, 1e-9), ("peaked", 100, 3000, 1e-7), ("normal", 1024, 1000, 1e-7)]]


@pytest.mark.parametrize("kind,cap,V,t", CASES)
def test_against_the_oracle(kind, cap, V, t):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2410_11744_amd as dy
    print(f"{kind} cap={cap} V={V} t={t}", flush=True)
    batch = dy.Batch.from_sizes([cap])
    for k in range(8):                      # a table with a decision at a margin below the bar is followed by the next one
        rng = np.random.default_rng(cap * 40000 + V + 7 * k)
        x = rng.standard_normal((cap, V)) * {"flat": 0.01, "normal": 3.0, "few": 3.0, "peaked": 60.0}[kind]
        if kind == "few":
            x[rng.random((cap, V)) < 0.99] = -np.inf
            x[:, 5] = 0.5
        x = x.astype(np.float32)
        seed = next_seed(cap + V, k)
        built, _ = dy.build_tree_threshold(torch.from_numpy(x).cuda(), batch, (0.8,), t, seed)
        torch.cuda.synchronize()
        if compare_threshold_trees(built, batch, x, (0.8,), (t,), seed) == 1:
            return
    raise AssertionError("no table in 8 had all margins above 1e-9")
