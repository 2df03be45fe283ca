"""dyspec_build_tree_threshold against the oracle where one wave's draws from a row in LDS can go wrong: vocabularies
around a leaf (32 tokens), a group (512) and a sweep of the workgroup (4096), draws around 64 (written out
64 at a time), rows that run empty, weights over many orders of magnitude.

Values: a value is a product of factors 1 - R, each computed with an absolute error of 2^-53 (rounding of R and of the
difference).  No factor is below the value, so with values >= t the relative error is below 100 x 2^-52 / t where R comes
close to 1: 2e-7 for the peaked table at t = 1e-7, inside the comparison's 1e-6 (at t = 1e-12 it would not be)."""
import threading

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


@pytest.mark.parametrize("threads", [1, 8, 24])
def test_calls_at_the_same_time(threads):
    """Each thread on a stream of its own, trees of different depths: every call gets the levels of its own tree,
    also where more calls run than the library has host memory for (8)."""
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2410_11744_amd as dy
    sizes, temps, times = ([16, 200], [1], [64, 3, 500], [400]), (0.8,), 12
    x = torch.from_numpy(np.random.default_rng(5).standard_normal((700, 1000)).astype(np.float32) * 3).cuda()
    jobs = []
    for k in range(threads):
        batch = dy.Batch.from_sizes(sizes[k % 4])
        jobs.append((x[k:k + batch.total_nodes].clone(), batch, (0.004, 0.05, 0.3)[k % 3], 70 + k))

    def build(job):
        d, batch, t, seed = job
        built, levels = dy.build_tree_threshold(d, batch, temps * batch.n_seq, t, seed)
        return levels, built.n_built.cpu().tolist(), built.tree.token.cpu().tolist(), built.tree.parent.cpu().tolist()

    want = [build(j) for j in jobs]
    wrong = []

    def work(k):
        try:
            with torch.cuda.stream(torch.cuda.Stream()):
                for _ in range(times):
                    if build(jobs[k]) != want[k]:
                        wrong.append(k)
        except Exception as e:          # reported by the main thread
            wrong.append(repr(e))

    torch.cuda.synchronize()
    pool = [threading.Thread(target=work, args=(k,)) for k in range(threads)]
    for t in pool:
        t.start()
    for t in pool:
        t.join()
    assert not wrong
    torch.cuda.synchronize()


def test_refused_under_capture():
    """The call waits for its levels: on a capturing stream it returns an error, having launched nothing, and the
    capture goes on."""
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2410_11744_amd as dy
    batch = dy.Batch.from_sizes([32])
    x = torch.from_numpy(np.random.default_rng(6).standard_normal((32, 500)).astype(np.float32) * 3).cuda()
    want = dy.build_tree_threshold(x, batch, (0.8,), 0.05, 3)[0].tree.token.clone()
    y = torch.zeros(32, device="cuda")
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        with pytest.raises(dy.DyspecError):
            dy.build_tree_threshold(x, batch, (0.8,), 0.05, 3)
        y += 1.0
    for k in range(3):
        graph.replay()
        torch.cuda.synchronize()
        assert y.eq(k + 1.0).all()
        assert torch.equal(dy.build_tree_threshold(x, batch, (0.8,), 0.05, 3)[0].tree.token, want)
