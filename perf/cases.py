"""The calls whose speed is followed: one speculative step and its parts, through the package's public functions.

Sizes are those of the benchmark's configurations (bench.py, paper_2410_11744_amd/synth.py), of the paper's random-tree
table and of the ranges the tests draw from.  A case is a dict of plain values; `kind` says which call it times:

  step        build_tree, tree_attn for every layer, verify: what a decode loop does once per step
  attention   tree_attn, `layers` calls on tensors of their own (prepared once, as a loop over layers does)
  stacked     tree_attn_layers, all layers in one call
  verify      vocabulary softmax of every tree row and the verification walk
  greedy      build_tree (Algorithm 1)
  threshold   build_tree_threshold (Algorithm 2)
  tree_only   dfs_reorder of a tree and tree_attn on the renamed tree, without a prefix

`nodes` and `prefix` are comma-separated sizes, one per sequence of the batch (a root counts as a node).
"""
import heapq
import math

import numpy as np
import torch

import paper_2410_11744_amd as dy

DEVICE = "cuda"
INTS = ("parent", "token", "sib_rank", "first_child", "next_sibling", "depth")


def listed():
    return [
        # the smallest step: one fp32 layer, 32 rows, 1000 tokens; launches and latency decide
        dict(name="step_tiny_f32", kind="step", nodes="32", prefix="128", q_heads=8, kv_heads=8, head_dim=64, layers=1,
             dtype="f32", vocab=1000, logits="normal", sigma=2.0, noise=0.5, temp="1.0", target_temp="1.0"),
        # a whole step of the 32-layer shape, budget 128: short attention calls one after the other
        dict(name="step_7b", kind="step", nodes="128", prefix="1024", q_heads=32, kv_heads=32, head_dim=128, layers=32,
             dtype="bf16", vocab=32000, logits="normal", sigma=3.0, noise=1.0, temp="0.6", target_temp="0.6"),
        # layers of the 40-head shape, budget 256: between bound by latency and by the matrix cores
        dict(name="attention_13b", kind="attention", nodes="256", prefix="2048", q_heads=40, kv_heads=40, head_dim=128, layers=8, dtype="bf16"),
        # layers of the headline shape, grouped heads, budget 512: bound by the matrix cores
        dict(name="attention_70b", kind="attention", nodes="512", prefix="4096", q_heads=64, kv_heads=8, head_dim=128, layers=4, dtype="bf16"),
        # a serving batch: eight sequences, no size a multiple of a tile; the largest attention call
        dict(name="attention_70b_ragged8", kind="attention", nodes="754,102,259,334,466,351,156,95",
             prefix="5832,6795,1186,6816,4385,4718,5542,3072", q_heads=64, kv_heads=8, head_dim=128, layers=2, dtype="bf16"),
        # a narrow tree behind a long prefix: the K/V stream from memory is the work
        dict(name="attention_70b_n32", kind="attention", nodes="32", prefix="4096", q_heads=64, kv_heads=8, head_dim=128, layers=8, dtype="bf16"),
        # the 32-layer shape with all layers in one call
        dict(name="stacked_7b", kind="stacked", nodes="128", prefix="1024", q_heads=32, kv_heads=32, head_dim=128, layers=32, dtype="bf16"),
        # verification at the headline shape: 131 MB of logits, then a short walk
        dict(name="verify_70b", kind="verify", nodes="512", vocab=32000, dtype="f32", logits="normal", sigma=3.0, noise=0.8,
             temp="0.6", target_temp="0.6"),
        # verification of the serving batch on bf16 tables, temperature-0 requests among the others, targets further from the draft
        dict(name="verify_ragged8_bf16", kind="verify", nodes="754,102,259,334,466,351,156,95", vocab=32000, dtype="bf16",
             logits="normal", sigma=3.0, noise=1.5, temp="0.6,0.6,0.6,0.6,1.0,1.0,1.0,1.0", target_temp="0.6,0.0,0.6,0.6,1.0,1.0,0.0,1.0"),
        # Algorithm 1 at the headline table
        dict(name="greedy_70b", kind="greedy", nodes="512", vocab=32000, logits="normal", sigma=3.0, temp="0.6"),
        # Algorithm 2 on Zipf-shaped rows, threshold about 1 / budget, capacity 1.5 times the budget
        dict(name="threshold_13b", kind="threshold", nodes="384", vocab=32000, logits="zipf", sigma=0.3, temp="1.0", threshold=1.0 / 256),
        # the last row of the paper's random-tree table: depth-first renaming and attention among the tree's own rows
        dict(name="tree_only_2048", kind="tree_only", nodes="2048", prefix="0", q_heads=64, kv_heads=64, head_dim=128, layers=1, dtype="bf16"),
    ]


def draw(rng):
    def size(lo, hi):                       # spread over the logarithm, odd values among them
        return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))

    def sizes(n, lo, hi):
        return [size(lo, hi) for _ in range(n)]

    text = lambda xs: ",".join(str(x) for x in xs)
    kind = rng.choice(["step", "attention", "attention", "attention", "stacked", "verify", "verify", "greedy", "threshold", "tree_only"])
    n_seq = rng.choice([1, 1, 1, 2, 4, 8])
    temps = [rng.choice([0.6, 1.0]) for _ in range(n_seq)]
    logits, sigma = rng.choice([("normal", 2.0), ("normal", 3.0), ("zipf", 0.3)])
    table = dict(vocab=rng.choice([1000, 32000, 32000, 32768, size(1000, 32768)]), logits=logits, sigma=sigma, temp=text(temps))
    q_heads, kv_heads = rng.choice([(32, 32), (40, 40), (64, 8)])
    heads = dict(q_heads=q_heads, kv_heads=kv_heads, head_dim=rng.choice([128, 128, 64]), dtype="bf16")
    if kind in ("attention", "stacked"):
        nodes, prefix = sizes(n_seq, 8, 768), sizes(n_seq, 64, 8192)
        flops = 4 * q_heads * heads["head_dim"] * sum(n * (p + n) for n, p in zip(nodes, prefix))
        layers = int(min(32 if kind == "stacked" else 8, 5e11 // flops, 2e8 // (sum(prefix) * kv_heads)))
        if layers < 1:                      # past the largest listed call: the first sequence alone
            nodes, prefix, layers = nodes[:1], prefix[:1], 1
        return dict(kind=kind, nodes=text(nodes), prefix=text(prefix), layers=layers, **heads)
    if kind == "step":
        if rng.random() < 0.3:
            heads = dict(q_heads=8, kv_heads=8, head_dim=64, dtype="f32")
            return dict(kind=kind, nodes=text(sizes(1, 8, 64)), prefix=text(sizes(1, 16, 256)), layers=1, noise=0.5,
                        target_temp=text(temps[:1]), **heads, **dict(table, temp=text(temps[:1]), vocab=size(500, 4000)))
        return dict(kind=kind, nodes=text(sizes(1, 16, 192)), prefix=text(sizes(1, 64, 1536)), layers=rng.choice([4, 8, 16]), noise=1.0,
                    target_temp=text(temps[:1]), **heads, **dict(table, temp=text(temps[:1])))
    if kind == "verify":
        targets = [t if rng.random() < 0.75 else 0.0 for t in temps]
        return dict(kind=kind, nodes=text(sizes(n_seq, 16, 768)), dtype=rng.choice(["f32", "bf16"]), noise=rng.choice([0.5, 0.8, 1.5, 2.0]),
                    target_temp=text(targets), **table)
    if kind == "greedy":
        return dict(kind=kind, nodes=text(sizes(n_seq, 16, 512)), **table)
    if kind == "threshold":
        budget = sizes(n_seq, 16, 340)
        return dict(kind=kind, nodes=text([b * 3 // 2 for b in budget]), threshold=1.0 / max(budget), **table)
    h = rng.choice([32, 64])
    return dict(kind=kind, nodes=text(sizes(1, 64, 2048)), prefix="0", q_heads=h, kv_heads=h, head_dim=128, layers=1, dtype="bf16")


# ---------------------------------------------------------------------------------------- inputs

def numbers(text, n=None):
    xs = [float(x) for x in str(text).split(",")]
    return xs * (n if n and len(xs) == 1 else 1)


def ints(text):
    return [int(x) for x in numbers(text)]


class Bag:
    """The state of a case: what a program holds before the call."""

    def __init__(self, **kw):
        self.__dict__.update(kw)


def generator(seed):
    g = torch.Generator(device=DEVICE)
    g.manual_seed(int(seed) * 1000003 + 17)
    return g


def normal(g, *shape):
    return torch.randn(shape, generator=g, device=DEVICE, dtype=torch.float32)


def draft_table(case, rows, g):
    """Draft logits fp32 [rows, vocab]: independent normal rows, or Zipf-shaped ones in a ranking of their own."""
    V = case["vocab"]
    x = normal(g, rows, V) * case["sigma"]
    if case["logits"] == "zipf":
        ranks = torch.argsort(torch.rand((rows, V), generator=g, device=DEVICE), dim=1)
        x += -1.1 * torch.log(torch.arange(1, V + 1, device=DEVICE, dtype=torch.float32))[ranks]
    return x


def grown_tree(n, rng):
    """Parents of a tree grown as Algorithm 1 grows one, with acceptance rates from a Beta law in place of a draft
    model's: early siblings get most of the budget, depth and width vary from node to node."""
    parent = np.full(n, -1, np.int32)
    rates = rng.beta(0.5, 1.5, n)
    heap, opened = [(-1.0, 0, 0)], 1
    for i in range(1, n):
        v, _, p = heapq.heappop(heap)
        parent[i] = p
        heapq.heappush(heap, (v * (1.0 - rates[i]), opened, p))
        heapq.heappush(heap, (v * rates[i], opened + 1, i))
        opened += 2
    return parent


def random_tree(n, rng):
    """The paper's random tree: the parent of a node is any earlier node."""
    parent = np.full(n, -1, np.int32)
    parent[1:] = [rng.integers(0, i) for i in range(1, n)]
    return parent


def linked(parent):
    """first_child, next_sibling, depth, rank among the siblings; children in index order."""
    n = len(parent)
    first, after, last = (np.full(n, -1, np.int32) for _ in range(3))
    depth, rank = np.zeros(n, np.int32), np.zeros(n, np.int32)
    for i in range(1, n):
        p = parent[i]
        depth[i] = depth[p] + 1
        if last[p] < 0:
            first[p] = i
        else:
            after[last[p]] = i
            rank[i] = rank[last[p]] + 1
        last[p] = i
    return first, after, depth, rank


def visible(parent):
    """Boolean [n, n]: row j sees itself and its ancestors."""
    n = len(parent)
    m = np.zeros((n, n), bool)
    for j in range(n):
        if parent[j] >= 0:
            m[j] = m[parent[j]]
        m[j, j] = True
    return m


def mask_words(parents):
    """Ancestor masks of a batch as the library stores them: 64 keys to a word, int64 [rows, words]."""
    words = (max(len(p) for p in parents) + 63) // 64
    rows = []
    for p in parents:
        wide = np.zeros((len(p), 64 * words), bool)
        wide[:, : len(p)] = visible(p)
        rows.append(np.packbits(wide, axis=1, bitorder="little").view(np.int64))
    return torch.from_numpy(np.concatenate(rows)).to(DEVICE)


def case_trees(case, seed):
    rng = np.random.default_rng([int(seed), 29])
    grow = random_tree if case["kind"] == "tree_only" else grown_tree
    return [grow(n, rng) for n in ints(case["nodes"])]


def attention_tensors(case, g):
    """q, k_prefix, v_prefix, k_tree, v_tree ~ N(0, 1), each [layers, rows, heads, head_dim]."""
    dt = torch.float32 if case["dtype"] == "f32" else torch.bfloat16
    N, P, L, d = sum(ints(case["nodes"])), sum(ints(case["prefix"])), case["layers"], case["head_dim"]
    rows = [(N, case["q_heads"]), (P, case["kv_heads"]), (P, case["kv_heads"]), (N, case["kv_heads"]), (N, case["kv_heads"])]
    out = [torch.empty((L, r, h, d), dtype=dt, device=DEVICE) for r, h in rows]
    for layer in range(L):
        for t in out:
            t[layer].copy_(normal(g, *t.shape[1:]))
    return out


def sampled_tokens(draft, parent, temp, offset, g):
    """A token for every node but the root: the children of a node are a sample without replacement of the softmax of
    its draft row (largest perturbed logits first, which is the order of the draws)."""
    token = torch.full((len(parent),), -1, dtype=torch.int32, device=DEVICE)
    for p in sorted(set(parent[1:].tolist())):
        kids = np.flatnonzero(parent == p)
        u = torch.rand(draft.shape[1], generator=g, device=DEVICE).clamp_(1e-7, 1.0 - 1e-7)
        keys = draft[offset + p].float() / temp - torch.log(-torch.log(u))
        token[torch.from_numpy(kids).to(DEVICE)] = torch.topk(keys, len(kids)).indices.int()
    return token


def clear_verify_output(batch):
    out = dy.VerifyOutput.empty(batch, DEVICE)
    for t in (out.row_stats, out.accept_ratio, out.accepted_nodes, out.n_accepted, out.final_token, out.min_margin):
        t.zero_()                           # accepted_nodes is written as far as the path goes
    return out


def inputs(case, seed):
    """The case's tensors and trees, from the seed alone (what prepare() and exact() share)."""
    kind, g = case["kind"], generator(seed)
    nodes = ints(case["nodes"])
    s = Bag(seed=int(seed), nodes=nodes, prefix=ints(case.get("prefix", ",".join("0" * len(nodes)))))
    if "layers" in case:
        s.tensors = attention_tensors(case, g)
        s.scale = float(np.float32(1.0 / math.sqrt(case["head_dim"])))
    if "vocab" in case:
        s.temps = numbers(case["temp"], len(nodes))
        s.draft = draft_table(case, sum(nodes), g)
    if kind in ("step", "verify"):
        s.target_temps = numbers(case["target_temp"], len(nodes))
        s.target = s.draft + normal(g, *s.draft.shape) * case["noise"]
    if kind in ("attention", "stacked", "verify", "tree_only"):
        s.parents = case_trees(case, seed)
    if kind == "verify":
        if case["dtype"] == "bf16":
            s.draft, s.target = s.draft.to(torch.bfloat16), s.target.to(torch.bfloat16)
        offset, tokens = 0, []
        for p, t in zip(s.parents, s.temps):
            tokens.append(sampled_tokens(s.draft, p, t, offset, g))
            offset += len(p)
        s.tokens = torch.cat(tokens)
    return s


def device_tree(parents, tokens=None):
    links = [linked(p) for p in parents]
    whole = lambda xs: torch.from_numpy(np.concatenate(xs).astype(np.int32)).to(DEVICE)
    token = tokens if tokens is not None else whole([np.arange(len(p)) - 1 for p in parents])
    return dy.Tree(whole(parents), token, whole([x[3] for x in links]), whole([x[0] for x in links]), whole([x[1] for x in links]),
                   whole([x[2] for x in links]))


def prepare(case, seed):
    kind, s = case["kind"], inputs(case, seed)
    s.kind = kind
    s.batch = dy.Batch.from_sizes(s.nodes, s.prefix)
    if kind == "tree_only":                 # token-aligned tensors already follow the renamed order
        s.tree = device_tree(s.parents)
        s.out = torch.empty_like(s.tensors[0][0])
    elif kind in ("attention", "stacked", "step"):
        s.out = torch.empty_like(s.tensors[0])
        s.layers = [tuple(t[layer] for t in s.tensors) for layer in range(case["layers"])]
    if kind in ("attention", "stacked"):
        s.mask = mask_words(s.parents)
    if kind == "attention":
        s.calls = [dy.tree_attn_call(*one, s.mask, s.batch, s.scale, out=s.out[layer]) for layer, one in enumerate(s.layers)]
    if kind == "verify":
        s.tree = device_tree(s.parents, s.tokens)
    if kind in ("verify", "step"):
        s.verified = clear_verify_output(s.batch)
    if kind == "threshold":
        s.threshold = case["threshold"]
    return s


# ---------------------------------------------------------------------------------------- the calls

def tree_arrays(tree):
    return {k: getattr(tree, k) for k in INTS}


def built_arrays(built):
    return dict(tree_arrays(built.tree), est_value=built.est_value, anc_mask=built.anc_mask, n_built=built.n_built)


def verify_arrays(v):
    return {k: getattr(v, k) for k in ("row_stats", "accept_ratio", "accepted_nodes", "n_accepted", "final_token", "min_margin")}


def run(s):
    if s.kind == "attention":
        for call in s.calls:
            call()
        return s.out
    if s.kind == "stacked":
        return dy.tree_attn_layers(*s.tensors, s.mask, s.batch, s.scale, out=s.out)
    if s.kind == "verify":
        return verify_arrays(dy.verify(s.draft, s.target, s.batch, s.tree, s.temps, s.target_temps, s.seed, out=s.verified))
    if s.kind == "greedy":
        return built_arrays(dy.build_tree(s.draft, s.batch, s.temps, s.seed))
    if s.kind == "threshold":
        built, levels = dy.build_tree_threshold(s.draft, s.batch, s.temps, s.threshold, s.seed)
        return dict(built_arrays(built), levels=levels)
    if s.kind == "tree_only":
        re = dy.dfs_reorder(s.tree, s.batch)
        q, kp, vp, kt, vt = (t[0] for t in s.tensors)
        out = dy.tree_attn(q, kp, vp, kt, vt, re.anc_mask, s.batch, s.scale, out=s.out)
        return dict(tree_arrays(re.tree), order=re.order, anc_mask=re.anc_mask, out=out)
    built = dy.build_tree(s.draft, s.batch, s.temps, s.seed)
    for layer, one in enumerate(s.layers):
        dy.tree_attn(*one, built.anc_mask, s.batch, s.scale, out=s.out[layer])
    v = dy.verify(s.draft, s.target, s.batch, built.tree, s.temps, s.target_temps, s.seed, out=s.verified)
    return dict(built=built_arrays(built), out=s.out, verified=verify_arrays(v))


# ---------------------------------------------------------------------------------------- what the path cannot do without

def work(case):
    nodes = ints(case["nodes"])
    N, total = sum(nodes), {"bytes": 0.0, "flops": 0.0}
    if "layers" in case:
        prefix, L, d = ints(case["prefix"]), case["layers"], case["head_dim"]
        size = 4 if case["dtype"] == "f32" else 2
        rows_q, rows_kv = 2 * N * case["q_heads"], 2 * (sum(prefix) + N) * case["kv_heads"]
        total["bytes"] += L * size * d * (rows_q + rows_kv) + 8 * N * ((max(nodes) + 63) // 64)
        # every row sees the prefix, itself and the root; what it sees of the tree beyond that depends on the tree
        total["flops"] += L * 4.0 * d * case["q_heads"] * sum(n * p + 2 * n - 1 for n, p in zip(nodes, prefix))
    if "vocab" in case:
        tables = 2 if case["kind"] in ("step", "verify") else 1
        size = 2 if case.get("dtype") == "bf16" and case["kind"] == "verify" else 4
        values = float(tables * N * case["vocab"])
        total["bytes"] += size * values + 48.0 * N
        total["flops"] += 4.0 * values      # scale, subtract, exponential, sum
    if case["kind"] == "tree_only":
        total["bytes"] += 4.0 * N * 13
    return total


def tolerance(case):
    if case["kind"] == "verify":            # fp32 sums of 32000 exponentials; ratios of rows renormalised child by child
        return {"rel": 1e-5, "max": 1e-3}
    if case["kind"] in ("greedy", "threshold"):      # decided in fp64, values stored in fp32
        return {"rel": 5e-7, "max": 2e-6}
    if case["dtype"] == "f32":
        return {"rel": 1e-5, "max": 1e-3}
    return {"rel": 1e-2, "max": 6e-2}       # bf16 tensors and probabilities, fp32 accumulation


# ---------------------------------------------------------------------------------------- the same in 64 bits

def exact_attention(s, parents):
    q, kp, vp, kt, vt = s.tensors
    L, _, Hq, d = q.shape
    Hkv = kt.shape[2]
    G = Hq // Hkv
    out = torch.empty(q.shape, dtype=torch.float64, device=DEVICE)
    a = b = 0
    for n, P, parent in zip(s.nodes, s.prefix, parents):
        hidden = torch.from_numpy(np.repeat(~visible(parent), G, axis=0)).to(DEVICE)
        for layer in range(L):
            for h in range(Hkv):
                rows = q[layer, a:a + n, h * G:(h + 1) * G].reshape(n * G, d).double()
                k = torch.cat([kp[layer, b:b + P, h], kt[layer, a:a + n, h]]).double()
                v = torch.cat([vp[layer, b:b + P, h], vt[layer, a:a + n, h]]).double()
                score = torch.mm(rows, k.t().contiguous()) * s.scale
                score[:, P:].masked_fill_(hidden, -math.inf)
                out[layer, a:a + n, h * G:(h + 1) * G] = torch.mm(torch.softmax(score, dim=1), v).reshape(n, G, d)
        a, b = a + n, b + P
    return out


def exact_stats(s):
    """[rows, 4]: maximum and sum of exponentials of draft / T, then of target / T (temperature 0: largest logit, its index)."""
    out = torch.empty((sum(s.nodes), 4), dtype=torch.float64, device=DEVICE)
    a = 0
    for n, td, tt in zip(s.nodes, s.temps, s.target_temps):
        for table, t, col in ((s.draft, td, 0), (s.target, tt, 2)):
            for r in range(a, a + n, 256):
                x = table[r:min(r + 256, a + n)].double()
                top, at = x.max(dim=1)
                if t == 0.0:
                    at = (x == top[:, None]).int().argmax(dim=1).double()
                else:
                    t32 = float(np.float32(t))
                    top, at = top / t32, torch.exp((x - top[:, None]) / t32).sum(dim=1)
                out[r:r + len(x), col], out[r:r + len(x), col + 1] = top, at
        a += n
    return out


def philox(counter, key):
    """Philox4x32-10 (Salmon et al., SC'11)."""
    c, k = list(counter), list(key)
    for _ in range(10):
        a, b = 0xD2511F53 * c[0], 0xCD9E8D57 * c[2]
        c = [(b >> 32) ^ c[1] ^ k[0], b & 0xFFFFFFFF, (a >> 32) ^ c[3] ^ k[1], a & 0xFFFFFFFF]
        k = [(k[0] + 0x9E3779B9) & 0xFFFFFFFF, (k[1] + 0xBB67AE85) & 0xFFFFFFFF]
    return c


class Sampler:
    """The draft rows of one sequence: draws without replacement by inverse CDF, named by the path of sibling ranks."""

    def __init__(self, table, temp, seed, seq):
        self.table, self.temp, self.key = table, float(np.float32(temp)), (seed & 0xFFFFFFFF, seed >> 32)
        self.path, self.weights = {0: (seq, 0)}, {}

    def child(self, node, of, rank):
        self.path[node] = tuple(philox((*self.path[of], rank, 0), self.key)[:2])

    def draw(self, node, rank):
        """Token and its probability in what is left of the node's row; None when nothing is left."""
        w = self.weights.get(node)
        if w is None:
            x = self.table[node].astype(np.float64) / self.temp
            w = self.weights[node] = np.exp(x - x.max())
        c = np.cumsum(w)
        if not c[-1] > 0.0:
            return None
        u = (philox((*self.path[node], rank, 1), self.key)[0] >> 8) / 16777216.0
        y = min(int(np.searchsorted(c, u * c[-1], side="right")), int(np.flatnonzero(w)[-1]))
        r = 1.0 if np.count_nonzero(w) == 1 else w[y] / c[-1]
        w[y] = 0.0
        return y, r


def exact_greedy(table, n, temp, seed, seq):
    s = Sampler(table, temp, seed, seq)
    parent, value, kids = np.full(n, -1, np.int32), np.zeros(n), [0] * n
    value[0] = 1.0
    heap, opened = [(-1.0, 0, 0)], 1
    for i in range(1, n):
        if not heap:
            break
        v, _, p = heapq.heappop(heap)
        got = s.draw(p, kids[p])
        if got is None:
            break
        parent[i], value[i] = p, -v
        s.child(i, p, kids[p])
        kids[p] += 1
        for w, node in ((v * (1.0 - got[1]), p), (v * got[1], i)):
            if w < 0.0:
                heapq.heappush(heap, (w, opened, node))
                opened += 1
    return parent, value


def exact_threshold(table, n, temp, t, seed, seq):
    s = Sampler(table, temp, seed, seq)
    value, own = np.zeros(n), np.zeros(n)
    value[0] = own[0] = 1.0
    level, rows = [0], 1
    while level and rows < n:
        made = []
        for p in level:
            v, rank = own[p], 0
            while v >= t and rows < n:
                got = s.draw(p, rank)
                if got is None:
                    break
                value[rows], own[rows] = v, v * got[1]
                s.child(rows, p, rank)
                made.append(rows)
                v, rank, rows = v * (1.0 - got[1]), rank + 1, rows + 1
        level = made
    return value


def exact(case, seed):
    kind, s = case["kind"], inputs(case, seed)
    if kind in ("attention", "stacked"):
        return exact_attention(s, s.parents)
    if kind == "tree_only":                 # the tensors already follow the depth-first order of the tree
        parent, n = s.parents[0], s.nodes[0]
        first, after, _, _ = linked(parent)
        order, stack = [], [0]
        while stack:
            node = stack.pop()
            order.append(node)
            kids, c = [], first[node]
            while c >= 0:
                kids.append(c)
                c = after[c]
            stack.extend(reversed(kids))
        rank = np.empty(n, np.int64)
        rank[order] = np.arange(n)
        renamed = np.array([rank[parent[o]] if parent[o] >= 0 else -1 for o in order])
        return {**{k: None for k in INTS}, "order": None, "anc_mask": None, "out": exact_attention(s, [renamed])[0]}
    if kind == "verify":
        return {"row_stats": exact_stats(s), "accept_ratio": None, "accepted_nodes": None, "n_accepted": None, "final_token": None,
                "min_margin": None}
    parents, values, a = [], [], 0
    table = s.draft.cpu().numpy()
    for seq, (n, t) in enumerate(zip(s.nodes, s.temps)):
        if kind == "threshold":
            values.append(exact_threshold(table[a:a + n], n, t, case["threshold"], s.seed, seq))
        else:
            parent, value = exact_greedy(table[a:a + n], n, t, s.seed, seq)
            parents.append(parent)
            values.append(value)
        a += n
    built = {**{k: None for k in INTS}, "est_value": np.concatenate(values), "anc_mask": None, "n_built": None}
    if kind == "threshold":
        return dict(built, levels=None)
    if kind == "greedy":
        return built
    return {"built": built, "out": exact_attention(s, parents),
            "verified": {"row_stats": exact_stats(s), "accept_ratio": None, "accepted_nodes": None, "n_accepted": None, "final_token": None,
                         "min_margin": None}}
