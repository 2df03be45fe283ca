"""Shared pieces of the GPU parity tests: oracle runs per sequence and comparisons.

Tolerances (derived from the arithmetic of each side):
  * tree build: both sides decide in fp64, so every arg-max and inverse-CDF decision whose
    relative margin in the oracle is >= BUILD_MARGIN must agree bit for bit; est_value is
    stored as fp32 (rel 2^-24).
  * verify: the GPU works in fp32.  Row statistics within 1e-5 relative; accept ratios
    within RATIO_RTOL; accept / final-token decisions must agree when the oracle's margin is
    >= DECISION_MARGIN (1e-5, the bar the benchmark definition states).
  * attention: max abs error 2e-2 for bf16 tensors, 1e-5 (relative to the fp64 oracle, on
    outputs of order 1) for fp32 tensors.
"""
from __future__ import annotations

import numpy as np

import oracle

BUILD_MARGIN = 1e-9
DECISION_MARGIN = 1e-5
RATIO_RTOL = 2e-4
ATTN_TOL = {"bf16": 2e-2, "f32": 1e-5}


def f32(x) -> float:
    """The double that equals the fp32 value the GPU library receives."""
    return float(np.float32(x))


def oracle_trees(draft, cfg_nodes, temps, seed):
    """Oracle build per sequence; returns list of oracle.Tree."""
    out, off = [], 0
    for s, n in enumerate(cfg_nodes):
        out.append(oracle.build_tree(draft[off:off + n], n, f32(temps[s]), seed, seq=s))
        off += n
    return out


def compare_trees(built, batch, trees, check_values=True):
    """GPU BuiltTrees vs oracle trees.  Returns number of sequences compared in full."""
    g = {k: getattr(built.tree, k).cpu().numpy() for k in
         ("parent", "token", "sib_rank", "first_child", "next_sibling", "depth")}
    est = built.est_value.cpu().numpy()
    mask = built.anc_mask.cpu().numpy().view(np.uint64)
    nb = built.n_built.cpu().numpy()
    full = 0
    for s, t in enumerate(trees):
        a, b = int(batch.node_offset[s]), int(batch.node_offset[s + 1])
        n = b - a
        margins = np.minimum(t.margin_pop[1:t.n_built], t.margin_cdf[1:t.n_built])
        low = np.nonzero(margins < BUILD_MARGIN)[0]
        upto = n if low.size == 0 else int(low[0]) + 1        # nodes before the first doubtful decision
        if low.size == 0:
            full += 1
            assert nb[s] == t.n_built
        for k in ("parent", "token", "sib_rank", "depth"):
            np.testing.assert_array_equal(g[k][a:a + upto], getattr(t, k)[:upto], err_msg=f"seq {s} {k}")
        if low.size == 0:
            for k in ("first_child", "next_sibling"):
                np.testing.assert_array_equal(g[k][a:b], getattr(t, k), err_msg=f"seq {s} {k}")
            words = t.mask.shape[1]
            np.testing.assert_array_equal(mask[a:b, :words], t.mask, err_msg=f"seq {s} mask")
            assert not mask[a:b, words:].any()
            if check_values:
                np.testing.assert_allclose(est[a:b], t.est_value, rtol=1e-6, atol=1e-30)
    return full


def compare_verify(out, batch, trees, draft, target, temps_d, temps_t, seed, emit_bonus=True):
    """GPU VerifyOutput vs oracle.  `trees` = list of (token, first_child, next_sibling)
    or oracle.Tree.  Returns (sequences whose path was compared, sequences skipped)."""
    stats = out.row_stats.cpu().numpy()
    ratio = out.accept_ratio.cpu().numpy()
    acc = out.accepted_nodes.cpu().numpy()
    na = out.n_accepted.cpu().numpy()
    fin = out.final_token.cpu().numpy()
    mm = out.min_margin.cpu().numpy()
    compared = skipped = 0
    for s, t in enumerate(trees):
        a, b = int(batch.node_offset[s]), int(batch.node_offset[s + 1])
        tok, fc, ns = (t.token, t.first_child, t.next_sibling) if hasattr(t, "token") else t
        td, tt = f32(temps_d[s]), f32(temps_t[s])
        d, tg = draft[a:b], target[a:b]
        want_stats = oracle.softmax_stats(d, tg, td, tt)
        np.testing.assert_allclose(stats[a:b], want_stats, rtol=1e-5, atol=1e-6, err_msg=f"seq {s} stats")
        want_ratio = oracle.accept_ratio_all(d, tg, tok, fc, ns, td, tt)
        got = ratio[a:b]
        tested = got >= 0                      # -1 marks children behind an exhausted draft
        fin_mask = np.isfinite(want_ratio) & tested
        np.testing.assert_allclose(got[fin_mask], want_ratio[fin_mask], rtol=RATIO_RTOL, atol=1e-7,
                                   err_msg=f"seq {s} accept_ratio")
        assert np.all(np.isinf(got[tested & ~np.isfinite(want_ratio)]))
        r = oracle.verify(d, tg, tok, fc, ns, td, tt, seed, seq=s, emit_bonus=emit_bonus)
        if r.min_accept_margin < DECISION_MARGIN:
            skipped += 1
            continue
        assert na[s] == r.n_accepted, f"seq {s}: accepted {na[s]} vs oracle {r.n_accepted}"
        np.testing.assert_array_equal(acc[a:a + na[s]], r.accepted_nodes, err_msg=f"seq {s} path")
        if np.isfinite(r.min_accept_margin):
            assert mm[s] == np.float32(mm[s]) and abs(mm[s] - r.min_accept_margin) < 1e-4 * max(1.0, r.min_accept_margin)
        if r.resid_margin >= DECISION_MARGIN or r.final_token < 0:
            assert fin[s] == r.final_token, f"seq {s}: final token {fin[s]} vs oracle {r.final_token}"
        compared += 1
    return compared, skipped


def next_seed(seed, k):
    """k-th seed tried for a case: the case's own seed first, then fresh ones (a case in which the
    oracle took a decision at a margin below the bar is generated again with the next seed)."""
    return seed + 7919 * k


def build_in_full(dy, draft_dev, draft_host, batch, nodes, temps, seed, tries=8):
    """dyspec_build_tree compared with the oracle in full.  A seed at which some oracle decision has
    a margin below BUILD_MARGIN (its trees are still compared up to that decision) is followed by the
    next one, until every sequence was compared row by row.  Returns (built, oracle trees, seed)."""
    import torch
    for k in range(tries):
        sd = next_seed(seed, k)
        built = dy.build_tree(draft_dev, batch, temps, sd)
        torch.cuda.synchronize()
        trees = oracle_trees(draft_host, nodes, temps, sd)
        if compare_trees(built, batch, trees) == len(nodes):
            return built, trees, sd
    raise AssertionError(f"no seed in {tries} tries gave build margins >= {BUILD_MARGIN} in every sequence")


def verify_in_full(run, batch, trees, draft, target, temps_d, temps_t, seed, emit_bonus=True, tries=8):
    """run(seed) -> VerifyOutput of the GPU library; compared with the oracle.  A seed at which some
    sequence's walk has an acceptance margin below DECISION_MARGIN (statistics and ratios are still
    compared) is followed by the next one, until the accepted path of EVERY sequence was compared.
    Returns (output, seed)."""
    import torch
    for k in range(tries):
        sd = next_seed(seed, k)
        out = run(sd)
        torch.cuda.synchronize()
        compared, skipped = compare_verify(out, batch, trees, draft, target, temps_d, temps_t, sd, emit_bonus=emit_bonus)
        assert compared + skipped == len(trees)
        if skipped == 0:
            return out, sd
    raise AssertionError(f"no seed in {tries} tries gave acceptance margins >= {DECISION_MARGIN} in every sequence")


def oracle_attention_rows(q, kp, vp, kt, vt, mask_u64, batch, seq, scale, rows_j, rows_h):
    """fp64 oracle on sampled (node, head) rows of one sequence; inputs are host fp32 arrays."""
    a, b = int(batch.node_offset[seq]), int(batch.node_offset[seq + 1])
    k0 = int(batch.kv_offset[seq])
    P = int(batch.prefix_len[seq])
    words = (b - a + 63) // 64
    return oracle.tree_attn_rows(q[a:b], kp[k0:k0 + P], vp[k0:k0 + P], kt[a:b], vt[a:b],
                                 np.ascontiguousarray(mask_u64[a:b, :words]), scale, rows_j, rows_h)


def attn_in_form(dy, form, q, kp, vp, kt, vt, mask, batch, scale):
    """dyspec_tree_attn launched as `form` (see binding.tree_attn_form) whatever the sizes would choose, with a workspace of its own
    whose counters are zero before and must be zero after."""
    import ctypes

    import torch

    from paper_2410_11744_amd import binding
    lib = dy.load_library()
    total, Hq, d = q.shape
    Hkv = int(kt.shape[1])
    cb, f = batch._c(), (ctypes.c_int32 * 3)(*form)
    need = int(lib.dyspec_workspace_bytes(binding.WS_TREE_ATTN, ctypes.byref(cb), 0, Hq, Hkv, d))
    ws = torch.zeros((max(need, 8 << 20) + 3) // 4, dtype=torch.float32, device=q.device)
    out = torch.full_like(q, float("nan"))
    p = lambda t: ctypes.c_void_p(t.data_ptr())
    st = lib.dyspec_tree_attn_in_form(f, p(q), p(kp), p(vp), p(kt), p(vt), p(mask), ctypes.byref(cb), Hq, Hkv, d, binding.BF16,
                                      ctypes.c_float(scale), p(out), p(ws), ctypes.c_size_t(ws.numel() * 4),
                                      ctypes.c_void_p(torch.cuda.current_stream().cuda_stream))
    binding._check(st, "dyspec_tree_attn_in_form")
    torch.cuda.synchronize()
    assert int(ws[:1024].view(torch.int32).abs().max().item()) == 0
    return out
