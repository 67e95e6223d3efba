"""GPU parity of srt_accept_lmhead (the LM head applied at the visited nodes,
fused with the acceptance walk) against the oracle.

* Integer-valued bf16 inputs make every partial sum of the head exact in
  fp32, so the GPU walk must equal the oracle's bit for bit: ragged
  vocabularies (V = 1, 129, 4099, 50001), d_model of one to several 64-wide
  chunks, more than 256 sequences (two sequence blocks), ties (sparse hidden
  states), greedy and Gumbel at several temperatures, depth caps, root-only
  trees and node counts outside [1, N].  It must also equal srt_accept on
  the materialised logits.
* Real-valued bf16 inputs: every step of the GPU walk must be valid against
  the oracle's fp64 scores within the fp32 summation bound, and nearly all
  walks must equal the oracle's.
* Heads and passes on both sides of every rule that picks their tiles, rows
  and lists (128- and 256-row tiles, one or two a workgroup, 64, 128 and 256
  rows and more sequences than that, scratches below the full size).
* The 7B-shaped head (V = 152064, d_model = 3584, 256 sequences, N = 64,
  Dmax = 12): all sequences against srt_accept on the materialised logits,
  sampled sequences against the oracle.
* Scratch reuse across calls of different sizes."""
import random

import numpy as np
import pytest
import torch

from oracle import accept as AC
from oracle import lmhead as LH
from paper_2601_09083_amd import srt
from paper_2601_09083_amd import workload as W
from tests.gpu_util import assert_accept_equal, say
from tests.test_gpu_accept import random_trees

pytestmark = pytest.mark.gpu

U32 = 2.0 ** -24


def chain_trees(B, N, Dmax, token=0):
    """Every tree a chain of `token` (the only tree shape a one-token
    vocabulary allows), of length 1 .. min(N, Dmax + 1)."""
    tt = np.full((B, N), -1, np.int32)
    tp = np.full((B, N), -1, np.int32)
    nn = np.zeros(B, np.int32)
    for b in range(B):
        n = 1 + b % min(N, Dmax + 1)
        tt[b, :n] = token
        tp[b, 1:n] = np.arange(n - 1)
        nn[b] = n
    return {"tree_tokens": tt, "tree_parent": tp, "n_nodes": nn}


def tree_tensors(tree):
    t = lambda a: torch.as_tensor(a, device="cuda")
    return t(tree["tree_tokens"]), t(tree["tree_parent"]), t(tree["n_nodes"])


def run_fused(hidden, w, gumbel, inv_t, tree, Dmax, scratch=None):
    tt, tp, nn = tree_tensors(tree)
    acc = srt.srt_accept_lmhead(hidden, w, gumbel, inv_t, tt, tp, nn, Dmax, scratch=scratch)
    return {k: v.cpu().numpy() for k, v in acc.items()}


def run_materialised(hidden, w, gumbel, inv_t, tree, Dmax):
    """srt_accept on logits formed by a plain fp32 product (exact for the
    integer inputs these comparisons use)."""
    B, N, d = hidden.shape
    logits = (hidden.float().reshape(B * N, d) @ w.float().t().contiguous()).reshape(B, N, -1).contiguous()
    tt, tp, nn = tree_tensors(tree)
    acc = srt.srt_accept(logits, gumbel, inv_t, tt, tp, nn, Dmax)
    del logits
    return {k: v.cpu().numpy() for k, v in acc.items()}


def oracle_rows(hidden, w, gumbel, inv_t, tree, seqs, Dmax):
    h = hidden.float().cpu().numpy()
    wn = w.float().cpu().numpy()
    g = None if gumbel is None else gumbel.cpu().numpy()
    return LH.accept_lmhead_batch(h, wn, g, inv_t, tree["tree_tokens"], tree["tree_parent"], tree["n_nodes"],
                                  Dmax, seqs=seqs)


def assert_same(a, b, B):
    for k in ("n_accepted", "out_tokens", "out_nodes", "n_emitted"):
        assert np.array_equal(a[k], b[k]), k


@pytest.mark.parametrize("V,d,B,sampled,inv_t,plant,density", [
    (1000, 128, 24, False, 1.0, 0.8, 1.0),
    (1000, 128, 24, True, 1.0, 0.8, 1.0),
    (129, 64, 5, True, 0.7, 0.8, 1.0),       # one full tile and a 1-row tail
    (1, 64, 3, False, 1.0, 0.0, 1.0),        # a single token
    (4099, 256, 300, True, 1.0, 0.8, 1.0),   # two sequence blocks, ragged tail
    (2000, 192, 40, False, 1.0, 0.5, 0.02),  # sparse hidden states: many tied scores
    (2000, 192, 40, True, 1.0, 0.5, 0.02),
    (50001, 512, 64, True, 1.3, 0.9, 1.0),
])
def test_exact_integer_inputs(V, d, B, sampled, inv_t, plant, density):
    rng = random.Random(V * 31 + d + B)
    N, Dmax = 32, 8
    say(f"lmhead exact: V={V} d={d} B={B} sampled={sampled} invT={inv_t} plant={plant} density={density}")
    tree = random_trees(rng, B, N, Dmax, V) if V > 1 else chain_trees(B, N, Dmax)
    hidden, w = W.make_head(B, N, d, V, device="cuda", seed=V + d, kind="int", tree_tokens=tree["tree_tokens"],
                            tree_parent=tree["tree_parent"], n_nodes=tree["n_nodes"], plant_p=plant,
                            density=density)
    cfg = W.Config("lmh", 0, n_prompts=B, seqs_per_prompt=1, vocab=V, rollouts_per_prompt=0,
                   rollout_len=W.Dist("fixed", 1), ctx_len=W.Dist("fixed", 1), n_nodes=N, max_depth=Dmax,
                   hq=1, hkv=1, head_dim=64)
    gumbel = W.make_gumbel(cfg, B, device="cuda", seed=V + 5) if sampled else None
    got = run_fused(hidden, w, gumbel, inv_t, tree, Dmax)
    want = oracle_rows(hidden, w, gumbel, inv_t, tree, range(B), Dmax)
    for b in range(B):
        assert_accept_equal(got, b, want[b], Dmax)
    assert_same(got, run_materialised(hidden, w, gumbel, inv_t, tree, Dmax), B)
    if plant >= 0.8 or V == 1:
        assert got["n_accepted"].max() >= 2  # the walks do go deep


def test_depth_cap_root_only_and_clamped_counts():
    rng = random.Random(5)
    B, N, V, d, Dmax = 6, 10, 300, 64, 3
    tree = random_trees(rng, B, N, 9, V)  # deeper than Dmax on purpose
    tree["n_nodes"] = tree["n_nodes"].copy()
    tree["n_nodes"][0] = 1      # root only
    tree["n_nodes"][1] = 0      # clamped to 1
    tree["n_nodes"][2] = 999    # clamped to N
    hidden, w = W.make_head(B, N, d, V, device="cuda", seed=9, kind="int", tree_tokens=tree["tree_tokens"],
                            tree_parent=tree["tree_parent"], n_nodes=np.minimum(np.maximum(tree["n_nodes"], 1), N),
                            plant_p=1.0)
    for Dm in (0, Dmax):
        got = run_fused(hidden, w, None, 1.0, tree, Dm)
        want = oracle_rows(hidden, w, None, 1.0, tree, range(B), Dm)
        for b in range(B):
            assert_accept_equal(got, b, want[b], Dm)
        assert got["n_accepted"].max() <= Dm
    assert got["n_accepted"][0] == 0 and got["n_accepted"][1] == 0


def test_scratch_reuse_across_sizes():
    rng = random.Random(11)
    scratch = torch.empty(srt.srt_accept_lmhead_scratch_bytes(300, 16, 3000), dtype=torch.uint8, device="cuda")
    for B, V, d, seed in ((300, 3000, 128, 1), (17, 700, 64, 2), (300, 3000, 128, 1)):
        N, Dmax = 16, 6
        tree = random_trees(random.Random(seed), B, N, Dmax, V)
        hidden, w = W.make_head(B, N, d, V, device="cuda", seed=seed, kind="int",
                                tree_tokens=tree["tree_tokens"], tree_parent=tree["tree_parent"],
                                n_nodes=tree["n_nodes"], plant_p=0.9)
        got = run_fused(hidden, w, None, 1.0, tree, Dmax, scratch=scratch)
        assert_same(got, run_fused(hidden, w, None, 1.0, tree, Dmax), B)
        want = oracle_rows(hidden, w, None, 1.0, tree, range(B), Dmax)
        for b in range(B):
            assert_accept_equal(got, b, want[b], Dmax)


def check_valid_walk(got, b, h, wn, g, inv_t, tree, Dmax):
    """Every step of the GPU walk of sequence b is a valid choice: its token
    scores within the fp32 summation bound of the best score, it descends
    exactly when a child carries the token, and it stops at Dmax."""
    tt, tp = tree["tree_tokens"][b], tree["tree_parent"][b]
    n = min(max(int(tree["n_nodes"][b]), 1), tt.shape[0])
    k = int(got["n_accepted"][b])
    toks = got["out_tokens"][b]
    nodes = got["out_nodes"][b]
    u = 0
    for s in range(k + 1):
        exact = wn.astype(np.float64) @ h[u].astype(np.float64)
        err = LH.logit_error_bound(h[u], wn)
        x = exact * inv_t if g is not None else exact
        tol = err * (inv_t if g is not None else 1.0)
        if g is not None:
            x = x + g[b, s].astype(np.float64)
        tol = tol + 4 * U32 * np.abs(x) + 1e-30  # roundings of the product and the sum
        t = int(toks[s])
        j = int(np.argmax(x))
        assert 0 <= t < wn.shape[0], (b, s, t)
        assert x[t] >= x[j] - (tol[t] + tol[j]), (b, s, t, j, x[t], x[j])
        child = [c for c in range(u + 1, n) if tp[c] == u and tt[c] == t]
        if s < k:
            assert child and int(nodes[s]) == child[0], (b, s)
            u = child[0]
        else:
            assert not child or s == Dmax, (b, s)
    assert int(got["n_emitted"][b]) == k + 1


@pytest.mark.parametrize("V,d,sampled", [(5000, 256, False), (5000, 256, True), (32000, 1024, True)])
def test_real_valued_walks_valid(V, d, sampled):
    rng = random.Random(V + d)
    B, N, Dmax = 48, 32, 8
    say(f"lmhead real-valued: V={V} d={d} sampled={sampled}")
    tree = random_trees(rng, B, N, Dmax, V)
    hidden, w = W.make_head(B, N, d, V, device="cuda", seed=V * 3 + d, kind="normal",
                            tree_tokens=tree["tree_tokens"], tree_parent=tree["tree_parent"],
                            n_nodes=tree["n_nodes"], plant_p=0.8)
    cfg = W.Config("lmh", 0, n_prompts=B, seqs_per_prompt=1, vocab=V, rollouts_per_prompt=0,
                   rollout_len=W.Dist("fixed", 1), ctx_len=W.Dist("fixed", 1), n_nodes=N, max_depth=Dmax,
                   hq=1, hkv=1, head_dim=64)
    gumbel = W.make_gumbel(cfg, B, device="cuda", seed=V + 7) if sampled else None
    got = run_fused(hidden, w, gumbel, 1.0, tree, Dmax)
    h = hidden.float().cpu().numpy()
    wn = w.float().cpu().numpy()
    g = None if gumbel is None else gumbel.cpu().numpy()
    for b in range(B):
        check_valid_walk(got, b, h[b], wn, g, 1.0, tree, Dmax)
    want = oracle_rows(hidden, w, gumbel, 1.0, tree, range(B), Dmax)
    same = sum(int(got["n_accepted"][b]) == want[b][0] and got["out_tokens"][b, :want[b][0] + 1].tolist() == want[b][1]
               for b in range(B))
    assert same >= B - 2, same
    assert got["n_accepted"].max() >= 2


def test_qwen7b_head_sampled():
    """The 7B-shaped head and batch: V = 152064, d_model = 3584, B = 256,
    N = 64, Dmax = 12, T = 1 Gumbel; integer inputs so that every sequence
    can be compared bit for bit."""
    V, d, B, N, Dmax = 152064, 3584, 256, 64, 12
    rng = random.Random(7)
    say("lmhead qwen7b-shaped: building inputs")
    tree = random_trees(rng, B, N, Dmax, V)
    hidden, w = W.make_head(B, N, d, V, device="cuda", seed=77, kind="int", tree_tokens=tree["tree_tokens"],
                            tree_parent=tree["tree_parent"], n_nodes=tree["n_nodes"], plant_p=0.9)
    cfg = W.Config("lmh7b", 0, n_prompts=B, seqs_per_prompt=1, vocab=V, rollouts_per_prompt=0,
                   rollout_len=W.Dist("fixed", 1), ctx_len=W.Dist("fixed", 1), n_nodes=N, max_depth=Dmax,
                   hq=1, hkv=1, head_dim=64)
    gumbel = W.make_gumbel(cfg, B, device="cuda", seed=78)
    say("lmhead qwen7b-shaped: fused walk")
    got = run_fused(hidden, w, gumbel, 1.0, tree, Dmax)
    say("lmhead qwen7b-shaped: materialised logits + srt_accept")
    assert_same(got, run_materialised(hidden, w, gumbel, 1.0, tree, Dmax), B)
    deep = int(np.argmax(got["n_accepted"]))
    seqs = sorted({deep, 0, B - 1, 131})
    say(f"lmhead qwen7b-shaped: oracle on {seqs} (deepest walk {got['n_accepted'][deep]})")
    wn = w.float().cpu().numpy()
    for b in seqs:
        n = int(tree["n_nodes"][b])
        rows = LH.head_logits(hidden[b, :n].float().cpu().numpy(), wn)  # every node of the tree, fp64 -> fp32
        g = gumbel[b].cpu().numpy()
        want = AC.accept(lambda u: rows[u], lambda k: g[k], 1.0, tree["tree_tokens"][b], tree["tree_parent"][b],
                         n, Dmax)
        assert_accept_equal(got, b, want, Dmax)
    assert got["n_accepted"].max() >= 4


def planted_tree(rng, B, N, Dmax, V, deep):
    """Random trees with a long chain first (`deep` nodes), the rest hanging on
    random earlier nodes; tokens distinct among siblings as far as V allows."""
    tt = np.full((B, N), -1, np.int32)
    tp = np.full((B, N), -1, np.int32)
    nn = rng.integers(1, N + 1, size=B).astype(np.int32)
    nn[0] = N
    for b in range(B):
        n = int(nn[b])
        chain = np.sort(rng.choice(np.arange(1, n), size=min(deep, n - 1), replace=False)) if n > 1 else []
        last, on = 0, set(int(c) for c in chain)
        for i in range(1, n):
            tp[b, i] = last if i in on else rng.integers(0, i)
            last = i if i in on else last
        tt[b, :n] = rng.integers(0, V, size=n)
    return {"tree_tokens": tt, "tree_parent": tp, "n_nodes": nn}


def least_scratch(B, N, V):
    """Bytes that passes over the walking sequences' own nodes need."""
    up = lambda x: -(-x // 256) * 256
    return 4096 + up(8 * B) + up(4 * B) + up(4 * B * N) + up(8 * max(B, 128) * -(-V // 128))


@pytest.mark.parametrize("B,N,Dmax,V,d,sampled", [
    (1, 1, 3, 1, 64, False), (300, 1, 4, 300, 64, True), (300, 2, 4, 300, 64, False), (5000, 2, 2, 40, 64, False),
    (16, 32, 8, 3000, 128, True), (257, 16, 8, 1000, 64, True), (2, 300, 20, 5000, 64, False), (40, 20, 9, 33000, 64, True)])
def test_smaller_scratch_makes_smaller_passes(B, N, Dmax, V, d, sampled):
    """From the full scratch down to the least one, that of passes without
    looking ahead: the same walks, nothing written past the buffer's end."""
    rng = random.Random(B + N)
    say(f"lmhead scratch sizes: B={B} N={N} Dmax={Dmax} V={V}")
    tree = random_trees(rng, B, N, Dmax, V) if V > 1 else chain_trees(B, N, Dmax)
    hidden, w = W.make_head(B, N, d, V, device="cuda", seed=B, kind="int", tree_tokens=tree["tree_tokens"],
                            tree_parent=tree["tree_parent"], n_nodes=tree["n_nodes"], plant_p=0.9)
    gumbel = torch.randint(-3, 4, (B, Dmax + 1, V), device="cuda").float() if sampled else None
    tt, tp, nn = tree_tensors(tree)
    full, least = srt.srt_accept_lmhead_scratch_bytes(B, N, V), least_scratch(B, N, V)
    want = run_fused(hidden, w, gumbel, 1.0, tree, Dmax)
    buf = torch.empty(max(full, least) + 4096, dtype=torch.uint8, device="cuda")
    out = srt._walk_outputs(B, Dmax, "cuda")
    p = lambda x: None if x is None else x.data_ptr()

    def call(nbytes):
        buf.fill_(0x5A)
        return srt.lib().srt_accept_lmhead(
            B, N, d, V, Dmax, p(hidden), p(w), p(gumbel), 1.0, p(tt), p(tp), p(nn), p(out["n_accepted"]),
            p(out["out_tokens"]), p(out["out_nodes"]), p(out["n_emitted"]), p(buf), nbytes,
            torch.cuda.current_stream().cuda_stream)

    for nbytes in sorted({full, least, *(least + (full - least) * i // 4 // 256 * 256 for i in (1, 2, 3) if full > least)}):
        assert call(nbytes) == srt.SRT_OK, nbytes
        assert_same({k: v.cpu().numpy() for k, v in out.items()}, want, B)
        assert bool((buf[nbytes:] == 0x5A).all()), nbytes
    # the binding hands the caller's scratch over instead of allocating another
    buf.fill_(0x5A)
    before = torch.cuda.memory_stats()["allocation.all.allocated"]
    srt.srt_accept_lmhead(hidden, w, gumbel, 1.0, tt, tp, nn, Dmax, out=out, scratch=buf[:least])
    assert torch.cuda.memory_stats()["allocation.all.allocated"] == before
    assert bool((buf[:least] != 0x5A).any()) and bool((buf[least:] == 0x5A).all())
    assert_same({k: v.cpu().numpy() for k, v in out.items()}, want, B)
    assert call(min(full, least) - 256) == srt.SRT_ERR_CAPACITY
    assert call(full - 1) == srt.SRT_ERR_CAPACITY


@pytest.mark.parametrize("V,d,split", [
    (16384, 64, "small, 64 rows"), (16385, 192, "small, 64 or 128 rows"), (32768, 320, "small, 64 or 128 rows"),
    (32769, 320, "wide"), (40001, 2112, "wide"), (65537, 1088, "wide, two tiles a workgroup")])
@pytest.mark.parametrize("B,N,Dmax,sampled", [(30, 6, 5, False), (110, 4, 3, True), (300, 3, 2, True), (290, 5, 4, False)])
def test_both_divisions_of_the_head(V, d, split, B, N, Dmax, sampled):
    """The head on both sides of every line between its divisions, with
    vocabularies that are no multiple of a tile, a unit or 4 (noise rows then
    start at any float) and odd numbers of 64-wide steps (1, 3, 5, 17, 33),
    in passes of up to 64, up to 128, up to 256 and more rows (the sequences'
    own nodes and those looked ahead at)."""
    tiles = -(-V // 128)
    assert split == ("small, 64 rows" if tiles <= 128 else "small, 64 or 128 rows" if tiles <= 256 else
                     "wide" if V <= 65536 else "wide, two tiles a workgroup")
    rng = random.Random(V + B)
    say(f"lmhead divisions: V={V} d={d} ({split}) B={B} N={N} Dmax={Dmax} sampled={sampled}")
    tree = random_trees(rng, B, N, Dmax, V)
    hidden, w = W.make_head(B, N, d, V, device="cuda", seed=V + B, kind="int", tree_tokens=tree["tree_tokens"],
                            tree_parent=tree["tree_parent"], n_nodes=tree["n_nodes"], plant_p=0.9)
    gumbel = torch.randint(-3, 4, (B, Dmax + 1, V), device="cuda").float() if sampled else None
    got = run_fused(hidden, w, gumbel, 1.0, tree, Dmax)
    assert_same(got, run_materialised(hidden, w, gumbel, 1.0, tree, Dmax), B)
    seqs = sorted(rng.sample(range(B), 6)) + [int(np.argmax(got["n_accepted"]))]
    want = oracle_rows(hidden, w, gumbel, 1.0, tree, seqs, Dmax)
    for b in seqs:
        assert_accept_equal(got, b, want[b], Dmax)
    assert got["n_accepted"].max() >= 1


@pytest.mark.parametrize("B,N,Dmax,V,d,sampled", [
    (16, 16, 15, 500, 64, True),        # 256 nodes in all: one pass
    (17, 16, 15, 500, 64, False),       # 272: 256 of them, then what is left
    (16, 16, 2, 500, 64, True),         # short walks: 256 nodes, one pass
    (17, 16, 2, 500, 64, False),        # 272: 64 rows
    (254, 3, 2, 500, 64, True),         # 254 to 256 walkers of 762 and more nodes, a row each
    (255, 3, 4, 500, 64, False),
    (256, 3, 4, 500, 64, True),
    (70, 5, 1, 500, 128, False),        # 70 walkers in passes of 64 rows: their own nodes
    (40, 20, 6, 20480, 1024, False),    # a light head: 256 rows; one of a row more: 64
    (40, 20, 6, 20481, 1024, True),     # (24 of 40 walkers bring a second node)
    (16, 32, 6, 20481, 1024, False),    # 512 and 527 nodes: 256 and 64 rows
    (17, 31, 6, 20481, 1024, True),
    (64, 9, 3, 20481, 1024, False),     # 64 and 65 sequences: 64 and 128 rows
    (65, 9, 3, 20481, 1024, True),
    (40, 20, 7, 20481, 1024, True),     # deeper: 256 rows
    (40, 20, 7, 24576, 2048, False),    # until the head is large: 128
    (40, 20, 7, 24577, 2048, True),
    (129, 16, 4, 20481, 1024, False),   # 129 sequences of 16 and 17 nodes: 256 and 128 rows,
    (129, 17, 4, 20481, 1024, True),
    (129, 17, 7, 24577, 2048, False),   # when deeper 256 up to 64 nodes
    (129, 65, 7, 24577, 2048, True),
])
def test_rows_of_a_pass(B, N, Dmax, V, d, sampled):
    """Full trees on both sides of every rule that gives a pass its rows."""
    rng = np.random.default_rng(B * 100 + N)
    say(f"lmhead rows of a pass: B={B} N={N} Dmax={Dmax} V={V} d={d}")
    tree = planted_tree(rng, B, N, Dmax, V, N // 2)
    tree["n_nodes"][:] = N
    for b in range(B):
        for i in range(1, N):
            if tree["tree_parent"][b, i] < 0:
                tree["tree_parent"][b, i] = rng.integers(0, i)
                tree["tree_tokens"][b, i] = rng.integers(0, V)
    hidden, w = W.make_head(B, N, d, V, device="cuda", seed=B + N, kind="int", tree_tokens=tree["tree_tokens"],
                            tree_parent=tree["tree_parent"], n_nodes=tree["n_nodes"], plant_p=0.9)
    gumbel = torch.randint(-3, 4, (B, Dmax + 1, V), device="cuda").float() if sampled else None
    got = run_fused(hidden, w, gumbel, 1.0, tree, Dmax)
    assert_same(got, run_materialised(hidden, w, gumbel, 1.0, tree, Dmax), B)
    seqs = range(B) if V <= 500 else sorted(rng.choice(B, 4, replace=False).tolist()) + [int(np.argmax(got["n_accepted"]))]
    want = oracle_rows(hidden, w, gumbel, 1.0, tree, seqs, Dmax)
    for b in seqs:
        assert_accept_equal(got, b, want[b], Dmax)
    assert got["n_accepted"].max() >= 1


@pytest.mark.parametrize("B,N,Dmax,V,d", [
    (40, 20, 19, 24577, 2048),   # 128 rows, quotas of 3
    (24, 30, 29, 24577, 2048),   # of 5
    (2, 260, 63, 24577, 2048),   # of 64
    (4, 130, 6, 20481, 1024),    # 64 rows, quotas of 16
    (10, 60, 6, 20481, 1024),
    (100, 20, 19, 500, 64),      # 256 rows, quotas of 2
    (256, 8, 7, 500, 64),        # of 1
    (257, 8, 7, 500, 64),        # more walkers than rows
])
@pytest.mark.parametrize("step", [1, "quota", "past"])
def test_enough_passes_for_every_walk(B, N, Dmax, V, d, step):
    """Every walk follows its tree to the end and moves no further in a pass
    than it must: the path's next node is the next one, the last one of the
    pass or the first one after it, with the nodes between below it too."""
    look = 256 if V == 500 else 128 if Dmax > 6 else 64
    quota = max(1, look // B)
    s = {1: 1, "quota": max(1, quota - 1), "past": quota}[step]
    say(f"lmhead enough passes: B={B} N={N} Dmax={Dmax} V={V} d={d} step={s}")
    par = np.full(N, -1, np.int32)
    path = list(range(0, min(N, Dmax * s + 1), s))
    for i in range(1, N):
        par[i] = path[min((i - 1) // s, len(path) - 1)] if len(path) <= Dmax or i <= path[-1] else path[-2]
    rng = np.random.default_rng(B + N)
    tree = {"tree_parent": np.tile(par, (B, 1)), "n_nodes": np.full(B, N, np.int32),
            "tree_tokens": np.stack([rng.permutation(V)[:N] for _ in range(B)]).astype(np.int32)}
    hidden, w = W.make_head(B, N, d, V, device="cuda", seed=B + N, kind="int")
    for u, c in zip(path, path[1:]):  # the path's next token wins (scores of 4 d against about sqrt(16 d))
        hidden[:, u] = w[torch.as_tensor(tree["tree_tokens"][:, c], device="cuda").long()]
    got = run_fused(hidden, w, None, 1.0, tree, Dmax)
    assert (got["n_accepted"] >= len(path) - 1).all()
    assert (got["out_nodes"][:, :len(path) - 1] == path[1:]).all()
    want = oracle_rows(hidden, w, None, 1.0, tree, (0, B - 1), Dmax)
    for b in (0, B - 1):
        assert_accept_equal(got, b, want[b], Dmax)


@pytest.mark.parametrize("B,N,Dmax,V,d,deep,sampled", [
    (1, 64, 20, 4096, 64, 20, True),      # one sequence: its whole tree in one pass
    (2, 300, 40, 300, 128, 40, False),    # trees longer than a pass's list
    (1, 1100, 63, 257, 64, 63, False),    # more nodes than the staged parents
    (3, 200, 12, 17, 320, 12, True),      # fewer head rows than a tile has
    (31, 40, 10, 4113, 192, 10, False),   # uneven quotas, a last tile of 17 head rows
    (129, 24, 8, 65553, 64, 8, True),     # 129 walkers: wide tiles of 256 rows, two a workgroup
    (256, 8, 6, 1000, 128, 6, False),     # exactly as many walkers as rows
    (257, 16, 6, 1000, 448, 6, True),     # more walkers than rows: one node each
])
def test_passes_look_ahead(B, N, Dmax, V, d, deep, sampled):
    rng = np.random.default_rng(B * 1000 + N)
    say(f"lmhead passes: B={B} N={N} Dmax={Dmax} V={V} d={d}")
    tree = planted_tree(rng, B, N, Dmax, V, deep)
    hidden, w = W.make_head(B, N, d, V, device="cuda", seed=B + N, kind="int", tree_tokens=tree["tree_tokens"],
                            tree_parent=tree["tree_parent"], n_nodes=tree["n_nodes"], plant_p=0.9)
    # the chain's next token wins at most of its nodes (integers: sums stay exact)
    for b in range(B):
        for i in range(1, int(tree["n_nodes"][b])):
            u = int(tree["tree_parent"][b, i])
            if rng.random() < 0.3:
                hidden[b, u] = w[int(tree["tree_tokens"][b, i])]
    gumbel = torch.randint(-3, 4, (B, Dmax + 1, V), device="cuda").float() if sampled else None
    got = run_fused(hidden, w, gumbel, 1.0, tree, Dmax)
    if N <= 256:
        assert_same(got, run_materialised(hidden, w, gumbel, 1.0, tree, Dmax), B)
    else:  # beyond srt_accept's trees
        want = oracle_rows(hidden, w, gumbel, 1.0, tree, range(B), Dmax)
        for b in range(B):
            assert_accept_equal(got, b, want[b], Dmax)
    assert got["n_accepted"].max() >= 2
