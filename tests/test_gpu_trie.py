"""GPU parity of the cache (srt_trie_insert / srt_trie_export) against the
oracle's substring counts, bit-exact: full inserts, chunked online inserts,
order independence, depths 1, 2 and 64, segments longer than a workgroup,
and the sticky error flags."""
import random

import numpy as np
import pytest
import torch

from oracle import trie as TR
from paper_2601_09083_amd import srt
from paper_2601_09083_amd import workload as W
from paper_2601_09083_amd.pipeline import Caches
from tests.gpu_util import say

pytestmark = pytest.mark.gpu


def build(streams_by_prompt, D, chunks=None, rng=None, capacity=None):
    """Insert every stream (optionally split into random chunks over several
    calls, in random order) and return the Caches."""
    P = len(streams_by_prompt)
    n_streams = sum(len(s) for s in streams_by_prompt)
    total = sum(len(x) for s in streams_by_prompt for x in s)
    cap = capacity if capacity is not None else total * D + 64
    c = Caches.create(P, n_streams + 4, D, cap)
    items = [(p, st) for p in range(P) for st in streams_by_prompt[p]]
    ids = c.new_streams(len(items))
    if chunks is None:
        c.insert([p for p, _ in items], ids, [st for _, st in items])
    else:
        pos = [0] * len(items)
        while any(pos[i] < len(items[i][1]) for i in range(len(items))):
            sel = [i for i in range(len(items)) if pos[i] < len(items[i][1]) or rng.random() < 0.1]
            rng.shuffle(sel)
            segs = []
            for i in sel:
                k = rng.randrange(0, chunks + 1)
                segs.append(items[i][1][pos[i]:pos[i] + k])
                pos[i] += k
            c.insert([items[i][0] for i in sel], ids[sel], segs)
    return c


def check_prompt(c, p, streams, D):
    got = c.export(p)
    want = TR.substring_counts(streams, D)
    assert got == want, f"prompt {p}: {len(got)} vs {len(want)} strings"


def test_tiny_config_cache_exact():
    cfg = W.CONFIGS["tiny"]
    tw = W.make_tokens(cfg)
    say("cache: tiny config, full insert")
    streams = [tw.streams_of_prompt(p) for p in range(cfg.n_prompts)]
    c = build(streams, cfg.trie_depth)
    assert c.status()["flags"] == 0
    for p in range(cfg.n_prompts):
        check_prompt(c, p, streams[p], cfg.trie_depth)


@pytest.mark.parametrize("seed", range(3))
def test_chunked_online_insert_equals_full(seed):
    rng = random.Random(seed)
    D = rng.choice([3, 6, 12])
    streams = [[np.array([rng.randrange(4) for _ in range(rng.randrange(0, 120))]) for _ in range(5)]
               for _ in range(3)]
    say(f"cache: chunked inserts seed={seed} D={D}")
    c = build(streams, D, chunks=7, rng=rng)
    assert c.status()["flags"] == 0
    for p in range(3):
        check_prompt(c, p, streams[p], D)


def test_long_streams_small_vocab():
    rng = np.random.default_rng(5)
    D = 20
    streams = [[rng.integers(0, 3, size=3000) for _ in range(4)], [rng.integers(0, 50, size=2000)]]
    say("cache: long streams, vocab 3")
    c = build(streams, D)
    for p in range(2):
        check_prompt(c, p, streams[p], D)


def test_flags_and_stream_reset():
    D = 4
    c = Caches.create(2, 8, D, 1000)
    say("cache: flags")
    c.insert([0], np.array([0], np.int32), [np.array([1, 2, 3])])
    c.insert([1], np.array([0], np.int32), [np.array([4, 5])])          # stream 0 belongs to prompt 0
    st = c.status()
    assert st["flags"] & srt.SRT_FLAG_STREAM and not st["flags"] & srt.SRT_FLAG_CAPACITY
    assert c.export(1) == {}
    c.insert([2], np.array([1], np.int32), [np.array([4])])             # prompt out of range
    assert c.status()["flags"] & srt.SRT_FLAG_PROMPT
    c.insert([0], np.array([99], np.int32), [np.array([4])])            # stream out of range
    srt.srt_trie_reset_streams(c.ws, torch.tensor([0], dtype=torch.int32, device="cuda"))
    c.insert([1], np.array([0], np.int32), [np.array([4, 5])])          # rebinding after reset works
    assert c.export(1) == TR.substring_counts([[4, 5]], D)
    assert c.export(0) == TR.substring_counts([[1, 2, 3]], D)
    c.insert([0], np.array([2], np.int32), [np.array([], dtype=np.int64)])  # empty segment
    assert c.export(0) == TR.substring_counts([[1, 2, 3]], D)
    c.insert([0], np.array([3], np.int32), [np.array([1, -2, 3])])      # negative token: entry rejected
    assert c.export(0) == TR.substring_counts([[1, 2, 3]], D)


def test_capacity_overflow_is_sticky():
    D = 8
    c = Caches.create(1, 4, D, 50)
    say("cache: capacity overflow")
    c.insert([0], np.array([0], np.int32), [np.arange(100) % 37])
    st = c.status()
    assert st["status"] == srt.SRT_ERR_CAPACITY and st["flags"] & srt.SRT_FLAG_CAPACITY
    before = st["nodes"]
    c.insert([0], np.array([1], np.int32), [np.arange(40)])
    assert c.status()["nodes"] == before  # later inserts are dropped


def test_export_truncation_reports_capacity():
    D = 3
    c = Caches.create(1, 2, D, 1000)
    c.insert([0], np.array([0], np.int32), [np.array([1, 2, 3, 4, 5])])
    with pytest.raises(srt.SrtError) as e:
        srt.srt_trie_export(c.ws, 0, 4)
    assert e.value.status == srt.SRT_ERR_CAPACITY


@pytest.mark.parametrize("D,chunks", [(64, 9), (64, None), (1, 5), (2, None)])
def test_depth_extremes(D, chunks):
    # D = 64: every stream keeps 63 active nodes between chunks; D = 1 and 2:
    # none or one
    rng = random.Random(D * 7 + (chunks or 0))
    streams = [[np.array([rng.randrange(3) for _ in range(rng.randrange(0, 150))]) for _ in range(4)]
               for _ in range(2)]
    say(f"cache: depth extremes D={D} chunks={chunks}")
    c = build(streams, D, chunks=chunks, rng=rng)
    assert c.status()["flags"] == 0
    for p in range(2):
        check_prompt(c, p, streams[p], D)


def test_segments_longer_than_a_workgroup():
    # one call appends 3000 tokens to a stream (more substring starts than
    # threads in the workgroup) and 1100 tokens to another that already has
    # active nodes
    rng = random.Random(99)
    D = 6
    s0 = np.array([rng.randrange(5) for _ in range(3000)])
    s1 = np.array([rng.randrange(5) for _ in range(1300)])
    c = Caches.create(1, 4, D, (len(s0) + len(s1)) * D + 64)
    ids = c.new_streams(2)
    say("cache: 3000- and 1100-token segments")
    c.insert([0], ids[1:], [s1[:200]])
    c.insert([0, 0], ids, [s0, s1[200:]])
    assert c.status()["flags"] == 0
    check_prompt(c, 0, [s0, s1], D)


@pytest.mark.parametrize("D,width", [(1, 961), (2, 1089), (20, 960), (20, 961), (20, 2500), (64, 1500)])
def test_long_segments_beside_short_and_rejected_ones(D, width):
    # Segments above 960 tokens go to several workgroups each: a new stream,
    # one that continues, short and empty entries of the same call, an entry
    # rejected for its last token and one of a prompt out of range.  Every
    # stream then grows by a few tokens (the short path reads the active
    # nodes that the long one left), then by a long segment again.
    rng = np.random.default_rng(1000 * D + width)
    base = rng.integers(0, 40, size=2 * width + 200)
    draw = lambda n: np.where(rng.random(n) < 0.1, rng.integers(0, 40, n), base[:n])
    c = Caches.create(2, 16, D, 40 * width * D)
    ids = np.arange(6, dtype=np.int32)
    prompts = [0, 0, 0, 1, 0, 1]
    have = [list(draw(n)) for n in (0, 70, 0, 3, 130, 0)]
    say(f"cache: long segments D={D} width={width}")
    c.insert(prompts, ids, [np.array(h, dtype=np.int64) for h in have])
    for lens in ((width, width - 1, 5, 129, 0, 128), (3, 1, 4, 0, 2, 7), (1, width, 127, width, 64, D)):
        segs = [draw(n) for n in lens]
        bad = np.concatenate([draw(width - 1), [-5]]) if lens[0] == width else np.array([4, -1])
        c.insert(prompts + [0, 2], np.concatenate([ids, [7, 8]]).astype(np.int32), segs + [bad, draw(width)])
        for h, s in zip(have, segs):
            h.extend(s)
        st = c.status()
        assert st["flags"] == srt.SRT_FLAG_STREAM | srt.SRT_FLAG_PROMPT
        for p in range(2):
            check_prompt(c, p, [np.array(h) for h, q in zip(have, prompts) if q == p], D)


@pytest.mark.parametrize("D,lens,capacity", [(8, [3000], 15000), (20, [1500, 2500, 5, 1800], 60000), (64, [1000], 52500)])
def test_long_segments_that_overflow_the_capacity_are_counted_whole(D, lens, capacity):
    # the capacity is passed in the middle of the call, the table has slots for
    # all of it: every string is counted, and every node is charged
    rng = np.random.default_rng(D)
    segs = [rng.integers(0, 50000, size=n) for n in lens]
    c = Caches.create(1, len(lens), D, capacity)
    say(f"cache: long segments past the capacity, D={D} lens={lens}")
    c.insert([0] * len(lens), np.arange(len(lens), dtype=np.int32), segs)
    st = c.status()
    want = TR.substring_counts(segs, D)
    assert capacity < len(want) < st["slots"] and st["flags"] == srt.SRT_FLAG_CAPACITY
    parent, token, count = srt.srt_trie_export(c.ws, 0, len(want) + 10)
    assert len(count) == len(want) and st["nodes"] == len(want) + 1
    check_prompt(c, 0, segs, D)


@pytest.mark.parametrize("capacity,n,width", [(100, 3, 2000), (8000, 8, 3000)])
def test_a_table_without_slots_ends_the_call(capacity, n, width):
    # far more strings than slots: what found a slot is charged and linked
    D = 8
    rng = np.random.default_rng(capacity)
    c = Caches.create(2, n, D, capacity)
    say(f"cache: table of {c.status()['slots']} slots filled up")
    c.insert([0] * n, np.arange(n, dtype=np.int32), [rng.integers(0, 50000, size=width) for _ in range(n)])
    st = c.status()
    assert st["flags"] == srt.SRT_FLAG_CAPACITY and capacity < st["nodes"] <= st["slots"]
    parent, token, count = srt.srt_trie_export(c.ws, 0, st["slots"])
    assert len(count) == st["nodes"] - 2  # the roots are no strings
    tail = torch.full((1, 8), 3, dtype=torch.int32, device="cuda")
    one = torch.ones(1, dtype=torch.int32, device="cuda")
    srt.srt_draft(c.ws, one, tail, 8 * one, 8, 16, 4)  # lookups end too
    torch.cuda.synchronize()


def test_long_segment_after_overflow_is_dropped():
    D = 8
    c = Caches.create(1, 4, D, 200)
    say("cache: long segment into a full cache")
    c.insert([0], np.array([0], np.int32), [np.arange(100)])
    before = c.status()
    assert before["flags"] & srt.SRT_FLAG_CAPACITY
    c.insert([0, 0], np.array([0, 1], np.int32), [np.arange(1200), np.arange(1200)])
    assert c.status()["nodes"] == before["nodes"]


def test_a_workspace_of_another_layout_is_left_alone():
    # the layout's mark in the header (its first word) of an older library
    D = 6
    c = Caches.create(1, 2, D, 20000)
    say("cache: workspace of another layout")
    seg = np.arange(40) % 7
    c.insert([0], np.array([0], np.int32), [seg])
    words = c.ws.view(torch.int32)
    mark = int(words[0])
    words[0] = 0x53525431
    before = c.ws.clone()
    for width in (10, 1000):
        c.insert([0], np.array([1], np.int32), [np.arange(width)])
    srt.srt_trie_reset_streams(c.ws, torch.tensor([0], dtype=torch.int32, device="cuda"))
    one = torch.ones(1, dtype=torch.int32, device="cuda")
    tail = torch.tensor([[3, 4, 5, 6]], dtype=torch.int32, device="cuda")
    args = (c.ws, 0 * one, tail, 40 * one, 4, 8, 2)
    assert srt.srt_draft(*args)["n_nodes"].item() == 1
    with pytest.raises(srt.SrtError):
        c.status()
    assert torch.equal(c.ws, before)
    words[0] = mark
    assert srt.srt_draft(*args)["n_nodes"].item() > 1
    check_prompt(c, 0, [seg], D)


@pytest.mark.parametrize("D", [1, 20, 64])
def test_segments_at_the_edge_of_one_workgroup(D):
    # rows wide enough for long segments: the chains of a stream's segment
    # (tokens and active nodes) number 255, 256 and 257, empty ones between, then
    # one more token for every stream
    rng = np.random.default_rng(D)
    have = [list(rng.integers(0, 30, size=n)) for n in (0, 0, 0, 100, 100, 100, 3, 0)]
    c = Caches.create(2, 8, D, 20000 * D)
    ids, prompts = np.arange(8, dtype=np.int32), [0, 1] * 4
    say(f"cache: segments around one workgroup's chains, D={D}")
    c.insert(prompts, ids, [np.array(h, dtype=np.int64) for h in have])
    for step in range(2):
        segs = []
        for i, h in enumerate(have):
            m = min(len(h), D - 1)
            n = (255, 256, 257, 255 - m, 256 - m, 257 - m, 0, 1200)[i] if step == 0 else 1
            segs.append(rng.integers(0, 30, size=n))
        c.insert(prompts, ids, segs)
        for h, s in zip(have, segs):
            h.extend(s)
        assert c.status()["flags"] == 0
        for p in range(2):
            check_prompt(c, p, [np.array(h) for h, q in zip(have, prompts) if q == p], D)
