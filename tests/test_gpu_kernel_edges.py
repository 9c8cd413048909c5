"""Kernels at the sizes where their tiling can go wrong, against the CPU oracle: edges of tiles,
remainders, the smallest and largest shapes of a variant.  Bit-exact like every result of the library."""
import gc
from concurrent.futures import ThreadPoolExecutor

import numpy as np
import pytest
import torch

from oracle import st_oracle as O
from paper_2511_14881_amd import binding as st
from paper_2511_14881_amd import synth as S
from tests.test_gpu_expr import check_expr_search, check_ivf, pack
from tests.test_gpu_parity import check_search, oracle_index, ragged_workload
from tests.test_oracle_expr_pins import postfix

pytestmark = pytest.mark.gpu


def _u64(t):
    return t.detach().cpu().numpy().view(np.uint64)


# row blocks of 32, passes of 512 rows, 1 to 8 tiles per workgroup of the export; last tile full, one item, one missing
@pytest.mark.parametrize("m", [1, 33, 64, 65, 192, 257, 511, 512, 513, 1024, 1100])
@pytest.mark.parametrize("n", [1, 1023, 8 * 1024, 9 * 1024 + 1])
def test_index_build_and_export_at_tile_edges(n, m):
    print(f"[edges] build/export n={n} m={m}", flush=True)
    rng = np.random.default_rng(n * 7919 + m)
    lens = rng.integers(0, 20, n)
    off = np.concatenate([[0], np.cumsum(lens)]).astype(np.int64)
    ids = rng.integers(0, 1 << 62, int(off[-1])).astype(np.int64)
    bloom = st.st_bloom_build(torch.from_numpy(off).cuda(), torch.from_numpy(ids).cuda(), n, m, 3)
    got = _u64(st.st_bloom_export_signatures(bloom))
    assert np.array_equal(got, O.bloom_build(off, ids.view(np.uint64), m, 3))


# Lists of 0 to 40 ids (pairs of ids begin at odd places and end with one id), hashes that are written out and counted ones, one
# slab of rows and two.
@pytest.mark.parametrize("n,m,k,most", [(512 * 1024 + 3, 512, 4, 40), (512 * 1024, 100, 5, 26), (511 * 1024, 64, 2, 40),
                                        (530_001, 128, 3, 25), (530_001, 256, 3, 20), (525_000, 96, 7, 33), (3_000, 1100, 2, 40),
                                        (70_001, 1024, 1, 9)])
def test_index_build_of_long_and_short_lists(n, m, k, most):
    rng = np.random.default_rng(n + m)
    off = np.concatenate([[0], np.cumsum(rng.integers(0, most + 1, n))]).astype(np.int64)
    ids = rng.integers(0, 1 << 62, int(off[-1])).astype(np.int64)
    bloom = st.st_bloom_build(torch.from_numpy(off).cuda(), torch.from_numpy(ids).cuda(), n, m, k)
    got = _u64(st.st_bloom_export_signatures(bloom))
    bloom.free()
    assert np.array_equal(got, O.bloom_build(off, ids.view(np.uint64), m, k))


# From 12 ids to an item on, 512 tiles on and with rows in a power of two, four lanes share a list: every number of hashes that is
# written out and two that are counted.  One lane, by each of these limits, for the same; lists of fewer than four ids with
# counted hashes (an id to a load); two slabs of rows.
@pytest.mark.parametrize("n,m,k,most,lanes", [
    (511 * 1024 + 3, 512, 4, 40, 4), (511 * 1024 + 1, 256, 2, 26, 4), (530_001, 128, 3, 25, 4), (512 * 1024, 64, 5, 33, 4), (525_000, 512, 7, 26, 4),
    (524_289, 32, 1, 28, 4), (512 * 1024, 100, 5, 26, 1), (511 * 1024, 64, 2, 40, 1), (530_001, 256, 3, 20, 1), (525_000, 96, 7, 33, 1),
    (70_001, 256, 4, 9, 1), (50_003, 128, 5, 12, 1), (9_001, 2048, 6, 30, 1), (70_001, 512, 8, 5, 1), (40_000, 1024, 1, 3, 1),
    (33_333, 64, 16, 6, 1)])
def test_every_form_of_the_index_build(n, m, k, most, lanes):
    rng = np.random.default_rng(n + m)
    off = np.concatenate([[0], np.cumsum(rng.integers(0, most + 1, n))]).astype(np.int64)
    assert (m <= 1024 and m & (m - 1) == 0 and off[-1] >= 12 * n and n > 511 * 1024) == (lanes == 4)
    ids = rng.integers(0, 1 << 62, int(off[-1])).astype(np.int64)
    bloom = st.st_bloom_build(torch.from_numpy(off).cuda(), torch.from_numpy(ids).cuda(), n, m, k)
    got = _u64(st.st_bloom_export_signatures(bloom))
    bloom.free()
    assert np.array_equal(got, O.bloom_build(off, ids.view(np.uint64), m, k))


# Builds of several sizes above the default LDS limit share one kernel, and with it one limit, on any number of threads.
def test_indexes_of_several_sizes_built_by_threads_at_once():
    n, k, widths = 40_000, 3, (600, 1000, 700, 900)
    rng = np.random.default_rng(n)
    off = np.concatenate([[0], np.cumsum(rng.integers(0, 9, n))]).astype(np.int64)
    ids = rng.integers(0, 1 << 62, int(off[-1])).astype(np.int64)
    dev_off, dev_ids = torch.from_numpy(off).cuda(), torch.from_numpy(ids).cuda()
    torch.cuda.synchronize()

    def build(m):
        stream = torch.cuda.Stream()
        for _ in range(100):
            bloom = st.st_bloom_build(dev_off, dev_ids, n, m, k, stream=stream)
        got = st.st_bloom_export_signatures(bloom, stream=stream)
        stream.synchronize()
        return _u64(got)

    with ThreadPoolExecutor(len(widths)) as pool:
        for m, got in zip(widths, pool.map(build, widths)):
            assert np.array_equal(got, O.bloom_build(off, ids.view(np.uint64), m, k)), m


# The tables of a captured call are read again at every replay: eager calls in between (more than there are
# staging slots) must not get the slot.  Once without a seed pass, once with it.
@pytest.mark.parametrize("n", [20_000, 300_000])
def test_captured_search_replays_beside_eager_calls(n):
    print(f"[edges] graph n={n}", flush=True)
    w = S.make_workload(S.scaled(S.CONFIGS["mid"], n, batch=9, top_k=20), "cuda")
    cfg = w.cfg
    bloom = st.st_bloom_build(w.feat_offsets, w.feat_ids, n, cfg.m_bits, cfg.k_hashes)

    def call(fid, foff, buf):
        return st.st_search(bloom, w.items, w.item_scale, w.queries, w.query_scale, fid, foff, cfg.top_k, buffers=buf)

    buf, other = st.SearchBuffers(n, cfg.d, 9, 1, cfg.top_k), st.SearchBuffers(n, cfg.d, 9, 1, cfg.top_k)
    want = [t.clone() for t in call(w.filt_ids, w.filt_offsets, buf)]
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        call(w.filt_ids, w.filt_offsets, buf)
    no_filter = np.zeros(10, np.int64)
    for _ in range(3):
        for _ in range(20):
            call(np.zeros(0, np.uint64), no_filter, other)
        for t in (buf.ids, buf.scores, buf.count):
            t.zero_()
        graph.replay()
        torch.cuda.synchronize()
        assert all(torch.equal(a, b) for a, b in zip((buf.ids, buf.scores, buf.count), want))


def _programs(rng, B, vocab):
    """One filter program per query (none for some): a AND NOT b, a OR b, or a alone."""
    out = []
    for b in range(B):
        x, y = (int(v) for v in rng.integers(0, vocab, 2))
        out.append([([], []), ([O.LEAF, O.LEAF, O.NOT, O.AND], [x, y, 0, 0]), ([O.LEAF, O.LEAF, O.OR], [x, y, 0]),
                    ([O.LEAF], [x])][int(rng.integers(0, 4)) if b else 0])
    return out


def _replays_like_eager(call, buf, others):
    """call(buf): one search into buf.  Once eagerly, once captured, then replays beside eager calls of others(); every
    replay has to give what the eager call gave."""
    want = [t.clone() for t in call(buf)]
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        call(buf)
    for _ in range(3):
        for _ in range(20):
            others()
        for t in (buf.ids, buf.scores, buf.count):
            t.zero_()
        graph.replay()
        torch.cuda.synchronize()
        assert all(torch.equal(a, b) for a, b in zip((buf.ids, buf.scores, buf.count), want))


# A captured call finds a staging slot of its size after one eager call of its shape (200 programs: their
# tables and the search's fit a slot as it comes, a bound on the tables' size does not).  With and without a seed
# pass; probing per query and through mask rows.
@pytest.mark.parametrize("kind,n,B,probes", [("expr", 20_000, 200, 0), ("expr", 300_000, 100, 0), ("ivf", 20_000, 200, 9),
                                             ("ivf", 20_000, 40, 600)])
def test_captured_programs_and_probing(kind, n, B, probes):
    print(f"[edges] graph {kind} n={n} B={B} probes={probes}", flush=True)
    w = ragged_workload(n + B, n, 32, B, 24, 6, 128, 3)
    ops, ids, off = pack(_programs(np.random.default_rng(n + B), B, 24))
    items, iscale, foff, fids, q, qs = [t.cuda() for t in (w.items, w.item_scale, w.feat_offsets, w.feat_ids, w.queries,
                                                           w.query_scale)]
    bloom = st.st_bloom_build(foff, fids, n, 128, 3)
    if kind == "expr":
        bufs = [st.SearchBuffers(n, 32, B, 1, 20, n_expr_entries=int(off[-1])) for _ in range(2)]

        def call(buf):
            return st.st_search_expr(bloom, items, iscale, q, qs, ops, ids, off, 20, buffers=buf)
    else:
        cent, cs, coff = (t.cuda() for t in S.gen_clusters(w.cfg, 1000))
        bufs = [st.IvfBuffers(n, 32, B, 20, 1000, probes, int(off[-1])) for _ in range(2)]

        def call(buf):
            return st.st_search_ivf(bloom, items, iscale, cent, cs, coff, probes, q, qs, ops, ids, off, 20, buffers=buf)[:3]

    _replays_like_eager(call, bufs[0], lambda: call(bufs[1]))


# The first call with larger tables than any slot holds may itself be captured: its slot grows within the capture.
def test_staging_slot_grows_within_a_capture():
    n, B = 5_000, 2000
    w = ragged_workload(5, n, 16, B, 400, 6, 256, 3)
    w.filt_ids = np.random.default_rng(1).integers(0, 400, 2 * B).astype(np.uint64)
    w.filt_offsets = np.arange(0, 2 * B + 1, 2).astype(np.int64)
    assert st.st_search_host_plan(n, 16, B, 1, 5, 256, 3, w.filt_ids, w.filt_offsets)["table_bytes"] > 200_000
    items, iscale, foff, fids, q, qs = [t.cuda() for t in (w.items, w.item_scale, w.feat_offsets, w.feat_ids, w.queries,
                                                           w.query_scale)]
    bloom = st.st_bloom_build(foff, fids, n, 256, 3)

    def call(buf, b):
        return st.st_search(bloom, items, iscale, q[:b], qs[:b], w.filt_ids[:2 * b], w.filt_offsets[:b + 1], 5, buffers=buf)

    small, buf, eager = (st.SearchBuffers(n, 16, b, 1, 5) for b in (300, B, B))
    call(small, 300)
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        call(buf, B)
    want = call(eager, B)
    for _ in range(2):
        for t in (buf.ids, buf.scores, buf.count):
            t.zero_()
        graph.replay()
        torch.cuda.synchronize()
        assert all(torch.equal(a, b) for a, b in zip((buf.ids, buf.scores, buf.count), want))


# More captured calls than there are staging slots, all kept for replay, and queues of eager calls between them.
def test_more_graphs_than_staging_slots():
    n = 20_000
    w = S.make_workload(S.scaled(S.CONFIGS["mid"], n, batch=9, top_k=20), "cuda")
    cfg = w.cfg
    bloom = st.st_bloom_build(w.feat_offsets, w.feat_ids, n, cfg.m_bits, cfg.k_hashes)

    def call(buf):
        return st.st_search(bloom, w.items, w.item_scale, w.queries, w.query_scale, w.filt_ids, w.filt_offsets, cfg.top_k,
                            buffers=buf)

    bufs = [st.SearchBuffers(n, cfg.d, 9, 1, cfg.top_k) for _ in range(19)]
    want = [t.clone() for t in call(bufs[18])]
    torch.cuda.synchronize()
    graphs = []
    for i in range(18):
        graphs.append(torch.cuda.CUDAGraph())
        with torch.cuda.graph(graphs[i]):
            call(bufs[i])
        for _ in range(40):
            call(bufs[18])
    for _ in range(2):
        for g, b in zip(graphs, bufs):
            for t in (b.ids, b.scores, b.count):
                t.zero_()
            g.replay()
            torch.cuda.synchronize()
            assert all(torch.equal(a, c) for a, c in zip((b.ids, b.scores, b.count), want))
            call(bufs[18])


# Freed index memory is the program's again: at once when the last index is freed, and on request while another one
# lives (128 MB each).
def test_freed_index_memory_goes_back_to_the_driver():
    n, m, mb = 1 << 20, 1024, 128 << 20
    gc.collect()
    off, ids = torch.zeros(n + 1, dtype=torch.int64, device="cuda"), torch.zeros(1, dtype=torch.int64, device="cuda")
    st.st_bloom_build(off, ids, n, 64, 1).free()
    st.st_bloom_trim()

    def free_bytes():
        torch.cuda.synchronize()
        return torch.cuda.mem_get_info()[0]

    start = free_bytes()
    first = st.st_bloom_build(off, ids, n, m, 1)
    assert free_bytes() < start - mb + mb // 4
    first.free()
    assert free_bytes() > start - mb // 2
    first, second = (st.st_bloom_build(off, ids, n, m, 1) for _ in range(2))
    first.free()
    st.st_bloom_trim()
    assert start - 2 * mb < free_bytes() < start - mb + mb // 4
    third = st.st_bloom_build(off, ids, n, m, 1)
    second.free()
    third.free()
    assert free_bytes() > start - mb // 2


# Batches whose queries hardly share filters (the products of all pairs, or of the passing ones where a wavefront has
# few): row lengths of every variant, one query block and several, two and three rows of the grid (of equal and other widths), ragged last segment
# and word, few and many signature rows, no filter, filters that pass 10 %, 1 % and nothing, tied scores; a corpus whose
# filters pass everything in some stretches and nothing in others (wavefronts change between the two forms), and
# no filter at all (no signature row is named); scales of many sizes (a wavefront's bounds move as it meets larger ones), some
# words of items beyond those that a bound is formed for, scores that are all negative (no bound), rows with a common mean, whose
# bounds are beyond the digits' range (scales of one size, and some ten times as large); whole rounds of 8 words to each of 256
# workgroups, and one item more, with a sampled first level (of 1024 words) and with a seed pass.  The last selection would make good for lost candidates, so no
# query that passes enough items may have needed that.
@pytest.mark.parametrize("n,d,B,m,kind", [(600_001, 64, 16, 64, "mixed"), (530_049, 96, 33, 100, "mixed"),
                                          (400_003, 128, 130, 512, "mixed"), (524_288 + 31, 192, 40, 257, "mixed"),
                                          (420_000, 256, 300, 128, "mixed"), (600_000, 64, 64, 512, "rare"),
                                          (350_000, 128, 140, 512, "rare"), (400_001, 64, 150, 128, "ties"),
                                          (430_013, 256, 48, 300, "stretches"), (330_077, 96, 260, 64, "stretches"),
                                          (300_011, 96, 20, 257, "none"), (380_001, 128, 130, 256, "scales"),
                                          (300_031, 64, 40, 64, "scales"), (350_000, 192, 70, 512, "beyond"),
                                          (400_007, 64, 150, 100, "beyond"), (330_000, 256, 100, 300, "negative"),
                                          (420_000, 96, 200, 64, "negative"), (300_031, 128, 32, 512, "mixed"),
                                          (350_001, 192, 31, 100, "stretches"), (400_003, 96, 32, 64, "ties"),
                                          (330_000, 64, 24, 257, "negative"), (310_017, 128, 17, 128, "beyond"),
                                          (300_011, 192, 16, 64, "scales"), (320_009, 256, 32, 128, "mixed"),
                                          (300_000, 128, 257, 128, "stretches"), (310_001, 64, 641, 300, "mixed"),
                                          (400_009, 256, 225, 512, "rare"), (300_007, 192, 65, 64, "outliers"),
                                          (300_001, 256, 130, 128, "mean"), (330_031, 128, 40, 64, "mean"), (300_007, 64, 20, 300, "mean"),
                                          (310_003, 192, 200, 64, "mean, large scales"), (340_009, 96, 70, 128, "mean, large scales"),
                                          (458_752, 64, 130, 64, "mixed"), (458_753, 128, 150, 128, "mixed"),
                                          (393_216, 96, 20, 64, "mixed"), (393_217, 192, 40, 100, "mixed")])
def test_own_filters(n, d, B, m, kind):
    w = ragged_workload(n, n, d, B, 40, 8, m, 3)
    filters = []
    for b in range(B):
        one = [(b // 3) % 40]
        two = [b % 40, (7 * b + b // 40 + 1) % 40]
        filters.append([] if b == 0 else [999] if b == 1 else one if b % 3 == 0 and kind != "rare" else two + [(b * 11 + 3) % 40] * (b % 2))
    if kind == "none":
        filters = [[] for _ in range(B)]
    w.filt_ids = np.array([x for f in filters for x in f], np.uint64)
    w.filt_offsets = np.concatenate([[0], np.cumsum([len(f) for f in filters])]).astype(np.int64)
    if kind == "ties":
        w.items = w.items[:997].repeat(n // 997 + 1, 1)[:n].contiguous()
        w.item_scale = w.item_scale[:997].repeat(n // 997 + 1)[:n].contiguous()
    elif kind == "stretches":  # all 40 features, none, or two of them, for 700 items each (in no order)
        turn = np.random.default_rng(d).integers(0, 3, n // 700 + 1).repeat(700)[:n]
        lens = np.array([0, 40, 2])[turn]
        off = np.concatenate([[0], np.cumsum(lens)]).astype(np.int64)
        ids = (np.arange(off[-1]) - off[:-1].repeat(lens) + (np.arange(n) * (turn == 2)).repeat(lens)) % 40
        w.feat_offsets, w.feat_ids = torch.from_numpy(off), torch.from_numpy(ids.astype(np.int64))
    elif kind == "scales":
        w.item_scale = torch.from_numpy(np.exp2(np.random.default_rng(n).uniform(-20, 20, n)).astype(np.float32))
    elif kind == "beyond":  # word by word: up to 2^110, ordinary ones, all below 2^-90
        rng = np.random.default_rng(n)
        lo, hi = np.array([(-110, 110), (-3, 3), (-110, -95)])[rng.integers(0, 3, n // 64 + 1).repeat(64)[:n]].T
        w.item_scale = torch.from_numpy(np.exp2(rng.uniform(lo, hi)).astype(np.float32))
    elif kind == "outliers":  # a twentieth of the items far below the others' scales: the bounds' reference is not theirs
        w.item_scale = torch.from_numpy(np.where(np.random.default_rng(n).random(n) < 0.05, 1e-6, 1.0).astype(np.float32)) * w.item_scale
    elif kind.startswith("mean"):
        rng = np.random.default_rng(n)
        mu = rng.uniform(-127, 127, d)
        def rows(r):
            return torch.from_numpy((0.85 * mu + 0.5 * rng.uniform(-127, 127, (r, d))).round().clip(-127, 127).astype(np.int8))
        w.items, w.queries = rows(n), rows(B).view(w.queries.shape)
        if kind != "mean":
            w.item_scale = torch.from_numpy(np.where(rng.random(n) < 0.003, 10.0, 1.0).astype(np.float32)) * w.item_scale
    elif kind == "negative":
        w.items = w.items.abs().clamp(1, 127).to(torch.int8)
        w.queries = (-w.queries.abs().clamp(1, 127).to(torch.int16)).to(torch.int8)
    K = 60
    sigs = oracle_index(w)
    passing = [int(np.unpackbits(O.bloom_mask(sigs, m, 3, np.array(f, np.uint64)).view(np.uint8)).sum()) for f in filters]
    fast = [b for b in range(B) if passing[b] >= 40 * K] if kind not in ("ties", "beyond") else []
    assert kind in ("ties", "beyond") or len(fast) > B // 2
    check_search(w, K, sigs=sigs, queries=sorted({0, 1, 2, 3, B - 1, *range(0, B, max(1, B // 12))}), slow_path=([], fast),
                 label=f"own filters {kind}")


# The list of pairs that such a scan gathers, which goes from unit to unit: units of 64 items with 1 to 64 passing pairs, with up
# to the 112 that are gathered for more than 64 queries, and with more, which are multiplied, in short stretches, so that wavefronts
# enter and leave either form with a list that is part full.  Row lengths of every variant (each has its own split of a row over lanes).
@pytest.mark.parametrize("n,d,B,m", [(400_009, 64, 100, 512), (350_003, 96, 180, 256), (400_001, 128, 140, 512), (350_017, 192, 90, 512),
                                     (400_003, 256, 225, 512), (350_001, 256, 64, 512), (360_007, 96, 50, 256)])
def test_own_filters_few_pairs(n, d, B, m):
    w = ragged_workload(n, n, d, B, 40, 8, m, 3)
    rng = np.random.default_rng(n + d)
    # two ids of 40 to a filter: an item with L ids passes about (L / 40)^2 of them (ids 16 apart share no hashes)
    pairs = rng.choice((15, 40, 60, 75, 100, 115, 200), n // 320 + 1).repeat(320)[:n]
    want = 40 * np.sqrt(pairs / (64 * B))
    lens = (np.floor(want) + (rng.random(n) < want % 1)).astype(np.int64)
    w.feat_offsets = torch.from_numpy(np.concatenate([[0], np.cumsum(lens)]).astype(np.int64))
    w.feat_ids = torch.from_numpy(16 * rng.integers(0, 40, int(lens.sum())).astype(np.int64))
    filters = [(b % 40 * 16, (7 * b + b // 40 * 2 + 1) % 40 * 16) for b in range(B)]
    w.filt_ids = np.array([x for f in filters for x in f], np.uint64)
    w.filt_offsets = np.arange(0, 2 * B + 1, 2).astype(np.int64)
    K = 40
    sigs = oracle_index(w)
    masks = np.stack([O.bloom_mask(sigs, m, 3, np.array(f, np.uint64)) for f in filters]).view(np.uint64)
    unit = np.bitwise_count(masks).sum(0, dtype=np.int64)
    limit = 64 if B <= 64 else 112
    for lo, hi in ((1, 32), (33, 64), (65, limit), (limit + 1, 1 << 30)):
        assert lo > hi or np.mean((unit >= lo) & (unit <= hi)) > 0.1, (lo, hi, np.percentile(unit, (5, 25, 50, 75, 95)))
    got = st.st_search_host_plan(n, d, B, 1, K, m, 3, w.filt_ids, w.filt_offsets)
    assert got["mfma_groups"] == 0, got
    passing = np.bitwise_count(masks).sum(1, dtype=np.int64)
    fast = [b for b in range(B) if passing[b] >= 40 * K]
    assert len(fast) > B // 2
    check_search(w, K, sigs=sigs, queries=sorted({0, 1, B - 1, *range(0, B, max(1, B // 16))}), slow_path=([], fast), label="own filters, few pairs")


# Scales (finite and > 0) whose scores leave the normal range, in every form of the scans that tests pairs by an
# integer bound first.  "tiny": scores of two or three units of 2^-149, so that dots up to half a unit away round to the
# score of the threshold and, with the lower id, come before it.  "huge": dot * s_q overflows for the largest dots, so
# that items of small scales score infinity beside thresholds that are finite.
def _extreme_scales(w, kind):
    n, B = w.items.shape[0], w.queries.shape[0]
    rng = np.random.default_rng(n + B)
    top = (w.items[:4000].double() @ w.queries.double().T).amax(0).numpy()  # about the 4000th part of the best
    if kind == "tiny":
        w.item_scale = torch.full((n,), 2.0 ** -85)
        w.query_scale = torch.from_numpy((rng.uniform(1.5, 4, B) * 2.0 ** -64 / top).astype(np.float32))
    else:
        w.item_scale = torch.from_numpy(np.exp2(rng.uniform(-80, -60, n)).astype(np.float32))
        w.query_scale = torch.from_numpy((2.0 ** 128 / top).astype(np.float32))


# form: the scan for filters of their own behind a seed pass and behind a first level of its own; the MFMA scan of four
# wavefronts; of eight: rows of 512, few items to a filter, more filters than the form by units takes, and that form.
@pytest.mark.parametrize("kind", ["tiny", "huge"])
@pytest.mark.parametrize("form,n,d,B,groups,vocab,plan", [
    ("own, seed", 300_000, 64, 128, 128, 40, dict(mfma_groups=0, seed_pass=1)),
    ("own", 400_000, 256, 160, 160, 40, dict(mfma_groups=0, seed_pass=0)),
    ("own, one block", 300_000, 96, 32, 32, 40, dict(mfma_groups=0, seed_pass=1)),
    ("four", 300_000, 128, 64, 8, 12, dict(dot_groups=0, waves=4)),
    ("rows of 512", 400_000, 512, 140, 4, 12, dict(dot_groups=0, waves=8)),
    ("few", 600_000, 256, 250, 8, 60, dict(dot_groups=0, waves=8)),
    ("many", 500_000, 64, 1000, 40, 40, dict(dot_groups=0)),
    ("units", 700_000, 128, 400, 4, 12, dict(dot_groups=0, waves=8))])
def test_scores_outside_the_normal_range(form, n, d, B, groups, vocab, plan, kind):
    w = ragged_workload(n + B, n, d, B, vocab, 30 if "own" in form else 12, 256, 1)
    pool = [[g % vocab] if form in ("four", "units", "many", "rows of 512") else [g % vocab, (g * 7 + 1 + g // vocab) % vocab]
            for g in range(groups)]
    filters = [pool[b % groups] for b in range(B)]
    w.filt_ids = np.array([x for f in filters for x in f], np.uint64)
    w.filt_offsets = np.concatenate([[0], np.cumsum([len(f) for f in filters])]).astype(np.int64)
    _extreme_scales(w, kind)
    K = 20
    got = st.st_search_host_plan(n, d, B, 1, K, 256, 1, w.filt_ids, w.filt_offsets)
    assert all(got[key] == v for key, v in plan.items()), got
    check_search(w, K, queries=range(0, B, max(1, B // 20)), label=f"{kind} scores, {form}")


# The same scan over rows of evaluated programs: few of them (all rows are staged) and more than 64 (the named ones are).
@pytest.mark.parametrize("n,B", [(300_011, 37), (270_400, 100), (400_000, 140)])
def test_own_programs(n, B):
    w = ragged_workload(n, n, 96, B, 24, 6, 128, 3)
    programs = [postfix(("and", ("leaf", b % 24), ("not", ("leaf", (b * 7 + 1 + b // 24) % 24)))) if b % 2 else
                postfix(("or", ("leaf", b % 24), ("leaf", (b // 24 + b + 3) % 24))) for b in range(B)]
    programs[3] = ([], [])
    check_expr_search(w, programs, 60, queries=sorted({0, 1, 2, 3, B - 1, *range(0, B, 9)}), label="own programs", fast_path_only=True)


# ... and behind cluster probing through mask rows, where most items pass for no query.
@pytest.mark.parametrize("n,d,B,n_c,n_p", [(800_003, 64, 17, 4000, 600), (900_000, 96, 70, 700, 520)])
def test_own_scan_behind_probing(n, d, B, n_c, n_p):
    w = ragged_workload(n, n, d, B, 24, 4, 64, 2)
    check_ivf(w, _programs(np.random.default_rng(n), B, 24), n_c, n_p, 50, queries=sorted({0, 1, 2, B - 1, *range(0, B, 12)}),
              label="own scan behind probing")


# The final ordering of K > 2048 cuts the score range into steps: scores of one size, a few far above the rest
# (cut again), spread over many powers of two, infinite ones, hundreds of keys to a score (general path), fewer
# passing items than K; one round of the key buffer and several.
@pytest.mark.parametrize("K", [2049, 16384, 17409, 40_000])
@pytest.mark.parametrize("kind", ["plain", "outliers", "spread", "ties", "few"])
def test_ordering_of_large_results(K, kind):
    n, B = 60_000, 3
    w = ragged_workload(900 + K, n, 16, B, 10, 3, 64, 2)
    w.filt_ids, w.filt_offsets = np.array([3], np.uint64), np.array([0, 1, 1, 1], np.int64)
    if kind == "outliers":
        w.item_scale[5::n // 7] *= 1e30
        w.item_scale[77] = float("inf")
    elif kind == "spread":
        w.item_scale = torch.from_numpy(np.exp2(np.random.default_rng(K).uniform(-60, 60, n)).astype(np.float32))
    elif kind == "ties":
        w.items = w.items[:60].repeat(n // 60, 1).contiguous()
        w.item_scale = w.item_scale[:60].repeat(n // 60).contiguous()
    elif kind == "few":
        w.filt_ids, w.filt_offsets = np.arange(9, dtype=np.uint64), np.array([0, 3, 6, 9], np.int64)
    check_search(w, K, label=f"ordering {kind}")


# Tied scores that overflow the regions: the slow exact path over several rounds of its buffer, with results above and
# below the LDS sort size (rounds of the large selection's 1024 threads and of the small one's 512).
@pytest.mark.parametrize("n,K", [(200_000, 3000), (300_001, 10_000), (200_000, 2048)])
def test_ties_on_the_slow_exact_path_over_several_rounds(n, K):
    w = ragged_workload(n + K, n, 16, 3, 10, 3, 64, 2)
    w.filt_ids, w.filt_offsets = np.array([3], np.uint64), np.array([0, 0, 1, 1], np.int64)
    w.items = w.items[:20].repeat(n // 20 + 1, 1)[:n].contiguous()
    w.item_scale = torch.full((n,), 0.01)
    check_search(w, K, slow_path=([0, 2], []), label="ties, slow path")


def _parts(n, B, n_c, n_p, K):
    """(workgroups to a query, keys of a workgroup's share, keys it hands on unpruned) by the host's rule."""
    k_pad = 1 << (K - 1).bit_length()
    room, scratch, words = K + 1024 * 512, k_pad if k_pad > 2048 else 0, n_p * (n // n_c // 64 + 1)
    parts = 1

    def fits(p):
        return p <= 16 and room // p - scratch >= 2 * K + 4096

    while fits(2 * parts) and 2 * B * parts <= 256 and words // (2 * parts) >= 64:
        parts *= 2
    while fits(2 * parts) and words // parts > 1024:
        parts *= 2
    return parts, room // parts - (scratch if parts > 1 else 0), max(K, 16384 // parts)


# What the workgroups of a probing query hand on, and its merge.  All clusters are probed and the first query has no
# filter, so that its n items go through: more than a workgroup hands on (pruned in LDS or in memory), more than its
# share of the key buffer holds (pruned on the way), one workgroup and 16, more results than a round of the merge holds,
# hundreds of keys to a score (the merge's general way), with the result ordered in LDS and in memory.
@pytest.mark.parametrize("n,B,K,kind,parts,pruned", [
    (100_000, 3, 1500, "plain", 16, "end"), (200_000, 3, 1500, "plain", 16, "end"), (200_000, 3, 3000, "plain", 16, "end"),
    (700_000, 2, 3000, "plain", 16, "round"), (700_000, 2, 10_000, "plain", 8, "round"), (60_000, 130, 3000, "plain", 1, "end"),
    (60_000, 130, 100, "plain", 1, "end"), (20_000, 3, 10_000, "plain", 4, "no"), (100_000, 3, 1500, "ties", 16, "end"),
    (200_000, 3, 3000, "ties", 16, "end"), (30_000, 20, 700, "ties", 4, "end"), (700_000, 2, 10_000, "ties", 8, "round"),
    (200_000, 3, 9000, "outliers", 8, "end")])
def test_probing_parts_and_merge(n, B, K, kind, parts, pruned):
    n_c = 50
    got, share, keep = _parts(n, B, n_c, n_c, K)
    mine = n // got
    assert got == parts and ("round" if mine > share else "end" if mine > keep else "no") == pruned, (got, share, keep, mine)
    w = ragged_workload(n + K, n, 16, B, 24, 4, 64, 2)
    if kind == "ties":
        w.items = w.items[:60].repeat(n // 60 + 1, 1)[:n].contiguous()
        w.item_scale = w.item_scale[:60].repeat(n // 60 + 1)[:n].contiguous()
    elif kind == "outliers":
        w.item_scale[5::n // 7] *= 1e30
    check_ivf(w, _programs(np.random.default_rng(n + B), B, 24), n_c, n_c, K, queries=sorted({0, 1, B - 1}), label=f"parts {kind}",
              fast_path_only=True)


# A lone workgroup with few words orders its query's keys itself, by the average cluster: here most items lie in one
# cluster that every query probes, or in clusters that none does.
@pytest.mark.parametrize("n,big,K", [(20_000, 0, 500), (20_000, 19_000, 500), (20_000, 7000, 2048), (300, 200, 512), (20_000, 19_999, 1),
                                     (40_000, 39_000, 2048)])
def test_probing_batch_with_few_words_to_a_query(n, big, K):
    B, n_c, n_p, d = 140, 400, 3, 16
    assert n_p * (n // n_c // 64 + 1) <= 64 and B > 128
    w = ragged_workload(n + big + K, n, d, B, 24, 4, 64, 2)
    programs = _programs(np.random.default_rng(n + B), B, 24)
    ops, ids, off = pack(programs)
    cent, cs, coff = S.gen_clusters(w.cfg, n_c)
    if big:  # cluster 7 wins every query (all queries' first value is positive); the others share the rest
        w.queries[:, 0] = 100
        cent[7] = 0
        cent[7, 0], cs[7] = 127, 1e6
        coff = torch.cat([torch.arange(8) * 0, torch.linspace(big, n, n_c - 7).long()]).contiguous()
    items, iscale, foff, fids, q, qs = [t.cuda() for t in (w.items, w.item_scale, w.feat_offsets, w.feat_ids, w.queries,
                                                           w.query_scale)]
    bloom = st.st_bloom_build(foff, fids, n, 64, 2)
    got = st.st_search_ivf(bloom, items, iscale, cent.cuda(), cs.cuda(), coff.cuda(), n_p, q, qs, ops, ids, off, K)
    got = [t.cpu().numpy() for t in got]
    sel = [0, 1, 2, 3, B - 1]
    want = O.search_ivf(oracle_index(w), 64, 2, w.items.numpy(), w.item_scale.numpy(), cent.numpy(), cs.numpy(), coff.numpy(), n_p,
                        w.queries.numpy()[sel], w.query_scale.numpy()[sel], *pack([programs[b] for b in sel]), K)
    if big:
        assert (got[3][:, 0] == 7).all() and got[2][0] >= min(K, big)
    for g, x in zip(got, want):
        x = np.asarray(x)
        assert np.array_equal(g[sel].view(np.uint32) if g.dtype == np.float32 else g[sel], x.view(np.uint32) if x.dtype == np.float32 else x)


# The scan by units of passing items (levels behind the first, one workgroup to a compute unit, filters broad enough that
# every wavefront fills units): each row length and number of tasks, filters with an odd number of 16-row blocks, up to
# 20 filters (several batches of eight), no filter, one that nothing passes, ragged last segment and word, few and many passing
# items (lists by lane and by word), more than 8 and 16 signature rows, scales of many sizes, scores that are all negative
# (no bound), tied scores, queries split over rows of workgroups.  units: whether the last level takes that form -- the
# host says whether it may, and from which count of passing pairs on; the others take it by another form: queries that do
# not fit its LDS, too few items for it, filters that pass little ("rare"), more filters than it takes ("many").
@pytest.mark.parametrize("n,d,B,T,groups,m,k,kind,units", [
    (700_001, 64, 700, 0, 5, 128, 2, "plain", True), (700_001, 64, 560, 0, 12, 256, 2, "plain", True),
    (800_049, 128, 420, 0, 8, 128, 2, "plain", True), (800_049, 128, 330, 0, 12, 256, 2, "plain", True),
    (1_450_003, 256, 240, 0, 7, 256, 3, "plain", True), (800_001, 256, 480, 0, 5, 128, 2, "plain", True),
    (690_031, 128, 1000, 0, 2, 64, 1, "dense", True), (950_017, 128, 420, 0, 4, 1024, 7, "long", True),
    (1_450_003, 256, 230, 0, 4, 1024, 7, "long", True), (710_000, 128, 450, 0, 6, 128, 2, "scales", True),
    (800_001, 256, 500, 0, 4, 128, 2, "negative", True), (700_000, 128, 400, 0, 3, 64, 2, "ties", True),
    (1_000_000, 64, 400, 4, 5, 128, 2, "plain", True), (1_050_003, 64, 360, 4, 13, 256, 2, "plain", True),
    (1_050_003, 128, 220, 4, 8, 128, 2, "plain", True), (800_001, 256, 130, 4, 5, 128, 2, "plain", True),
    (800_001, 256, 75, 4, 10, 256, 2, "plain", True), (1_050_003, 64, 700, 2, 6, 128, 2, "plain", True),
    (1_450_003, 256, 250, 2, 4, 128, 2, "plain", True), (1_050_003, 128, 800, 1, 5, 128, 2, "plain", True),
    (1_050_003, 128, 200, 4, 20, 256, 2, "negative", True),
    (700_001, 64, 900, 0, 5, 128, 2, "plain", False), (800_049, 128, 500, 0, 8, 128, 2, "plain", False),
    (900_000, 256, 240, 0, 7, 256, 3, "plain", False), (900_000, 256, 1000, 0, 5, 512, 4, "plain", True),
    (680_000, 64, 1100, 0, 31, 256, 3, "plain", False), (700_011, 256, 250, 0, 4, 1024, 7, "long", False),
    (700_000, 256, 260, 0, 4, 128, 2, "negative", False), (600_000, 256, 250, 0, 8, 512, 4, "rare", False),
    (760_000, 64, 200, 4, 7, 128, 2, "plain", False), (800_007, 128, 128, 4, 8, 128, 2, "plain", False),
    (470_000, 256, 110, 2, 5, 128, 2, "plain", False), (780_001, 128, 420, 1, 3, 128, 2, "plain", False),
    (860_000, 128, 130, 4, 12, 256, 3, "negative", False), (300_000, 64, 1000, 0, 40, 256, 3, "many", False),
    (900_000, 128, 400, 0, 8, 512, 4, "rare", False)])
def test_scan_by_units(n, d, B, T, groups, m, k, kind, units):
    rng = np.random.default_rng(n + d)
    vocab, feats = (40, 4) if kind == "rare" else (40, 30) if kind == "many" else (12, 12)
    w = ragged_workload(n + d, n, d, B, vocab, feats, m, k, T=T)
    pool = [[] if g == 1 and kind != "rare" else [999] if g == 2 else [g % vocab] if g % 3 == 0 or kind == "dense" else
            [g % vocab, *(int(x) for x in rng.choice(vocab, 2 if kind == "long" else 1))] for g in range(groups)]
    if units:  # (the hashes of ids that differ in the bits of a hash's number alone are the same)
        w.feat_ids = w.feat_ids * 8
        pool = [[8 * x for x in f] for f in pool]
    pick = np.concatenate([np.arange(groups), rng.integers(0, groups, B - groups)])
    filters = [pool[g] for g in pick]
    w.filt_ids = np.array([x for f in filters for x in f], np.uint64)
    w.filt_offsets = np.concatenate([[0], np.cumsum([len(f) for f in filters])]).astype(np.int64)
    if kind == "scales":
        w.item_scale = torch.from_numpy(np.exp2(rng.uniform(-20, 20, n)).astype(np.float32))
    elif kind == "negative":  # every score is below zero
        w.items = w.items.abs().clamp(1, 127).to(torch.int8)
        w.queries = (-w.queries.abs().clamp(1, 127).to(torch.int16)).to(torch.int8)
    elif kind == "ties":
        w.items = w.items[:997].repeat(n // 997 + 1, 1)[:n].contiguous()
        w.item_scale = w.item_scale[:997].repeat(n // 997 + 1)[:n].contiguous()
    K = 50
    plan = st.st_search_host_plan(n, d, B, max(T, 1), K, m, k, w.filt_ids, w.filt_offsets)
    assert plan["waves"] == 8 and plan["levels"] >= 2, plan
    sigs = oracle_index(w)
    passing = {g: int(np.unpackbits(O.bloom_mask(sigs, m, k, np.array(pool[g], np.uint64)).view(np.uint8)).sum()) for g in range(groups)}
    enough, pairs = st.st_search_host_units(n, d, B, max(T, 1), T > 0, K, m, k, w.filt_ids, w.filt_offsets)
    counted = pairs * np.mean([passing[g] for g in pick]) / n  # (but for the sample's chance: well below a tenth)
    assert (enough >= 0 and counted >= 1.1 * enough) if units else (enough < 0 or counted <= 0.9 * enough), (enough, pairs, counted)
    fast = [b for b in range(B) if passing[pick[b]] >= 40 * K] if kind not in ("ties", "scales") else []
    assert kind in ("ties", "scales") or len(fast) > B // 2
    check_search(w, K, sigs=sigs, queries=sorted({0, 1, 2, B - 1, *range(0, B, max(1, B // 14))}), slow_path=([], fast),
                 label=f"units {kind}")


# Small corpora take one kernel for the whole search: the smallest and largest of its range (and one item or query more), a
# lone query (it reads the pinned tables), several tasks, more than eight signature rows, fewer passing items than K, none,
# all, ties, results of one key and as many as LDS orders.
@pytest.mark.parametrize("n,d,B,T,m,k,K,kind", [
    (1, 16, 1, 0, 64, 2, 5, "plain"), (63, 64, 3, 0, 64, 2, 70, "plain"), (64, 32, 1, 0, 64, 2, 64, "all"), (1025, 48, 2, 3, 100, 3, 20, "plain"),
    (12_288, 64, 256, 0, 128, 2, 10, "plain"), (12_288, 32, 257, 0, 128, 2, 10, "plain"), (12_289, 64, 2, 0, 128, 2, 10, "plain"),
    (12_288, 64, 1, 0, 128, 2, 2048, "all"), (12_288, 64, 5, 0, 128, 2, 2048, "ties"), (10_000, 64, 1, 0, 1024, 7, 1, "long"),
    (3_125, 128, 9, 0, 256, 3, 300, "plain"), (3_126, 128, 9, 0, 256, 3, 300, "plain"), (1_500, 256, 4, 0, 256, 3, 1500, "plain"),
    (2_000, 64, 7, 4, 256, 3, 100, "long"), (5_000, 64, 20, 0, 512, 4, 2049, "plain")])
def test_small_corpora(n, d, B, T, m, k, K, kind):
    w = ragged_workload(n + d + B, n, d, B, 12, 6, m, k, T=T)
    if kind == "all":
        w.filt_ids, w.filt_offsets = np.zeros(0, np.uint64), np.zeros(B + 1, np.int64)
    elif kind == "long":
        w.filt_ids, w.filt_offsets = np.tile(np.arange(3, dtype=np.uint64), B), np.arange(0, 3 * B + 1, 3).astype(np.int64)
    elif kind == "ties":
        w.items = w.items[:20].repeat(n // 20 + 1, 1)[:n].contiguous()
        w.item_scale = torch.full((n,), 0.01)
    if B > 2 and kind == "plain":  # nothing passes for one query
        w.filt_ids = np.concatenate([w.filt_ids, np.array([999_999], np.uint64)])
        w.filt_offsets[B] += 1
    check_search(w, K, label=f"small {kind}")


# ... also within a graph: a lone query's kernel reads the pinned tables at every replay.
@pytest.mark.parametrize("B", [1, 9])
def test_captured_search_over_a_small_corpus(B):
    n = 9000
    w = S.make_workload(S.scaled(S.CONFIGS["tiny"], n, batch=B, top_k=20), "cuda")
    cfg = w.cfg
    bloom = st.st_bloom_build(w.feat_offsets, w.feat_ids, n, cfg.m_bits, cfg.k_hashes)
    buf, other = st.SearchBuffers(n, cfg.d, B, 1, 20), st.SearchBuffers(n, cfg.d, B, 1, 20)

    def call(b, ids=w.filt_ids):
        return st.st_search(bloom, w.items, w.item_scale, w.queries, w.query_scale, ids, w.filt_offsets, 20, buffers=b)

    _replays_like_eager(call, buf, lambda: call(other, w.filt_ids + np.uint64(1)))
