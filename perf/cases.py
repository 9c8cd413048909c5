"""Timed cases of the retrieval library: what a program that uses it has it do, from the smallest
call to the largest, through the public entry points of ``paper_2511_14881_amd.binding``.

Corpora, features, queries and filters come from the repository's own seeded generators
(``synth``), on the GPU; the sizes are those of its five workloads, of the variants ``bench.py``
reports beside them, and odd ones in between.
"""
from __future__ import annotations

import math

import numpy as np
import torch

from paper_2511_14881_amd import binding as st
from paper_2511_14881_amd import synth

# Formula of the Value Model cases: if s2 > 0.5 then 0.4*s0 + 0.3*s1 + 0.2*s2 + 0.1*s3 else
# min(s0, s1) * 0.5, in postfix order (operation, constant); task t's score is operation t << 8.
_FORMULA = [(2 << 8, 0.0), (1, 0.5), (7, 0.0),
            (1, 0.4), (0 << 8, 0.0), (4, 0.0), (1, 0.3), (1 << 8, 0.0), (4, 0.0), (2, 0.0),
            (1, 0.2), (2 << 8, 0.0), (4, 0.0), (2, 0.0), (1, 0.1), (3 << 8, 0.0), (4, 0.0), (2, 0.0),
            (0 << 8, 0.0), (1 << 8, 0.0), (5, 0.0), (1, 0.5), (4, 0.0), (8, 0.0)]

_SEARCHES = ("search", "multitask", "programs", "probe")


def _search(name, kind="search", *, n, d, batch, k, tasks=0, bits=256, hashes=3, terms=2, feats=8, vocab=100_000,
            zipf=1.1, dist="gauss", sel=0.10, pool=8, clusters=0, probes=0):
    case = {"kind": kind, "n": n, "d": d, "batch": batch, "k": k, "tasks": tasks, "bits": bits, "hashes": hashes,
            "terms": terms, "feats": feats, "vocab": vocab, "zipf": zipf, "dist": dist, "sel": sel, "pool": pool,
            "clusters": clusters, "probes": probes}
    if name:
        case["name"] = name
    return case


def listed():
    return [
        # one visitor against a small catalogue: launches and latency are all there is
        _search("tiny-1", n=10_000, d=64, batch=1, k=10, bits=64, hashes=2, terms=1, feats=4, vocab=1_000, zipf=0.0,
                dist="uniform", sel=0.0, pool=1),
        # an ordinary online batch on one index of a million items
        _search("mid-64", n=1_000_000, d=128, batch=64, k=100),
        # the largest index whose batch is bound by memory
        _search("large-256", n=10_000_000, d=256, batch=256, k=500, bits=512, hashes=4, terms=3, feats=16, vocab=1_000_000,
                zipf=1.05, sel=0.05),
        # the same index, and every visitor brings a filter of their own (no sharing within the batch)
        _search("large-own-filters-256", n=10_000_000, d=256, batch=256, k=500, bits=512, hashes=4, terms=3, feats=16,
                vocab=1_000_000, zipf=1.05, sel=0.05, pool=256),
        # several objectives per visitor, one weighted list
        _search("multi-128x4", "multitask", n=5_000_000, d=128, batch=128, k=200, tasks=4),
        # offline scoring of many users at once under broad filters: a dense contraction
        _search("broad-1024", n=20_000_000, d=128, batch=1024, k=1000, bits=128, hashes=2, terms=1, sel=0.50, pool=2),
        # a pre-filter that hands ten thousand items each to a later ranking stage
        _search("prefilter-k10000", n=1_000_000, d=128, batch=64, k=10_000),
        # AND / OR / NOT filters on an index of odd sizes (a row length that is no power of two, a ragged last tile)
        _search("programs-odd-37", "programs", n=777_777, d=96, batch=37, k=77),
        # cluster probing in front of the filter: a small batch against a large index
        _search("probe-16", "probe", n=20_000_000, d=128, batch=16, k=2048, clusters=4096, probes=32),
        # publishing: the filter index of a corpus is built and its signatures are exported for storage
        {"name": "build-10m", "kind": "build", "n": 10_000_000, "bits": 512, "hashes": 4, "feats": 16, "vocab": 1_000_000,
         "zipf": 1.05},
        # publishing: an fp32 embedding table is quantised
        {"name": "quantize-2m", "kind": "quantize", "n": 2_000_000, "d": 256},
        # a Value Model formula over the task scores of every item
        {"name": "formula-10m", "kind": "formula", "n": 10_000_000, "tasks": 4},
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def _cost_ms(c):
    """Rough upper estimate of a search, to keep drawn cases below the largest listed ones."""
    tasks = max(c["tasks"], 1)
    pairs = c["n"] * c["batch"] * tasks * max(c["sel"], 0.01)
    dense = c["d"] in (64, 128, 256, 512) and tasks in (1, 2, 4) and c["pool"] < c["batch"]
    ops = pairs * c["d"] / (4e11 if dense else 1e10)
    rows = min(c["pool"], c["batch"]) * c["n"] * (c["terms"] * c["hashes"] / 8 + max(c["sel"], 0.01) * (c["d"] + 4)) / 3e9
    return ops + rows + c["batch"] * c["k"] / 1e6


def draw(rng):
    kind = rng.choice(("search",) * 5 + ("multitask",) * 2 + ("programs",) * 2 + ("probe", "build", "quantize", "formula"))
    if kind == "build":
        feats = rng.randint(2, 24)
        return {"kind": kind, "n": _log(rng, 10_000, 100_000_000 // feats), "bits": rng.choice((64, 100, 128, 256, 512, 768)),
                "hashes": rng.randint(2, 5), "feats": feats, "vocab": rng.choice((10_000, 100_000, 1_000_000)), "zipf": 1.1}
    if kind == "quantize":
        d = rng.choice((32, 48, 64, 96, 128, 200, 256, 384, 512, 768))
        return {"kind": kind, "n": _log(rng, 1_000, 500_000_000 // d), "d": d}
    if kind == "formula":
        return {"kind": kind, "n": _log(rng, 1_000, 10_000_000), "tasks": rng.randint(4, 8)}
    d = rng.choice((32, 64, 64, 96, 128, 128, 128, 192, 256, 256, 384, 512, 768))
    c = _search(None, kind, n=_log(rng, 10_000, min(20_000_000, 2_560_000_000 // d)), d=d, batch=_log(rng, 1, 512),
                k=_log(rng, 10, 4000), bits=rng.choice((128, 256, 256, 512)), hashes=rng.randint(2, 4), terms=rng.randint(1, 3),
                feats=rng.choice((4, 8, 8, 12, 16)), sel=rng.choice((0.005, 0.01, 0.02, 0.05, 0.1, 0.2)),
                pool=rng.choice((1, 2, 8, 8, 16)))
    if kind == "multitask":
        c["tasks"] = rng.choice((2, 3, 4, 4))
    if kind == "search" and rng.random() < 0.3:
        c["pool"] = c["batch"]  # a filter of their own for every query
    c["k"] = min(c["k"], c["n"] // 8)
    while _cost_ms(c) > 4.0:
        if c["batch"] > 4:
            c["batch"] = c["batch"] * 2 // 3
        else:
            c["n"] = c["n"] * 2 // 3
        c["k"] = min(c["k"], c["n"] // 8)
    c["pool"] = min(c["pool"], c["batch"])
    if kind == "probe":
        c["clusters"] = max(8, min(16_384, int(math.sqrt(c["n"]) * rng.uniform(0.5, 2.0))))
        c["probes"] = min(c["clusters"], _log(rng, 4, 128))
    return c


def _config(case, seed):
    return synth.Config("case", case["n"], case.get("d", 64), case.get("batch", 1), case.get("tasks", 0), case["bits"],
                        case["hashes"], case.get("terms", 1), case.get("k", 1), case["feats"], case["vocab"], case["zipf"],
                        case.get("dist", "gauss"), case.get("sel", 0.1), case.get("pool", 1), seed=seed)


def prepare(case, seed):
    kind = case["kind"]
    if kind == "quantize":
        gen = torch.Generator(device="cuda").manual_seed(seed)
        return {"kind": kind, "x": torch.randn((case["n"], case["d"]), generator=gen, device="cuda")}
    if kind == "formula":
        gen = torch.Generator(device="cuda").manual_seed(seed)
        return {"kind": kind, "scores": torch.rand((case["n"], case["tasks"]), generator=gen, device="cuda"),
                "ops": np.array([f[0] for f in _FORMULA], np.int32), "consts": np.array([f[1] for f in _FORMULA], np.float32),
                "out": torch.empty(case["n"], device="cuda")}
    cfg = _config(case, seed)
    if kind == "build":
        offsets, ids = synth.gen_features(cfg, "cuda")
        return {"kind": kind, "cfg": cfg, "offsets": offsets, "ids": ids, "bloom": None}
    w = synth.make_workload(cfg, "cuda")
    s = {"kind": kind, "cfg": cfg, "w": w, "bloom": st.st_bloom_build(w.feat_offsets, w.feat_ids, cfg.n_items, cfg.m_bits,
                                                                      cfg.k_hashes)}
    w.feat_offsets = w.feat_ids = None  # a serving program keeps the index, not the lists it was built from
    tasks = max(cfg.n_tasks, 1)
    if kind in ("programs", "probe"):
        s["ops"], s["ids"], s["off"], _ = synth.gen_filter_programs(cfg, pool=case["pool"])
    if kind == "probe":
        s["clusters"] = synth.gen_clusters(cfg, case["clusters"], "cuda")
        s["probes"] = case["probes"]
        s["buffers"] = st.IvfBuffers(cfg.n_items, cfg.d, cfg.batch, cfg.top_k, case["clusters"], case["probes"], int(s["off"][-1]))
    else:
        s["buffers"] = st.SearchBuffers(cfg.n_items, cfg.d, cfg.batch, tasks, cfg.top_k,
                                        n_expr_entries=int(s["off"][-1]) if kind == "programs" else None)
    return s


def run(s):
    kind = s["kind"]
    if kind == "quantize":
        return st.st_quantize_global(s["x"])
    if kind == "formula":
        return st.st_value_model(s["scores"], s["ops"], s["consts"], out=s["out"])
    cfg = s["cfg"]
    if kind == "build":
        # the new index takes the place of the one that the program held so far
        s["bloom"] = st.st_bloom_build(s["offsets"], s["ids"], cfg.n_items, cfg.m_bits, cfg.k_hashes)
        return st.st_bloom_export_signatures(s["bloom"])
    w, buf = s["w"], s["buffers"]
    if kind == "search":
        return st.st_search(s["bloom"], w.items, w.item_scale, w.queries, w.query_scale, w.filt_ids, w.filt_offsets, cfg.top_k,
                            buffers=buf)
    if kind == "multitask":
        return st.st_search_multitask(s["bloom"], w.items, w.item_scale, w.queries, w.query_scale, w.task_weight, w.filt_ids,
                                      w.filt_offsets, cfg.top_k, buffers=buf)
    if kind == "programs":
        return st.st_search_expr(s["bloom"], w.items, w.item_scale, w.queries, w.query_scale, s["ops"], s["ids"], s["off"],
                                 cfg.top_k, buffers=buf)
    cent, cent_scale, cent_off = s["clusters"]
    return st.st_search_ivf(s["bloom"], w.items, w.item_scale, cent, cent_scale, cent_off, s["probes"], w.queries, w.query_scale,
                            s["ops"], s["ids"], s["off"], cfg.top_k, buffers=buf)


def work(case):
    """Bytes and operations of one pass: feature lists, tables and scores once in and once out; of a search, the
    signature rows its distinct filters name, the rows of the items that pass some filter (by the selectivity
    asked for), the dot products of the passing pairs, queries and results."""
    kind = case["kind"]
    n = case["n"]
    if kind == "quantize":
        return {"bytes": n * (5 * case["d"] + 4), "flops": 2 * n * case["d"]}
    if kind == "formula":
        return {"bytes": n * (4 * case["tasks"] + 4), "flops": n * 14}
    words = (n + 63) // 64
    if kind == "build":
        return {"bytes": 8 * (n + 1) + 8 * n * case["feats"] + 2 * 8 * words * case["bits"] + 8 * n * ((case["bits"] + 63) // 64),
                "flops": 0}
    tasks, d = max(case["tasks"], 1), case["d"]
    sel = case["feats"] / case["vocab"] if case["zipf"] == 0 else case["sel"]
    filters = min(case["pool"], case["batch"])
    leaves = case["terms"] * case["hashes"]
    if kind in ("programs", "probe"):
        sel, leaves = 0.10, 3.5 * case["hashes"]  # a broad term AND (b OR c), every second one AND NOT a fourth
    union = 1 - (1 - sel) ** filters
    out = case["batch"] * (case["k"] * 12 + 4) + case["batch"] * tasks * (d + 4)
    if kind == "probe":
        share = min(1.0, case["probes"] / case["clusters"])
        seen = n * share * case["batch"]
        return {"bytes": case["clusters"] * (d + 12) + seen * (leaves / 8 + sel * (d + 4)) + out,
                "flops": 2 * d * case["batch"] * case["clusters"] + 2 * d * seen * sel}
    rows = min(filters * leaves, 32 * case["hashes"], case["bits"])  # filters name the 32 most frequent features
    return {"bytes": rows * words * 8 + union * n * (d + 4) + out, "flops": 2 * d * tasks * n * sel * case["batch"]}


def tolerance(case):
    """Every result is defined bit for bit: masks and int32 dot products are exact, a score is two correctly rounded
    fp32 products, an aggregate a fixed chain of fmaf, ties go to the lower id."""
    return "exact"
