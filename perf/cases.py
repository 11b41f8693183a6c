"""Timed cases: what a program does with this library once an index stands, and the two steps of
index construction that run on the GPU.

A case is a dict of plain values; `listed()` gives the fixed ones, `draw(rng)` another one of the
same ranges.  `prepare(case, seed)` makes what the program has in hand before the call -- queries
or vectors from the seed, and the index handle, which does not depend on the seed: a program
uploads an index once and sends it many batches.  `run(state)` is one call through the binding.

The data are the seeded Gaussian mixtures of datagen.py (same parameters, drawn on the GPU), cut to
sizes whose index is built in seconds; index sizes, list counts, batch sizes, K, bigK and nprobe
are those of datagen.WORKLOADS, bench.py and its variants where they are listed.
"""
from __future__ import annotations

import math
from collections import OrderedDict
from dataclasses import replace

import numpy as np
import torch

from paper_2601_07183_amd import binding, datagen, index_build

INDEX_SEED = 20                      # of the mixture's base vectors; queries come from the case's seed
KEPT_INDEXES = 16                    # uploaded indexes that stay on the GPU, least recently used first out


def _case(name, op, kind, n, d, M, nlist, **kw):
    c = dict(name=name, op=op, kind=kind, n=n, d=d, M=M, nlist=nlist, comps=1000, metric="l2")
    c.update(kw)
    return c


def _search(name, index, nq, k, refine_k, nprobe, mode="eager", **kw):
    return _case(name, "search", **index, nq=nq, k=k, refine_k=refine_k, nprobe=nprobe, mode=mode, **kw)


TINY = dict(kind="gmm", n=20_000, d=32, M=16, nlist=64, comps=100)
SIFT = dict(kind="sift", n=1_000_000, d=128, M=64, nlist=1024)
DENSE = dict(kind="dense", n=200_000, d=960, M=240, nlist=1024)
SPHERE = dict(kind="sphere", n=2_000_000, d=96, M=48, nlist=4096, comps=4000)
SPHERE_IP = dict(kind="sphere", n=200_000, d=96, M=48, nlist=1024, comps=4000, metric="ip")
BYTES = dict(kind="sift", n=8_000_000, d=128, M=64, nlist=16384, comps=10_000)


def listed():
    return [
        # the smallest call: one query against an index of a few megabytes (a lookup inside another service)
        _search("small_index_one_query", TINY, 1, 10, 40, 4),
        # one query at a time against the 1M x 128 index: interactive search, latency counts
        _search("one_query", SIFT, 1, 10, 100, 23),
        # the same recorded once as a HIP graph and replayed
        _search("one_query_graph", SIFT, 1, 10, 100, 23, mode="graph"),
        # a small batch, as a server that gathers requests for a few milliseconds sees
        _search("batch_of_100", SIFT, 100, 10, 100, 32),
        # the throughput workload: 10,000 queries at the nprobe that reaches recall@10 0.9
        _search("batch_of_10000", SIFT, 10_000, 10, 100, 23),
        # many results per query (K = 100, bigK = 400), a ragged batch
        _search("top_100", SIFT, 2_999, 100, 400, 32),
        # high-dimensional vectors: 960 dimensions, M = 240
        _search("dim_960", DENSE, 1_000, 10, 100, 45),
        # unit vectors, 4,096 lists
        _search("unit_vectors", SPHERE, 10_000, 10, 100, 39),
        # inner-product index with SOAR's second lists, an odd batch size
        _search("inner_product", SPHERE_IP, 777, 10, 100, 16),
        # the largest: byte vectors, 16,384 lists, bigK = 200, high nprobe
        _search("byte_vectors_16384_lists", BYTES, 10_000, 10, 200, 98),
        # construction: PQ codes of a million vectors
        _case("encode_1m", "encode", **SIFT),
        # construction: the two lists of each of a million vectors
        _case("assign_1m", "assign", **SIFT, n_cands=10),
    ]


def _log_uniform(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


# (dimension, sub-quantizers, kind): vector lengths in use, mostly two dimensions a sub-quantizer
SHAPES = ((32, 16, "gmm"), (48, 24, "gmm"), (64, 32, "sift"), (96, 48, "sphere"), (100, 50, "sphere"),
          (128, 64, "sift"), (128, 64, "sift"), (128, 32, "sift"), (200, 100, "dense"), (256, 64, "dense"),
          (256, 128, "dense"), (480, 240, "dense"), (960, 240, "dense"))


def draw(rng):
    op = rng.choice(("search",) * 6 + ("encode", "assign"))
    d, M, kind = rng.choice(SHAPES)
    most = 400_000 if d <= 128 else 60_000
    metric = "ip" if op == "search" and kind == "sphere" and rng.random() < 0.5 else "l2"
    n = _log_uniform(rng, 20_000, 150_000 if metric == "ip" else most)
    nlist = _log_uniform(rng, max(64, n // 2000), max(128, min(2048, n // 150)))
    c = _case("", op, kind, n, d, M, nlist, comps=200, metric=metric)
    del c["name"]
    if op == "search":
        k, refine_k = rng.choice(((1, 10), (10, 40), (10, 100), (10, 100), (10, 200), (100, 400)))
        nprobe = _log_uniform(rng, 1, min(128, nlist))
        nq = _log_uniform(rng, 1, 10_000)
        # no dearer than the largest listed case
        cap = 5e10 / (nprobe * (2.0 * n / nlist) * M)
        c.update(nq=max(1, min(nq, int(cap))), k=k, refine_k=refine_k, nprobe=nprobe,
                 mode="graph" if nq <= 8 and rng.random() < 0.5 else "eager")
    elif op == "assign":
        c.update(n=_log_uniform(rng, 1_000, most), n_cands=rng.choice((5, 10, 10, 20)))
    else:
        c.update(n=_log_uniform(rng, 1_000, 128_000_000 // d))
    return c


# ---- data ----------------------------------------------------------------------------------------


def _workload(case):
    base = {"gmm": "tiny", "sift": "sift1m", "dense": "gist1m", "sphere": "sphere10m"}[case["kind"]]
    # 8M vectors and more are kept as bytes, as the 100M workload's are
    return replace(datagen.WORKLOADS[base], name="perf", n=case["n"], d=case["d"], comps=case["comps"],
                   nlist=case["nlist"], M=case["M"], raw_u8=case["kind"] == "sift" and case["n"] >= 8_000_000)


_mixtures = OrderedDict()


def _mixture(case):
    """The mixture's parameters on the GPU (datagen's, seeded there)."""
    key = (case["kind"], case["d"], case["comps"])
    if key not in _mixtures:
        m = datagen.Mixture(_workload(case))
        dev = {k: torch.from_numpy(np.ascontiguousarray(v)).cuda() for k, v in
               dict(mean=m.mean, basis=m.basis, scale=getattr(m, "scale", None)).items() if v is not None}
        _mixtures[key] = (m.sigma, m.rank, m.spread, dev)
        while len(_mixtures) > KEPT_INDEXES:
            _mixtures.popitem(last=False)
    return _mixtures[key]


def _vectors(case, n, seed, as_u8=False):
    """n vectors of the case's mixture on the GPU, datagen's recipe with torch's generator."""
    sigma, rank, spread, p = _mixture(case)
    d, kind = case["d"], case["kind"]
    g = torch.Generator(device="cuda")
    g.manual_seed(seed)
    out = torch.empty((n, d), dtype=torch.uint8 if as_u8 else torch.float32, device="cuda")
    step = max(1, (1 << 27) // (d * max(1, rank)))
    for lo in range(0, n, step):
        m = min(n, lo + step) - lo
        comp = torch.randint(0, case["comps"], (m,), generator=g, device="cuda")
        x = torch.randn((m, d), generator=g, device="cuda") * sigma + p["mean"][comp]
        if rank:
            z = torch.randn((m, rank), generator=g, device="cuda")
            x += spread * (z[:, :, None] * p["basis"][comp]).sum(1)
        if kind == "sift":
            x = x.round_().clamp_(0.0, 255.0)
        elif kind == "dense":
            x = (x * p["scale"]).clamp_(min=0.0)
        elif kind == "sphere":
            x /= x.norm(dim=1, keepdim=True).clamp_(min=1e-12)
        out[lo:lo + m] = x
    return out


def _train_pq(x, M):
    # (sums of floats by index are added in a fixed order, so that every process trains the same codebook)
    before = torch.are_deterministic_algorithms_enabled()
    torch.use_deterministic_algorithms(True)
    try:
        return index_build.train_pq(x, M, 8, 7)
    finally:
        torch.use_deterministic_algorithms(before)


_codebooks = OrderedDict()


def _codebook(case):
    """PQ codebook [M][16][d/M] on the GPU."""
    key = (case["kind"], case["d"], case["M"], case["comps"])
    if key not in _codebooks:
        x = _vectors(case, 32_768, INDEX_SEED + 1).cpu().numpy()
        _codebooks[key] = torch.from_numpy(_train_pq(x, case["M"])).cuda()
        while len(_codebooks) > KEPT_INDEXES:
            _codebooks.popitem(last=False)
    return _codebooks[key]


_indexes = OrderedDict()


def _index(case, n):
    """The uploaded index over n vectors of the case's mixture."""
    key = (case["kind"], n, case["d"], case["M"], case["nlist"], case["comps"], case["metric"])
    if key in _indexes:
        _indexes.move_to_end(key)
        return _indexes[key]
    w = _workload(dict(case, n=n))
    base = _vectors(case, n, INDEX_SEED, as_u8=w.raw_u8).cpu().numpy()
    centroids = index_build.kmeans(base, w.nlist, 4, 3, max_train=max(65_536, 8 * w.nlist))
    hx = index_build.add_vectors(base, centroids, _codebook(case).cpu().numpy(), metric=case["metric"],
                                 lam=1.0 if case["metric"] == "ip" else 0.5)
    _indexes[key] = binding.Index(hx)
    while len(_indexes) > KEPT_INDEXES:
        _indexes.popitem(last=False)
    return _indexes[key]


# ---- one case ------------------------------------------------------------------------------------


def prepare(case, seed):
    s = dict(op=case["op"])
    if case["op"] == "encode":
        s.update(codebook=_codebook(case), x=_vectors(case, case["n"], seed))
        return s
    if case["op"] == "assign":
        # the handle carries the centroids; its own vectors play no part, a few are enough
        s.update(index=_index(case, max(20_000, 8 * case["nlist"])), x=_vectors(case, case["n"], seed), n_cands=case["n_cands"])
        return s
    ix = _index(case, case["n"])
    q = _vectors(case, case["nq"], seed)
    s.update(index=ix, q=q, k=case["k"], nprobe=case["nprobe"], refine_k=case["refine_k"], graph=None)
    if case["mode"] == "graph":
        ids = torch.empty((case["nq"], case["k"]), dtype=torch.int64, device="cuda")
        dists = torch.empty((case["nq"], case["k"]), dtype=torch.float32, device="cuda")
        stream = torch.cuda.Stream()
        stream.wait_stream(torch.cuda.current_stream())
        s.update(out=(ids, dists), graph=ix.graph(q, case["k"], case["nprobe"], case["refine_k"], ids, dists, stream))
        torch.cuda.current_stream().wait_stream(stream)
    return s


def run(s):
    if s["op"] == "encode":
        return binding.pq_encode(s["codebook"], s["x"])
    if s["op"] == "assign":
        return s["index"].assign(s["x"], n_cands=s["n_cands"])
    if s["graph"] is not None:
        s["graph"].launch()
        return s["out"]
    return s["index"].search(s["q"], s["k"], s["nprobe"], s["refine_k"])


def work(case):
    """Each input read once and each output written once; operations of the defined arithmetic."""
    d, M, n, nlist = case["d"], case["M"], case["n"], case["nlist"]
    if case["op"] == "encode":
        # a difference, a square and a sum per dimension and codeword, a comparison per codeword
        return {"bytes": n * (4.0 * d + M / 2) + 64.0 * d, "flops": n * 16.0 * (3 * d + M)}
    if case["op"] == "assign":
        # distances as a product with the centroids, then two sums per candidate
        return {"bytes": n * (4.0 * d + 8) + 4.0 * nlist * d, "flops": n * (2.0 * nlist * d + 6.0 * case["n_cands"] * d)}
    nq, nprobe, refine_k = case["nq"], case["nprobe"], case["refine_k"]
    items = 2.0 * n / nlist                     # per list: every vector is in two
    row = d if case["kind"] == "sift" else 4 * d
    lists = min(nlist, nq * nprobe)
    nbytes = (4.0 * nq * d + 12.0 * nq * case["k"] + 4.0 * nlist * d + 64.0 * d + lists * items * M / 2 +
              min(nq * refine_k, n) * float(row))
    flops = 2.0 * nq * nlist * d + 48.0 * nq * d + nq * nprobe * items * M + 3.0 * nq * refine_k * d
    return {"bytes": nbytes, "flops": flops}


def tolerance(case):
    """The order of every floating-point operation that decides a result is part of the interface
    (include/rairs.h), and ties are broken by id: two correct implementations give the same bits."""
    return "exact"
