"""The few-query search (queries that share few lists) against the oracle: ids, distances and DCO."""
import numpy as np
import pytest
import torch

from oracle import oracle
from paper_2601_07183_amd import datagen
from paper_2601_07183_amd import index_build as ib

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def binding():
    from paper_2601_07183_amd import binding as b
    b.load()
    return b


def _check(binding, hx, q, cases):
    ox = oracle.OracleIndex(hx)
    ix = binding.Index(hx)
    try:
        dq = torch.from_numpy(np.ascontiguousarray(q, dtype=np.float32)).cuda()
        for nq, k, nprobe, refine_k in cases:
            print(f"case: n={hx.ntotal} d={hx.d} M={hx.M} nlist={hx.nlist} nq={nq} k={k} nprobe={nprobe} "
                  f"refine_k={refine_k}", flush=True)
            want = oracle.search(ox, q[:nq], k, nprobe, refine_k)
            ids, dists = ix.search(dq[:nq], k, nprobe, refine_k)
            torch.cuda.synchronize()
            assert (ids.cpu().numpy() == want.ids).all()
            # both sides sum in the defined order: equal bits
            assert (dists.cpu().numpy() == want.dists).all()
            assert (ix.dco(nq) == want.dco).all()
            assert ix.scan_kernel_name() == "few_scan_kernel"
            st = ix.scan_stats()
            assert st["queries"] == nq and st["survivors"] == st["logged"] > 0       # kept without a log
    finally:
        ix.free()


# M: whole code dwords (16, 48, 64), a partial last dword (24, 50), more than four dwords (240);
# d: whole and partial rounds of 64 dimensions
@pytest.mark.parametrize("d,M,metric", [(32, 16, "l2"), (128, 64, "l2"), (96, 48, "ip"), (48, 24, "l2"),
                                        (100, 50, "ip"), (960, 240, "l2"), (36, 12, "l2")])
def test_shapes(binding, d, M, metric):
    g = np.random.Generator(np.random.PCG64(d + M))
    n, nlist = 6000, 80
    base = (g.standard_normal((n, d)) + 3.0 * g.standard_normal((40, d))[g.integers(0, 40, n)]).astype(np.float32)
    q = (g.standard_normal((70, d)) + 3.0 * g.standard_normal((40, d))[g.integers(0, 40, 70)]).astype(np.float32)
    hx = ib.build_index(base, nlist, M, seed=3, coarse_iters=4, pq_iters=4, metric=metric)
    # one query, three (a query per front tile), five (a partial tile of four), the most that share
    # few enough lists; nprobe 1 with lists shorter than bigK (no bound), every list
    _check(binding, hx, q, [(1, 10, 4, 40), (3, 1, 80, 10), (5, 100, 7, 400), (64, 10, 5, 100), (70, 10, 1, 200),
                            (4, 1000, 80, 1024)])


def test_full_buffers_and_ties(binding):
    # every vector identical: no bound excludes anything, a workgroup's buffer is cut to the bigK
    # best again and again, and ids alone decide; more candidates than the finish kernel keeps in LDS
    count, nlist = 40_000, 64
    x = np.tile(datagen.random_vectors(50, 1, 8), (count, 1))
    q = datagen.random_vectors(51, 4, 8)
    cents = datagen.random_vectors(52, nlist, 8)
    cb = ib.train_pq(datagen.random_vectors(53, 300, 8), 4, 5, 2)
    g = np.random.Generator(np.random.PCG64(3))
    asg = np.sort(g.integers(0, nlist, size=(count, 2)), axis=1).astype(np.int32)
    hx = ib.add_vectors(x, cents, cb, assign=asg)
    _check(binding, hx, q, [(1, 10, 64, 64), (4, 5, 64, 1024), (4, 1, 3, 1), (2, 64, 64, 600)])


def test_equal_centroids_and_large_directory(binding):
    # centroids in groups of identical rows: list ids decide among equal distances, also at the
    # nprobe-th place; a directory of several thousand lists (four and sixteen keys per thread)
    g = np.random.Generator(np.random.PCG64(9))
    for nlist in (1500, 5000):
        n, d = 8000, 16
        base = g.standard_normal((n, d)).astype(np.float32)
        cents = np.repeat(g.standard_normal((nlist // 50, d)).astype(np.float32), 50, axis=0)
        cb = ib.train_pq(base[:2000], 8, 4, 2)
        asg = np.sort(g.integers(0, nlist, size=(n, 2)), axis=1).astype(np.int32)
        hx = ib.add_vectors(base, cents, cb, assign=asg)
        q = g.standard_normal((9, d)).astype(np.float32)
        _check(binding, hx, q, [(1, 10, 30, 40), (9, 10, 75, 100), (9, 5, 256, 50)])


def test_deleted_items(binding):
    g = np.random.Generator(np.random.PCG64(4))
    base = (0.1 * g.standard_normal((5000, 32)) + g.standard_normal((10, 32))[g.integers(0, 10, 5000)]).astype(np.float32)
    hx = ib.build_index(base, 64, 16, seed=3, coarse_iters=4, pq_iters=4)
    hx = ib.delete_ids(hx, g.permutation(5000)[:2500])
    _check(binding, hx, base[:20], [(1, 10, 8, 40), (20, 10, 12, 100), (3, 10, 64, 1024)])


# which search a batch takes: thousands of queries that only meet many distances (16,384 lists), or lists
# that are large where the average one is small, are list-major batches; both ways agree
@pytest.mark.parametrize("nlist,d,big,nprobe,few_nq,lm_nq", [(16384, 16, 0, 1, 200, 3000), (64, 32, 40000, 4, 100, 1500)])
def test_route(binding, nlist, d, big, nprobe, few_nq, lm_nq):
    g = np.random.Generator(np.random.PCG64(nlist))
    n = 2000 + big
    cents = g.standard_normal((nlist, d)).astype(np.float32)
    asg = np.sort(g.integers(0, nlist, size=(n, 2)), axis=1).astype(np.int32)
    asg[2000:] = (0, 1)
    base = g.standard_normal((n, d)).astype(np.float32)
    hx = ib.add_vectors(base, cents, ib.train_pq(base[:2000], 16, 3, 2), assign=asg)
    q = g.standard_normal((lm_nq, d)).astype(np.float32)
    ix = binding.Index(hx)
    try:
        dq = torch.from_numpy(q).cuda()
        for nq, few in ((1, True), (few_nq, True), (lm_nq, False)):
            print("case: route", nlist, d, nprobe, nq, flush=True)
            ix.set_scan_mode(False, list_major=True)
            want = ix.search(dq[:nq], 10, nprobe, 40)
            ix.set_scan_mode(False)
            ids, dists = ix.search(dq[:nq], 10, nprobe, 40)
            torch.cuda.synchronize()
            assert (ix.scan_kernel_name() == "few_scan_kernel") == few
            assert (ids == want[0]).all() and (dists == want[1]).all()
    finally:
        ix.free()
