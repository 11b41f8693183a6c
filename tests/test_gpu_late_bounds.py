"""Batches whose units are nearly all in flight at once, so that bounds fall while most of the scan is under way."""
from dataclasses import replace

import pytest
import torch

from paper_2601_07183_amd import datagen
from paper_2601_07183_amd import index_build as ib

pytestmark = pytest.mark.gpu


def _index(n, d, M, nlist):
    from paper_2601_07183_amd import binding
    w = replace(datagen.WORKLOADS["sphere10m"], name="late", n=n, d=d, comps=200, nlist=nlist, M=M)
    base = datagen.make_base(w)
    cents = ib.kmeans(base, nlist, 4, 3, max_train=65_536)
    hx = ib.add_vectors(base, cents, ib.train_pq(base, M, 8, 7))
    return binding.Index(hx), torch.from_numpy(datagen.make_queries(w, 500)).cuda()


# bigK close to its limit: by what waves stage and log under bounds that are some blocks old, the log must not run out
# (it did, at every run, with bounds four blocks old: 22,100 entries a query for a log of some 21,400; now 17,100)
@pytest.mark.parametrize("n,d,M,nlist", [(200_000, 96, 48, 400)])
def test_log_holds_what_late_bounds_let_pass(n, d, M, nlist):
    ix, q = _index(n, d, M, nlist)
    try:
        ix.set_scan_mode(True)
        want = [t.cpu() for t in ix.search(q, 10, 64, 1000)]
        ix.set_scan_mode(False, list_major=True)
        print("case:", M, flush=True)
        got = [t.cpu() for t in ix.search(q, 10, 64, 1000)]
        assert torch.equal(got[0], want[0]) and torch.equal(got[1], want[1])
        st = ix.scan_stats()
        print("   ", st, flush=True)
        assert st["redone"] == 0
    finally:
        ix.free()
