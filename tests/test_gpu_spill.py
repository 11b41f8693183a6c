"""Survivors beyond a query's buffer: the spill behind the survivor log, up to its edges."""
import numpy as np
import pytest
import torch

from oracle import oracle
from paper_2601_07183_amd import datagen
from paper_2601_07183_amd import index_build as ib

pytestmark = pytest.mark.gpu


# a buffer holds 1,024 entries at bigK = 64, the workgroup-wide select takes up to 4,096; a query with
# more is redone exactly.  Clumps of identical vectors in one pair of lists, multiples of 32, so that
# all of them are in shared blocks and a query of the clump has exactly that many survivors.
@pytest.mark.parametrize("counts,redone", [((1024, 1056), 0), ((1056, 2048), 0), ((4096, 64), 0), ((4128, 1056), 7)])
def test_spilled_survivors(counts, redone):
    _check(counts, (7, 8), (redone, redone), 8, 4)


# whole batches over their buffers, the log's unused chunks dealt out in buckets: a few hundred entries
# from each of 300 queries (all fit), and 3,072 from each of 220, which overfill theirs and are redone
@pytest.mark.parametrize("counts,queries,redone", [((1504, 64), (300, 300), (0, 0)), ((4096, 64), (220, 380), (1, 220))])
def test_many_spilled_queries(counts, queries, redone):
    _check(counts, queries, redone, 32, 16)


def _check(counts, queries, redone, d, M):
    from paper_2601_07183_amd import binding
    va = datagen.random_vectors(60, 1, d)
    vb = va + np.float32(40)
    e = np.zeros((1, d), np.float32)
    e[0, 0] = 0.5
    x = np.concatenate([np.tile(va, (counts[0], 1)), np.tile(vb, (counts[1], 1))])
    cents = np.concatenate([va + e, va - e, vb + e, vb - e]).astype(np.float32)
    asg = np.array([[0, 1]] * counts[0] + [[2, 3]] * counts[1], dtype=np.int32)
    cb = ib.train_pq(datagen.random_vectors(61, 300, d), M, 5, 2)
    noise = datagen.random_vectors(62, sum(queries), d) * np.float32(0.01)
    q = (np.concatenate([np.tile(va, (queries[0], 1)), np.tile(vb, (queries[1], 1))]) + noise).astype(np.float32)
    hx = ib.add_vectors(x, cents, cb, assign=asg)
    want = oracle.search(oracle.OracleIndex(hx), q, 10, 2, 64)
    ix = binding.Index(hx)
    try:
        dq = torch.from_numpy(q).cuda()
        for _ in range(2):
            print("case:", counts, flush=True)
            ids, dists = ix.search(dq, 10, 2, 64)
            torch.cuda.synchronize()
            assert (ids.cpu().numpy() == want.ids).all()
            assert (dists.cpu().numpy() == want.dists).all()
            assert (ix.dco(len(q)) == want.dco).all()
            st = ix.scan_stats()
            print("   ", st, flush=True)
            assert redone[0] <= st["redone"] <= redone[1]
            assert st["max_survivors"] == max(counts) and st["logged"] == st["survivors"]
    finally:
        ix.free()


# A log that runs out of chunks, both scan kernels: every query is redone exactly, no entry is counted that was
# not written, and nothing is touched outside of the caller's workspace.  One vector 30,016 times in one pair of
# lists: 21 million entries of 700 queries for a log of at most 17.6 million.  What stands in the workspace
# beforehand are entries of the first query with a score that no bound lets pass (a table's sums stay below it), so an
# entry that was read but never written shows as one logged and not among the survivors.
@pytest.mark.parametrize("M", [4, 34, 48, 64, 240])
def test_log_runs_out_of_chunks(M):
    from paper_2601_07183_amd import binding
    n, nq, bigk, guard = 30_016, 700, 64, 1 << 20
    rng = np.random.default_rng(M)
    cents = datagen.random_vectors(63, 2, M)
    hx = ib.add_vectors(np.tile(datagen.random_vectors(64, 1, M), (n, 1)), cents,
                        ib.train_pq(datagen.random_vectors(65, 64, M), M, 3, 2), assign=np.tile(np.int32([[0, 1]]), (n, 1)))
    lut = rng.integers(0, 256, (nq, M, 16), dtype=np.uint8)
    code = np.empty(M, np.int64)
    code[0::2], code[1::2] = hx.vec_codes[0] & 15, hx.vec_codes[0] >> 4
    want = lut[:, np.arange(M), code].astype(np.int64).sum(axis=1)
    probes = np.tile(np.int32([0, 1]), (nq, 1))
    ix = binding.Index(hx)
    try:
        ix.set_scan_mode(False, list_major=True)
        size = ix.workspace_bytes(nq, 2, bigk) + 255 & ~255
        room = torch.full(((size + 2 * guard) // 4,), -65536, dtype=torch.int32, device="cuda")     # {slot, 0xFFFF << 16 | query 0}
        ix.set_workspace(room.view(torch.uint8)[guard:guard + size])
        print("case:", M, flush=True)
        cand, score, dco = (t.cpu().numpy() for t in ix.scan(torch.from_numpy(lut).cuda(), torch.from_numpy(probes).cuda(), bigk))
        assert (room[:guard // 4] == -65536).all() and (room[(guard + size) // 4:] == -65536).all()
        assert (cand == np.arange(bigk)).all() and (score == want[:, None]).all() and (dco == n).all()
        st = ix.scan_stats()
        print("   ", st, flush=True)
        assert st["redone"] == nq and st["logged"] < nq * n
        assert st["logged"] == st["survivors"]
    finally:
        ix.free()
