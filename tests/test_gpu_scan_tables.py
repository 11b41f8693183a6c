"""The list-major scan's picks of one out of four, and its units in slices, against plain look-ups of the same table bytes."""
import numpy as np
import pytest
import torch

from paper_2601_07183_amd import datagen
from paper_2601_07183_amd import index_build as ib

pytestmark = pytest.mark.gpu


# numbers of sub-quantizers around whole dwords of codes; tables whose entries lie further apart than a signed
# byte holds (0 and 255 only: the entry that the groups not meant pick cannot be made zero) next to tables
# where that never happens; ragged tiles of 70 queries.  Integer scores: equal
@pytest.mark.parametrize("M", [2, 14, 16, 18, 24, 32, 34, 46, 48, 50, 62, 64, 66, 100, 128, 224, 226, 240, 242, 256])
def test_any_table_bytes(M):
    rng = np.random.default_rng(M)
    x = datagen.random_vectors(70 + M, 3000, M)
    hx = ib.build_index(x, 8, M, seed=3, coarse_iters=3, pq_iters=2)
    nq, nprobe, refine_k = 70, 5, 64
    probes = np.stack([rng.permutation(8)[:nprobe] for _ in range(nq)]).astype(np.int32)
    lut = rng.integers(0, 256, (nq, M, 16), dtype=np.uint8)
    lut[::3] = rng.choice(np.array([0, 255], np.uint8), lut[::3].shape)
    lut[1::3] = lut[1::3] // 3 + 90
    _check(hx, lut, probes, refine_k)


# units of several runs (vectors spread over the 66 pairs of 12 lists, six blocks a pair) cut into up to four slices by few
# queries with up to 6, and 8, probes; slices begin and end inside of runs, at their ends and behind the unit's last block
@pytest.mark.parametrize("M,n", [(16, 12_000), (48, 12_000), (50, 12_000), (64, 12_000), (64, 700)])
@pytest.mark.parametrize("nq,nprobe", [(1, 1), (7, 3), (40, 4), (40, 6), (50, 8)])
def test_slices_of_units(M, n, nq, nprobe):
    rng = np.random.default_rng(M + nq)
    asg = np.sort(np.stack([rng.permutation(12)[:2] for _ in range(n)]), axis=1).astype(np.int32)
    hx = ib.add_vectors(datagen.random_vectors(71, n, M), datagen.random_vectors(72, 12, M),
                        ib.train_pq(datagen.random_vectors(73, 300, M), M, 2, 2), assign=asg)
    probes = np.stack([rng.permutation(12)[:nprobe] for _ in range(nq)]).astype(np.int32)
    _check(hx, rng.integers(0, 256, (nq, M, 16), dtype=np.uint8), probes, 64)


def _check(hx, lut, probes, refine_k):
    from paper_2601_07183_amd import binding
    nq, M, _ = lut.shape
    codes = np.empty((len(hx.raw), M), np.int64)
    codes[:, 0::2], codes[:, 1::2] = hx.vec_codes & 15, hx.vec_codes >> 4
    ix = binding.Index(hx)
    try:
        ix.set_scan_mode(False, list_major=True)
        print("case:", M, nq, flush=True)
        cand, score, dco = (t.cpu().numpy() for t in ix.scan(torch.from_numpy(lut).cuda(), torch.from_numpy(probes).cuda(), refine_k))
        assert ix.scan_kernel_name() in ("scan_mfma_kernel", "scan_mfma_lds_kernel")
    finally:
        ix.free()
    for q in range(nq):
        member = np.flatnonzero(np.isin(hx.assign, probes[q]).any(axis=1))
        sums = lut[q][np.arange(M), codes[member]].astype(np.int64).sum(axis=1)
        order = np.lexsort((member, sums))[:refine_k]
        assert (cand[q][:len(order)] == member[order]).all() and (cand[q][len(order):] == -1).all()
        assert (score[q][:len(order)] == sums[order]).all()
