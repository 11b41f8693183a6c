"""The list-major scan's picks of one out of four against plain look-ups of the same table bytes."""
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
    from paper_2601_07183_amd import binding
    rng = np.random.default_rng(M)
    x = datagen.random_vectors(70 + M, 3000, M)
    hx = ib.build_index(x, 8, M, seed=3, coarse_iters=3, pq_iters=2)
    nq, nprobe, refine_k = 70, 5, 64
    probes = np.stack([rng.permutation(8)[:nprobe] for _ in range(nq)]).astype(np.int32)
    lut = rng.integers(0, 256, (nq, M, 16), dtype=np.uint8)
    lut[::3] = rng.choice(np.array([0, 255], np.uint8), lut[::3].shape)
    lut[1::3] = lut[1::3] // 3 + 90
    codes = np.empty((len(x), M), np.int64)
    codes[:, 0::2], codes[:, 1::2] = hx.vec_codes & 15, hx.vec_codes >> 4
    ix = binding.Index(hx)
    try:
        ix.set_scan_mode(False, list_major=True)
        print("case:", M, flush=True)
        cand, score, dco = (t.cpu().numpy() for t in ix.scan(torch.from_numpy(lut).cuda(), torch.from_numpy(probes).cuda(), refine_k))
        assert ix.scan_kernel_name() in ("scan_mfma_kernel", "scan_mfma_lds_kernel")
    finally:
        ix.free()
    for q in range(nq):
        member = np.flatnonzero(np.isin(hx.assign, probes[q]).any(axis=1))
        sums = lut[q][np.arange(M), codes[member]].astype(np.int64).sum(axis=1)
        order = np.lexsort((member, sums))[:refine_k]
        assert (cand[q] == member[order]).all()
        assert (score[q] == sums[order]).all()
