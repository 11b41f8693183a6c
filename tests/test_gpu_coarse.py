"""The coarse quantizer's shortlist route at the edges of its tiles and of its ways to a threshold, and the
assignment where its fp32 filter hands over to the definition."""
import numpy as np
import pytest
import torch

from oracle import oracle
from paper_2601_07183_amd import datagen
from paper_2601_07183_amd import index_build as ib

pytestmark = pytest.mark.gpu


# nlist: partial tiles, rows of 4-byte and 16-byte alignment, 64 / 256 / 1,024 half tiles and one tile
# more; d: partial steps of 16, one chunk of 128, partial and whole further ones; nprobe: around
# 3/4 of the half tiles and beyond the 256 entries that a wave narrows without a sort; batches of partial tiles
@pytest.mark.parametrize("nlist,d,nprobes,metric", [
    (64, 8, (1, 3, 4, 64), "l2"), (97, 24, (1, 5, 6, 97), "l2"), (1023, 128, (1, 10, 47, 48, 49, 130), "l2"),
    (1024, 96, (10, 48, 64, 300), "ip"), (1026, 136, (23, 49, 50), "l2"), (4096, 32, (39, 191, 192, 200, 201), "l2"),
    (4130, 64, (200, 201, 260), "ip"), (1000, 960, (45, 47), "l2"), (512, 256, (24, 25), "l2"), (8192, 16, (150, 192, 200), "l2"), (16384, 16, (98, 200), "l2"),
    (16416, 16, (98,), "l2"),
    (500, 100, (12, 40), "l2"), (300, 4, (7, 30), "ip"), (260, 140, (9, 30), "l2"), (130, 18, (9,), "l2")])
def test_probe_lists(nlist, d, nprobes, metric):
    from paper_2601_07183_amd import binding
    g = np.random.Generator(np.random.PCG64(nlist + d))
    cents = (g.standard_normal((nlist, d)) + 2.0 * g.standard_normal((20, d))[g.integers(0, 20, nlist)]).astype(np.float32)
    cents[1:nlist:7] = cents[0:nlist - 1:7]                        # equal centroids: ties go to the smaller id
    x = cents[:40] + np.float32(0.1) * g.standard_normal((40, d)).astype(np.float32)
    asg = np.sort(g.integers(0, nlist, size=(40, 2)), axis=1).astype(np.int32)
    M = next(m for m in (16, 12, 10, 8, 6, 4, 2) if d % m == 0)
    cb = ib.train_pq(datagen.random_vectors(5, 64, d), M, 5, 2)
    hx = ib.add_vectors(x.astype(np.float32), cents, cb, assign=asg, metric=metric)
    nq = 150
    q = (cents[g.integers(0, nlist, nq)] + 0.7 * g.standard_normal((nq, d))).astype(np.float32)
    q[7] = 0.0
    ox = oracle.OracleIndex(hx)
    ix = binding.Index(hx)
    try:
        dq = torch.from_numpy(q).cuda()
        for nprobe in nprobes:
            print("case:", nlist, d, metric, nprobe, flush=True)
            pid, pd = ix.coarse(dq, nprobe)
            torch.cuda.synchronize()
            pid, pd = pid.cpu().numpy(), pd.cpu().numpy()
            for i in range(nq):
                want, wd = oracle.coarse(ox, q[i], nprobe)
                assert (pid[i] == want).all(), i
                assert (pd[i] == wd).all(), i                      # the defined order of summation on both sides
    finally:
        ix.free()


def test_values_out_of_range():
    # components near the ends of the fp32 range, infinities and NaN in one query of the batch: the
    # other queries are not touched, and the large but finite ones still get the defined lists
    from paper_2601_07183_amd import binding
    g = np.random.Generator(np.random.PCG64(9))
    cents = g.standard_normal((256, 64)).astype(np.float32)
    asg = np.sort(g.integers(0, 256, size=(40, 2)), axis=1).astype(np.int32)
    cb = ib.train_pq(datagen.random_vectors(5, 64, 64), 16, 5, 2)
    hx = ib.add_vectors(cents[:40].copy(), cents, cb, assign=asg)
    q = g.standard_normal((40, 64)).astype(np.float32)
    q[3] *= np.float32(1e-20)
    q[4] *= np.float32(1e15)
    q[5, 2] = np.inf
    q[6, 3] = np.nan
    ox = oracle.OracleIndex(hx)
    ix = binding.Index(hx)
    try:
        pid, pd = ix.coarse(torch.from_numpy(q).cuda(), 9)
        torch.cuda.synchronize()
        for i in range(len(q)):
            if i in (5, 6):
                continue
            want, wd = oracle.coarse(ox, q[i], 9)
            assert (pid[i].cpu().numpy() == want).all(), i
            assert (pd[i].cpu().numpy() == wd).all(), i
    finally:
        ix.free()


# rows that are no quads, equal centroids (exact ties of the loss), all candidate counts of the last
# group of four, a huge and a negative lambda, values that overflow in fp32 (and a tiny vector, whose
# residuals are the centroids')
@pytest.mark.parametrize("d", [6, 20, 64, 130])
def test_assign_ties_and_ranges(d):
    from paper_2601_07183_amd import binding
    g = np.random.Generator(np.random.PCG64(d))
    cents = np.round(3.0 * g.standard_normal((70, d))).astype(np.float32)
    cents[1::5] = cents[0:-1:5]
    asg = np.sort(g.integers(0, 70, size=(40, 2)), axis=1).astype(np.int32)
    cb = ib.train_pq(datagen.random_vectors(5, 64, d), 2, 5, 2)
    hx = ib.add_vectors(cents[:40].copy(), cents, cb, assign=asg)
    x = np.concatenate([np.round(2.0 * g.standard_normal((300, d))), g.standard_normal((200, d))]).astype(np.float32)
    x[7] *= np.float32(1e-22)
    x[8] *= np.float32(1e17)
    ix = binding.Index(hx)
    try:
        for nc in (1, 2, 4, 5, 10, 16, 17, 32):
            for lam, strict in ((0.5, True), (0.5, False), (1e30, True), (-1.0, True)):
                print("case: assign", d, nc, lam, strict, flush=True)
                got = ix.assign(torch.from_numpy(x).cuda(), nc, lam, strict)
                torch.cuda.synchronize()
                assert (got.cpu().numpy() == oracle.rair_assign(cents, x, nc, lam, strict)).all()
    finally:
        ix.free()


# centroids and vectors so small that products of residuals underflow in fp32, beside a lambda that
# brings their sum back into its range: the filter has to leave these to the definition
@pytest.mark.parametrize("nlist,d", [(40, 4), (40, 6), (70, 20), (70, 64)])
def test_assign_residuals_that_underflow(nlist, d):
    from paper_2601_07183_amd import binding
    g = np.random.Generator(np.random.PCG64(nlist + d))
    cb = ib.train_pq(datagen.random_vectors(5, 64, d), 2, 5, 2)
    asg = np.sort(g.integers(0, nlist, size=(40, 2)), axis=1).astype(np.int32)
    for scale in (1e-16, 1e-19, 1e-21, 3e-23):
        cents = (scale * g.standard_normal((nlist, d))).astype(np.float32)
        if scale < 1e-22:                                # the nearest three: only the third is the minimum
            cents[:] = np.float32(1e-21)
            cents[0], cents[1], cents[2] = 2e-23, 2.8e-23, 0.0
            cents[2, 0] = 4.2e-23
        x = (0.2 * scale * g.standard_normal((300, d))).astype(np.float32)
        x[0] = 0.0
        hx = ib.add_vectors(x[:40].copy(), cents, cb, assign=asg)
        ix = binding.Index(hx)
        try:
            for lam, nc in ((1e10, 3), (1e10, 10), (-1e12, 10), (1e20, 10), (1e33, 5), (0.5, 10)):
                print("case: assign", d, scale, lam, nc, flush=True)
                got = ix.assign(torch.from_numpy(x).cuda(), nc, lam, True)
                torch.cuda.synchronize()
                assert (got.cpu().numpy() == oracle.rair_assign(cents, x, nc, lam, True)).all()
        finally:
            ix.free()
