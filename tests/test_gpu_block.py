"""The block sweep at the sizes where its parts change (GPU), against the
oracle: lattices on both sides of the small-workgroup limit (L = 10, 11), the
largest one whose occupation map is exact (L = 16), those whose map bits stand
for two and four sites (L = 17, 21), neighbourhoods with one row, with rows of
one, two and five sites, and blocks that do not fit the pair list (a dense
small lattice).  Integers: the bar is equality."""
import numpy as np
import pytest

from gpu_util import assert_same, oracle_batch, run_batch

pytestmark = pytest.mark.gpu

PERIODIC = 1


@pytest.mark.parametrize("L,masks,count,periodic", [
    (10, (0x01, 0x08, 0x7F), 12, False),
    (11, (0x01, 0x40, 0x7F), 12, False),
    (13, (0x2B, 0x14), 8, False),
    (16, (0x01, 0x20), 3, False),
    (17, (0x01, 0x63), 2, False),
    (21, (0x03,), 1, False),
    (10, (0x08, 0x7F), 8, True),
    (11, (0x01, 0x64), 8, True),
    (17, (0x03, 0x48), 2, True),
])
def test_block_sweep_matches_oracle(L, masks, count, periodic):
    """Plain and prefilled (half of the plain n*) samples of the same orders."""
    jobs = [dict(L=L, zone_mask=m, seed=0xB10C + L, nsamples=count, boundary=PERIODIC if periodic else 0) for m in masks]
    want = oracle_batch(jobs)
    gn, gm, _, _ = run_batch(jobs)
    assert_same(jobs, gn, gm, *want)
    pre = []
    for k, j in enumerate(jobs):
        n0 = int(np.min(want[0][k * count:(k + 1) * count])) // 2
        pre.append(dict(j, n0=max(1, n0), backoff=max(1, n0 // 4)))
    gn, gm, _, _ = run_batch(pre)
    assert_same(pre, gn, gm, *want)


def test_dense_blocks_are_halved():
    """From a prefill below the threshold of a small wide lattice the first
    block's sites see hundreds of occupied neighbours each: the pair list
    overflows and the block is added in halves."""
    jobs = [dict(L=L, zone_mask=0x7F, seed=0xDE, nsamples=20, boundary=b, band_hi=L**5) for L in (5, 6) for b in (0, 1)]
    jobs += [dict(L=4, zone_mask=m, seed=0xDF, nsamples=20, band_hi=4**5) for m in (0x60, 0x40, 0x7F)]
    gn, gm, _, _ = run_batch(jobs)
    assert_same(jobs, gn, gm, *oracle_batch(jobs))


@pytest.mark.parametrize("L,mask,lo,hi,n0,boundary", [
    (4, 0x7F, 1, 1024, -1, 0),          # to the last site: every block overflows the pair list
    (5, 0x20, 1, 900, -1, 1),
    (11, 0x01, 20000, 21500, 18000, 1),
    (13, 0x03, 12000, 12900, 10000, 0),
])
def test_block_windows_match_oracle(L, mask, lo, hi, n0, boundary):
    import oracle
    from paper_2607_18991_amd import nz

    got = nz.nz_smax_window(L, mask, 0x5A + L, 0, 4, lo, hi, n0=n0, boundary=boundary)
    want = oracle.smax_window(L, mask, 0x5A + L, 0, 4, lo, hi, periodic=boundary == 1)
    assert (got.astype(np.int64) == want).all()


def test_threads_share_the_device():
    """Two host threads with their own workspaces and streams, at once."""
    import threading

    import torch

    jobs = [[dict(L=8, zone_mask=m, seed=0x7E + m, nsamples=64)] for m in (0x01, 0x7F)]
    out = [None, None]

    def work(k):
        with torch.cuda.stream(torch.cuda.Stream()):
            out[k] = run_batch(jobs[k])

    ts = [threading.Thread(target=work, args=(k,)) for k in range(2)]
    for t in ts:
        t.start()
    for t in ts:
        t.join()
    for k in range(2):
        assert_same(jobs[k], out[k][0], out[k][1], *oracle_batch(jobs[k]))
