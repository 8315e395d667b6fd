"""Sparse prefill lists, whose labelling holds the occupation map in LDS (GPU),
against the oracle: lattices whose map is exact and those with 2, 4 and 8 sites
to a bit, lists shorter than a wave, of part of a workgroup and of several
passes, free, and periodic in largest-cluster windows.  A list that misses a link or makes a wrong one gives
another n* or mass.  Integers: the bar is equality."""
import numpy as np
import pytest

from gpu_util import assert_same, oracle_batch, run_batch

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("L,masks,count", [
    (9, (0x78, 0x7F), 20),
    (12, (0x0F, 0x40, 0x7F), 12),
    (16, (0x1C, 0x7F), 3),
    (17, (0x0F, 0x7F), 2),
    (20, (0x7F,), 2),
    (24, (0x7F,), 2),
])
def test_sparse_lists_match_oracle(L, masks, count):
    jobs = [dict(L=L, zone_mask=m, seed=0x5AB5 + L, nsamples=count) for m in masks]
    want = oracle_batch(jobs)
    for share in (0.05, 0.6, 0.9):   # of the smallest n*
        pre = []
        for k, j in enumerate(jobs):
            n0 = max(1, int(share * np.min(want[0][k * count:(k + 1) * count])))
            pre.append(dict(j, n0=n0, backoff=max(1, n0 // 4)))
        gn, gm, _, _ = run_batch(pre)
        assert_same(pre, gn, gm, *want)


@pytest.mark.parametrize("L,mask,lo,hi,n0", [(9, 0x7F, 300, 900, 250), (12, 0x7F, 900, 1500, 800), (17, 0x7F, 4000, 4300, 3800)])
def test_sparse_periodic_windows_match_oracle(L, mask, lo, hi, n0):
    import oracle
    from paper_2607_18991_amd import nz

    got = nz.nz_smax_window(L, mask, 0x5A5 + L, 0, 3, lo, hi, n0=n0, boundary=1)
    want = oracle.smax_window(L, mask, 0x5A5 + L, 0, 3, lo, hi, periodic=True)
    assert (got.astype(np.int64) == want).all()
