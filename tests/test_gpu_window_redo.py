"""Largest-cluster windows whose redo round mixes samples of unlike prefill lists
(GPU): n0 lies just below the window, so that about half of the samples reach it
and are redone from half of n0, beside samples of the full list whose band bucket
overflowed (test hook).  The lists differ by a factor of two, so one launch
labels both.  Integers: the bar is equality with the oracle."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("L,mask,lo,samples,boundary", [(9, 0x01, 10001, 64, 0), (8, 0x01, 3001, 96, 1)])
def test_redo_round_of_unlike_lists(monkeypatch, L, mask, lo, samples, boundary):
    import oracle
    from paper_2607_18991_amd import nz

    monkeypatch.setenv("NZ_DEBUG_BUCKET_CAP", "130")
    got = nz.nz_smax_window(L, mask, 0x3ED0 + L, 0, samples, lo, lo + 300, n0=lo - 1, boundary=boundary)
    stats = nz.nz_last_batch_stats()
    assert stats["backoffs"] > 0 and stats["bucket_redo"] > 0, stats
    want = oracle.smax_window(L, mask, 0x3ED0 + L, 0, samples, lo, lo + 300, periodic=boundary == 1)
    bad = np.nonzero(got.astype(np.int64) != want)[0]
    assert len(bad) == 0, (len(bad), bad[:5], got[bad[:5]], want[bad[:5]], stats)
