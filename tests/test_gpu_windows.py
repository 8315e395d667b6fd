"""Largest-cluster windows whose blocks are added at once, in halves and one by
one (GPU), against the oracle's running maximum: from the first site, where many
small clusters compete, through the threshold to where one cluster grows alone;
window ends at block edges; many short windows, whose sums are spread over
workgroups; prefilled sizes by ranges.  Integers: the bar is equality."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("L,mask,lo,hi,n0,boundary,samples", [
    (8, 0x01, 1, 6000, -1, 0, 3),
    (8, 0x01, 255, 258, -1, 1, 3),
    (9, 0x03, 1, 5000, -1, 1, 2),
    (10, 0x01, 9000, 18000, 8000, 0, 3),
    (10, 0x7F, 30, 1200, 20, 1, 3),
    (12, 0x01, 30000, 34000, 28000, 1, 3),
    (6, 0x01, 700, 1300, 600, 1, 70),
    (5, 0x01, 1, 3125, -1, 0, 40),
    # prefill lists of several ranges of 36864 sites, and of more than eight
    (13, 0x01, 52000, 52600, 50000, 1, 2),
    (19, 0x01, 346000, 346300, 340000, 0, 1),
])
def test_windows_match_oracle(L, mask, lo, hi, n0, boundary, samples):
    import oracle
    from paper_2607_18991_amd import nz

    got = nz.nz_smax_window(L, mask, 0x51A + L, 3, samples, lo, hi, n0=n0, boundary=boundary)
    want = oracle.smax_window(L, mask, 0x51A + L, 3, samples, lo, hi, periodic=boundary == 1)
    assert (got.astype(np.int64) == want).all()
