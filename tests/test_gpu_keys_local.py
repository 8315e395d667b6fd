"""Wide bands of many samples, whose keys run one workgroup per sample (GPU):
lattices of one wave, of a whole number of a wave's 8192 sites (L = 8), of a
remainder (L = 9), of exactly fewer waves than a workgroup holds (L = 10) and of
more than one pass (L = 12), plain and prefilled, free and periodic, against the
oracle and against the same samples in batches too small for that kernel.
Integers: the bar is equality."""
import numpy as np
import pytest

from gpu_util import assert_same, oracle_batch, run_batch

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("L,mask,count,few,periodic", [
    (3, 0x01, 1100, 300, False),
    (5, 0x03, 1024, 300, True),
    (8, 0x01, 256, 60, False),
    (8, 0x03, 300, 60, True),
    (9, 0x01, 130, 30, False),
    (10, 0x02, 90, 20, False),
    (12, 0x01, 64, 20, False),
    (12, 0x01, 70, 20, True),
])
def test_many_wide_bands_match_oracle(L, mask, count, few, periodic):
    job = dict(L=L, zone_mask=mask, seed=0x10CA1 + L, nsamples=count, boundary=1 if periodic else 0)
    want = oracle_batch([job])
    gn, gm, _, _ = run_batch([job])
    assert_same([job], gn, gm, *want)
    # prefilled below every sample's n*, up to the largest one
    lo, hi = int(np.min(want[0])), int(np.max(want[0]))
    pre = dict(job, n0=max(1, lo // 2), backoff=max(1, lo // 8), band_hi=min(L**5, hi + 8))
    gn, gm, _, _ = run_batch([pre])
    assert_same([pre], gn, gm, *want)
    gn, gm, _, _ = run_batch([dict(pre, sample0=count - few, nsamples=few)])
    assert_same([dict(pre, nsamples=few)], gn, gm, want[0][-few:], want[1][-few:])
