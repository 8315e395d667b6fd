"""More samples than CUs on lattices whose occupation map fits a CU twice (GPU):
the smallest and the largest of them (L = 11, 13), free and periodic, plain and
prefilled, against the oracle.  Integers: the bar is equality."""
import numpy as np
import pytest

from gpu_util import assert_same, oracle_batch, run_batch

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("L,mask,count,periodic", [
    (11, 0x01, 300, False),
    (11, 0x7F, 257, False),
    (13, 0x03, 260, False),
    (11, 0x03, 300, True),
    (12, 0x01, 270, True),
])
def test_two_workgroups_per_cu_match_oracle(L, mask, count, periodic):
    job = dict(L=L, zone_mask=mask, seed=0x2C0 + L, nsamples=count, boundary=1 if periodic else 0)
    want = oracle_batch([job])
    gn, gm, _, _ = run_batch([job])
    assert_same([job], gn, gm, *want)
    n0 = int(np.min(want[0])) // 2
    pre = dict(job, n0=n0, backoff=max(1, n0 // 4))
    gn, gm, _, _ = run_batch([pre])
    assert_same([pre], gn, gm, *want)
