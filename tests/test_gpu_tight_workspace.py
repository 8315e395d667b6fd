"""Workspaces that hold a prefilled sample with 4-byte records per bitset word but
not with 8-byte ones (GPU): the sample is swept plainly, and its n* and mass are the
oracle's.  Integers: the bar is equality."""
import pytest

from gpu_util import assert_same, oracle_batch, run_batch

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("L,mask,n0", [(10, 0x7F, 120), (12, 0x1F, 1000)])
def test_smallest_accepted_workspace(L, mask, n0):
    from paper_2607_18991_amd import nz

    N = L**5
    jobs = [dict(L=L, zone_mask=mask, seed=0x716, nsamples=3, n0=n0, backoff=n0 // 3, band_hi=4 * n0 + 1024),
            dict(L=4, zone_mask=0x01, seed=0x717, nsamples=5)]
    want = oracle_batch(jobs)
    low, high = 256, nz.nz_batch_workspace_bytes(jobs)
    while high - low > 256:
        mid = (low + high) // 512 * 256
        try:
            run_batch(jobs, ws_bytes=mid)
            high = mid
        except nz.NzError as e:
            assert e.code == nz.NZ_EWORKSPACE
            low = mid
    gn, gm, _, stats = run_batch(jobs, ws_bytes=high, fill=0xFF)
    assert_same(jobs, gn, gm, *want)
    assert stats["prefilled_sites"] == 0 and stats["chunks"] >= 3
    # half of the records more, and the prefill is back
    gn, gm, _, stats = run_batch(jobs, ws_bytes=high + N // 8 + 512, fill=0xFF)
    assert_same(jobs, gn, gm, *want)
    assert stats["prefilled_sites"] > 0
