"""Forms of the block sweep that no other test forces (GPU), against the oracle:
blocks cut to single sites in the wrapping and the largest-cluster sweep (test
hook: a block of several sites may touch no earlier root, or three), one-site
blocks against whole ones where the oracle is too slow, and the large workgroup on
lattices whose map bits stand for 32 sites and more (L = 28, 33).  Integers: the
bar is equality."""
import numpy as np
import pytest

from gpu_util import assert_same, oracle_batch, run_batch

pytestmark = pytest.mark.gpu

COMPACT = [0x01, 0x03, 0x07, 0x0F, 0x1F, 0x3F, 0x7F]


@pytest.mark.parametrize("cap", [0, 3])
@pytest.mark.parametrize("L,masks,count", [(5, (0x01, 0x7F), 16), (8, (0x01, 0x0C), 10), (11, (0x03, 0x7F), 4)])
def test_wrapping_blocks_cut_to_sites(monkeypatch, cap, L, masks, count):
    jobs = [dict(L=L, zone_mask=m, seed=0xB1 + L, nsamples=count, boundary=1) for m in masks]
    want = oracle_batch(jobs)
    n0 = [max(1, int(np.min(want[0][k * count:(k + 1) * count])) // 2) for k in range(len(masks))]
    jobs += [dict(j, n0=n, backoff=max(1, n // 4)) for j, n in zip(jobs, n0)]
    monkeypatch.setenv("NZ_DEBUG_BLOCK_OLD", str(cap))
    gn, gm, _, _ = run_batch(jobs)
    assert_same(jobs, gn, gm, np.tile(want[0], 2), np.tile(want[1], 2))


@pytest.mark.parametrize("cap", [0, 3])
@pytest.mark.parametrize("L,mask,lo,hi,n0,boundary", [
    (5, 0x01, 1, 1500, -1, 0), (5, 0x7F, 1, 300, -1, 1), (8, 0x01, 4000, 5200, 3800, 1), (10, 0x0C, 300, 900, 250, 0),
])
def test_window_blocks_cut_to_sites(monkeypatch, cap, L, mask, lo, hi, n0, boundary):
    import oracle
    from paper_2607_18991_amd import nz

    monkeypatch.setenv("NZ_DEBUG_BLOCK_OLD", str(cap))
    got = nz.nz_smax_window(L, mask, 0xB2 + L, 0, 6, lo, hi, n0=n0, boundary=boundary)
    want = oracle.smax_window(L, mask, 0xB2 + L, 0, 6, lo, hi, periodic=boundary == 1)
    assert (got.astype(np.int64) == want).all()


@pytest.mark.parametrize("L", [9, 12])
def test_blocks_of_one_site_equal_whole_ones(monkeypatch, L):
    from paper_2607_18991_amd import learned

    jobs = learned.PrefillModel.load().plan([dict(L=L, zone_mask=m, seed=1300 + L, nsamples=24) for m in COMPACT])
    whole = run_batch(jobs)
    monkeypatch.setenv("NZ_DEBUG_BLOCK_OLD", "0")
    single = run_batch(jobs)
    assert (whole[0] == single[0]).all() and (whole[1] == single[1]).all() and (whole[2] == single[2]).all()
    assert (whole[0] > 0).all()


@pytest.mark.parametrize("L,mask,boundary", [(28, 0x7F, 0), (28, 0x40, 1), (33, 0x7F, 0)])
def test_maps_of_32_sites_to_a_bit(L, mask, boundary):
    """Plain and prefilled (the list is shorter than the bitset has words, and the map
    is made from it)."""
    job = dict(L=L, zone_mask=mask, seed=0x32B + L, nsamples=2, boundary=boundary)
    want = oracle_batch([job])
    gn, gm, _, _ = run_batch([job])
    assert_same([job], gn, gm, *want)
    n0 = int(0.8 * np.min(want[0]))
    pre = dict(job, n0=n0, backoff=n0 // 4)
    gn, gm, _, _ = run_batch([pre])
    assert_same([pre], gn, gm, *want)


def test_map_from_the_bitset_at_32_sites_to_a_bit():
    """Zone 1 from a prefill of 13% of the sites: the list is longer than the bitset
    has words."""
    job = dict(L=28, zone_mask=0x01, seed=0x32C, nsamples=1, n0=int(0.13 * 28**5), backoff=28**5 // 50)
    assert job["n0"] > 28**5 // 32
    gn, gm, _, _ = run_batch([job])
    assert_same([job], gn, gm, *oracle_batch([job]))
