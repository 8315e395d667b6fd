"""nz_canonical on both sides of the line between its two forms (steps, values at
every n), against the oracle's long-double convolution (not GPU).  The bar is that
of the other comparisons: FP64 sums of at most N terms of weight sum one."""
import numpy as np
import pytest

from paper_2607_18991_amd import nz


def _held(N, share, where, seed):
    """A histogram with counts in `share` of its entries: anywhere, in the upper half,
    or nowhere in the blocks of 64 at multiples of N / 64."""
    rng = np.random.default_rng(seed)
    h = ((rng.random(N + 1) < share) * rng.integers(1, 50, N + 1)).astype(np.uint64)
    n = np.arange(N + 1)
    if where == "upper":
        h[: N // 2] = 0
    elif where == "between":
        h[(n % max(1, N // 64)) < 64] = 0
    h[N // 3] += 1
    return h


@pytest.mark.parametrize("N", [1, 63, 64, 1000, 4095, 4096, 20000, 65537])
@pytest.mark.parametrize("share,where", [(0.01, "any"), (0.12, "any"), (0.13, "any"), (1.0, "any"), (1.0, "upper"),
                                         (1.0, "between")])
def test_both_forms_match_the_oracle(nzo, N, share, where):
    h = _held(N, share, where, N)
    p = np.array([0.0, 1e-9, 0.07, 1 / 3, 0.5, 0.77, 1 - 1e-9, 1.0])
    assert np.max(np.abs(nz.nz_canonical(h, p) - nzo.canonical(h, p))) <= 1e-12


@pytest.mark.parametrize("share", [0.05, 1.0])
def test_counts_beyond_exact_sums(nzo, share):
    h = _held(3000, share, "any", 5) << np.uint64(46)
    p = np.linspace(0, 1, 11)
    assert np.max(np.abs(nz.nz_canonical(h, p) - nzo.canonical(h, p))) <= 1e-12


def test_only_samples_that_never_span():
    h = np.zeros(100, dtype=np.uint64)
    h[0] = 7
    assert (nz.nz_canonical(h, np.linspace(0, 1, 5)) == 0).all()


def _window(N, W, seed):
    rng = np.random.default_rng(seed)
    lo = int(0.14 * N) - W // 2
    return np.abs(rng.standard_normal(W)) * N, lo


@pytest.mark.parametrize("W,points", [(3000, 40), (30000, 3), (30000, 400)])
def test_windows_on_both_sides_of_the_look_match_the_oracle(nzo, W, points):
    """Windows narrower than the walks are looked through for their largest value, so
    that walks can end early; wider ones are not."""
    N = 10**5
    Q, lo = _window(N, W, 3) if W < 20000 else (np.abs(np.random.default_rng(4).standard_normal(W)) * N, 0)
    p = np.linspace(0.12, 0.16, points)
    a, ca = nz.nz_convolve_window(Q, lo, N, p)
    b, cb = nzo.convolve_window(Q, lo, N, p)
    assert np.allclose(a, b, rtol=1e-12, atol=1e-12 * N) and np.allclose(ca, cb, atol=1e-12)


def test_wide_window_costs_no_look_through_it():
    """One p on a window of two million entries walks some 73000 of them: as long as
    on a window of 80000 that holds them all, not thirty times as long."""
    import time

    N, p = 24**5, [0.14]

    def best(W):
        Q, lo = _window(N, W, 6)
        times = []
        for _ in range(9):
            t = time.perf_counter()
            nz.nz_convolve_window(Q, lo, N, p)
            times.append(time.perf_counter() - t)
        return min(times)

    wide, narrow = best(2_000_000), best(80_000)
    assert wide < 8 * narrow, (wide, narrow)
