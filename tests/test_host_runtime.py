"""The host side of the library with a stand-in for the HIP runtime (not GPU)."""
import ctypes
import os
import subprocess
import sys
import threading
import time

import numpy as np
import pytest

import host_lib

pytestmark = pytest.mark.skipif(host_lib.hipcc() is None, reason="hipcc missing")


@pytest.fixture(scope="module")
def lib(tmp_path_factory):
    return host_lib.build(str(tmp_path_factory.mktemp("host")))


def _ptr(a):
    return a.ctypes.data_as(ctypes.c_void_p)


def sweep(lib, L, mask, samples, boundary=0):
    ns = np.zeros(samples, dtype=np.int32)
    return lib.nz_sweep(L, mask, boundary, samples, 1, _ptr(ns), None)


@pytest.mark.parametrize("boundary", [0, 1])
def test_lds_limit_is_the_same_for_every_launch_of_a_kernel(lib, boundary):
    """The limit belongs to the kernel, not to a launch: were it that of the launch at
    hand, a second thread with a smaller lattice could lower it between another's
    setting and its launch."""
    lib.fake_reset()
    limits = {}
    for L, samples in ((11, 300), (12, 300), (14, 2), (15, 2), (16, 2), (18, 2), (14, 2)):
        assert sweep(lib, L, 0x01, samples, boundary) == 0, lib.nz_last_error()
    for name, lds, limit in host_lib.launches(lib):
        assert lds <= limit, (name, lds, limit)
        if lds > 16384 and "nz_sweep_kernel" in name:
            limits.setdefault(name, set()).add(limit)
    assert len(limits) == 2 and all(len(v) == 1 for v in limits.values()), limits


def test_wrap_displacements_are_not_narrowed(tmp_path):
    """A displacement is the sum of up to two steps of every site on a path, so the
    one between a pair's nodes takes any value up to twice the largest lattice."""
    src = tmp_path / "width.hip"
    kernels = os.path.join(host_lib.CSRC, "nz_kernels.hip")
    src.write_text(f'#include "{kernels}"\n' + """
#include <limits>
#include <type_traits>
#include <utility>
template <int NT, int B>
constexpr long long widest()
{
    using C = nz::BlkCfg<nz::BLK_WRAP, true, NT, B>;
    using T = std::remove_reference_t<decltype(std::declval<nz::BlkLds<C> &>().eq[0])>;
    return std::numeric_limits<T>::max();
}
constexpr long long bound = 2LL * 55 * 55 * 55 * 55 * 55;
static_assert(widest<256, 256>() >= bound && widest<512, 512>() >= bound && widest<1024, 512>() >= bound, "too narrow");
""")
    run = subprocess.run([host_lib.hipcc(), "--cuda-host-only", "--offload-arch=gfx950", "-std=c++17", "-fsyntax-only", str(src)],
                         capture_output=True, text=True, timeout=300)
    assert run.returncode == 0, run.stderr[-2000:]


def test_canonical_reports_failed_allocations(lib):
    """Every host allocation of the call fails in turn: a status, never an exception
    through the C interface (which would end the process; hence one of its own)."""
    code = """
import ctypes, sys
lib = ctypes.CDLL(sys.argv[1])
every = (ctypes.c_uint64 * 65)(*range(65))
few = (ctypes.c_uint64 * 65)(*[n == 20 or n == 30 for n in range(65)])
p = (ctypes.c_double * 3)(0.1, 0.5, 0.9)
R = (ctypes.c_double * 3)()
lib.nz_canonical.argtypes = [ctypes.c_void_p, ctypes.c_int64, ctypes.c_void_p, ctypes.c_int64, ctypes.c_void_p]
lib.fake_fail_new.argtypes = [ctypes.c_int64]
for h in (every, few):
    failed = 0
    while True:
        lib.fake_fail_new(failed)
        rc = lib.nz_canonical(h, 65, p, 3, R)
        lib.fake_fail_new(-1)
        if rc == 0:
            break
        assert rc == -3, rc
        failed += 1
    assert failed >= 1
"""
    run = subprocess.run([sys.executable, "-c", code, lib._name], capture_output=True, text=True, timeout=60)
    assert run.returncode == 0, (run.returncode, run.stderr[-500:])


def test_canonical_of_a_dense_histogram_keeps_one_array(lib):
    """A histogram with counts in every entry costs one table of N + 1 values, not
    three (the steps' places, their counts and their values, grown as they are met),
    which was most of such a call."""
    N = 1 << 18
    h, p, R = np.ones(N + 1, dtype=np.uint64), np.array([0.3]), np.zeros(1)
    lib.fake_reset_peak()
    assert lib.nz_canonical(_ptr(h), N + 1, _ptr(p), 1, _ptr(R)) == 0
    assert 8 * N <= lib.fake_peak() <= 12 * N
    assert abs(R[0] - 0.3) < 1e-5   # F(n) = n / (N + 1)


GIB = 1 << 30


def all_given_back(lib):
    """(A thread that has been joined may be about to end.)"""
    end = time.monotonic() + 10
    while lib.fake_device_bytes() and time.monotonic() < end:
        time.sleep(0.01)
    return lib.fake_device_bytes() == 0


def in_thread(f):
    """f() on a thread of its own."""
    out = []
    t = threading.Thread(target=lambda: out.append(f()))
    t.start()
    t.join()
    return out[0]


def test_kept_device_memory_is_reused_grown_and_given_back(lib):
    def work():
        lib.fake_reset()
        assert sweep(lib, 8, 0x01, 100) == 0
        small = lib.fake_device_bytes()
        assert small > 0 and (lib.fake_mallocs(), lib.fake_frees()) == (1, 0)
        assert sweep(lib, 8, 0x01, 100) == 0 and sweep(lib, 5, 0x7F, 100) == 0
        assert (lib.fake_mallocs(), lib.fake_frees()) == (1, 0)
        assert sweep(lib, 12, 0x01, 100) == 0   # a larger one takes its place
        assert (lib.fake_mallocs(), lib.fake_frees()) == (2, 1) and lib.fake_device_bytes() > small
        sums = np.zeros(50, dtype=np.uint64)    # windows use the same block
        assert lib.nz_smax_window(8, 1, 0, 1, 0, 10, -1, 100, 150, _ptr(sums)) == 0
        assert lib.fake_mallocs() == 2
        assert lib.nz_release() == 0
        assert lib.fake_frees() == 2 and lib.fake_device_bytes() == 0
        assert lib.nz_release() == 0 and lib.fake_frees() == 2
        assert sweep(lib, 8, 0x01, 100) == 0
        return lib.fake_device_bytes()

    lib.nz_release()
    assert all_given_back(lib)
    assert in_thread(work) > 0
    assert all_given_back(lib)   # the end of the thread gives back what it kept


def test_kept_device_memory_is_bounded(lib):
    """Over all threads no more than 8 GiB stay, and none of a block above 4 GiB."""
    lib.nz_release()
    assert all_given_back(lib)
    barrier = threading.Barrier(4)
    codes, kept = [], []

    def work():
        codes.append(sweep(lib, 16, 0x01, 400))   # some 3 GiB
        barrier.wait()
        kept.append(lib.fake_device_bytes())
        barrier.wait()

    ts = [threading.Thread(target=work) for _ in range(4)]
    for t in ts:
        t.start()
    for t in ts:
        t.join()
    assert codes == [0] * 4
    assert all(2 * GIB < k <= 8 * GIB for k in kept), kept
    assert all_given_back(lib)
    assert in_thread(lambda: (sweep(lib, 30, 0x01, 40), lib.fake_device_bytes())) == (0, 0)


def test_a_failed_allocation_is_tried_with_less(lib):
    def work():
        lib.fake_fail_mallocs(1)
        first = sweep(lib, 8, 0x01, 100)
        lib.fake_fail_mallocs(2)
        second = sweep(lib, 12, 0x01, 100)
        lib.fake_fail_mallocs(0)
        return first, second, sweep(lib, 12, 0x01, 100)

    assert in_thread(work) == (0, -3, 0)   # NZ_ENOMEM


@pytest.mark.parametrize("failing", [0, 1])
def test_one_group_of_a_batch_fails_and_the_other_ends(lib, failing):
    """Two groups side by side: the second one's keys wait for the first one's, which
    never come if its first copy fails.  The call ends with that failure all the
    same, and a later one runs."""
    from paper_2607_18991_amd import nz

    arr, n = nz.make_jobs([dict(L=6, zone_mask=m, seed=1, nsamples=300) for m in (0x01, 0x7F)])
    need = ctypes.c_size_t()
    assert lib.nz_batch_workspace_bytes(arr, n, None, ctypes.byref(need)) == 0
    space = np.zeros(need.value + 256, dtype=np.uint8)
    ws = ctypes.c_void_p((space.ctypes.data + 255) // 256 * 256)
    out = np.zeros(600, dtype=np.int32)
    stream = ctypes.c_void_p(0x77)

    def call():
        return lib.nz_sweep_batch(arr, n, ws, need.value, _ptr(out), None, None, None, stream), lib.nz_last_error()

    def work():
        first = call()
        lib.fake_reset()
        assert call()[0] == 0
        streams = {k for k in lib_streams(lib)}
        assert len(streams) == 2 and 0x77 in streams   # the two groups
        lib.fake_fail_copies(ctypes.c_void_p(0x77 if failing == 0 else (streams - {0x77}).pop()))
        second = call()
        lib.fake_reset()
        return first, second, call()

    done = []
    t = threading.Thread(target=lambda: done.append(work()), daemon=True)
    t.start()
    t.join(30)
    assert done, "the call hangs"
    first, second, third = done[0]
    assert first[0] == 0 and third[0] == 0
    assert second[0] == nz.NZ_EDEVICE and b"hipMemcpyAsync" in second[1]


def lib_streams(lib):
    lib.fake_launch_stream.restype = ctypes.c_void_p
    return [lib.fake_launch_stream(k) or 0 for k in range(lib.fake_launches())]


def aligned(nbytes):
    """(address, owner) of nbytes of memory on a 256-byte boundary."""
    space = np.zeros(nbytes + 256, dtype=np.uint8)
    return ctypes.c_void_p((space.ctypes.data + 255) // 256 * 256), space


@pytest.mark.parametrize("L,mask,samples,smallest", [(1, 0x01, 20000, 3410176), (2, 0x28, 20000, 3413504)])
def test_workspaces_of_many_small_samples(lib, L, mask, samples, smallest):
    """A chunk of 16384 samples needs a header for them beside its smallest sample: a
    workspace sized for that with descriptors of 176 bytes stays large enough."""
    from paper_2607_18991_amd import nz

    arr, n = nz.make_jobs([dict(L=L, zone_mask=mask, seed=1, nsamples=samples)])
    ws, space = aligned(smallest)
    out = np.zeros(samples, dtype=np.int32)
    assert lib.nz_sweep_batch(arr, n, ws, smallest, _ptr(out), None, None, None, None) == 0, lib.nz_last_error()
    assert lib.nz_sweep_batch(arr, n, ws, smallest - 65536, _ptr(out), None, None, None, None) == nz.NZ_EWORKSPACE
    del space


@pytest.mark.parametrize("mask", [0x06, 0x07, 0x0C])
def test_the_static_buffer_holds_one_sample_of_L36(lib, mask):
    """A prefilled sample of 60 million sites fits the 256 MiB with 4-byte records; with
    8-byte ones it is swept plainly."""
    from paper_2607_18991_amd import nz

    N, p = 36**5, 1.553 / (nz.nz_coordination(mask) + 1.01)
    arr, n = nz.make_jobs([dict(L=36, zone_mask=mask, seed=1, nsamples=1, n0=int(0.97 * p * N), backoff=int(0.03 * p * N),
                                band_hi=int(1.05 * p * N) + 1024)])
    out = np.zeros(1, dtype=np.int32)
    lib.nz_sweep_batch_static.argtypes = [ctypes.c_void_p, ctypes.c_int32] + [ctypes.c_void_p] * 5
    assert lib.nz_sweep_batch_static(arr, n, _ptr(out), None, None, None, None) == 0, lib.nz_last_error()
    arr[0].L = 37
    assert lib.nz_sweep_batch_static(arr, n, _ptr(out), None, None, None, None) == nz.NZ_EWORKSPACE


def test_the_keys_phase_holds_no_wait_for_the_other_group(lib):
    """The second group's keys wait for the first one's: that time is in the whole call,
    not in the milliseconds of the keys."""
    from paper_2607_18991_amd import nz

    arr, n = nz.make_jobs([dict(L=6, zone_mask=m, seed=1, nsamples=300) for m in (0x01, 0x7F)])
    need = ctypes.c_size_t()
    assert lib.nz_batch_workspace_bytes(arr, n, None, ctypes.byref(need)) == 0
    ws, space = aligned(need.value)
    out = np.zeros(600, dtype=np.int32)
    ms = (ctypes.c_double * 6)()
    lib.nz_set_timing(1)
    try:
        assert lib.nz_sweep_batch(arr, n, ws, need.value, _ptr(out), None, None, None, ctypes.c_void_p(0x77)) == 0
        assert lib.nz_last_batch_timing(ms) == 0
    finally:
        lib.nz_set_timing(0)
    keys, labelling, sort, sweep, _, launches = list(ms)
    assert launches == 2
    # per group: clearing and one keys launch, nothing to label, one sweep
    assert (keys, labelling, sort, sweep) == (4.0, 0.0, 0.0, 2.0)
    del space
