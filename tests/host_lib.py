"""The library's host code on a machine without a GPU: its sources compiled for the
host alone and linked with tests/host_runtime.cpp in place of the HIP runtime."""
import ctypes
import os
import shutil
import subprocess

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(HERE, "..", "paper_2607_18991_amd", "csrc")
SOURCES = ("nz_kernels.hip", "nz_mlp.hip", "nz_static.hip", "nz_api.cpp")


def hipcc():
    path = os.path.join(os.environ.get("ROCM_PATH", "/opt/rocm"), "bin", "hipcc")
    return shutil.which("hipcc") or (path if os.path.exists(path) else None)


def build(folder):
    """Compiles and links the host library in `folder` and loads it."""
    objs = []
    for src in [os.path.join(CSRC, s) for s in SOURCES] + [os.path.join(HERE, "host_runtime.cpp")]:
        obj = os.path.join(folder, os.path.basename(src) + ".o")
        subprocess.run([hipcc(), "--cuda-host-only", "--offload-arch=gfx950", "-Xclang", "-target-feature", "-Xclang",
                        "-packed-fp32-ops", "-O2", "-std=c++17", "-fPIC", "-fvisibility=hidden", "-c", src, "-o", obj],
                       check=True, capture_output=True, timeout=300)
        objs.append(obj)
    # the device code that a host object refers to is not there: any address will do
    undefined = subprocess.run(["nm", "-u", *objs], check=True, capture_output=True, text=True).stdout.split()
    images = sorted({n for n in undefined if n.startswith("__hip_fatbin")})
    out = os.path.join(folder, "libnzhost.so")
    subprocess.run(["g++", "-shared", "-o", out, *objs, "-Wl,-Bsymbolic", "-lpthread",
                    *[f"-Wl,--defsym={n}=0" for n in images]], check=True, capture_output=True, timeout=120)
    lib = ctypes.CDLL(out)
    lib.nz_last_error.restype = ctypes.c_char_p
    for name in ("fake_mallocs", "fake_frees", "fake_device_bytes", "fake_peak"):
        getattr(lib, name).restype = ctypes.c_int64
    lib.fake_launch.restype = ctypes.c_char_p
    lib.fake_fail_copies.argtypes = [ctypes.c_void_p]
    lib.fake_fail_new.argtypes = [ctypes.c_int64]
    i32, u32, i64, u64, P = ctypes.c_int32, ctypes.c_uint32, ctypes.c_int64, ctypes.c_uint64, ctypes.c_void_p
    lib.nz_sweep.argtypes = [i32, u32, i32, i64, u64, P, P]
    lib.nz_sweep_batch.argtypes = [P, i32, P, ctypes.c_size_t, P, P, P, P, P]
    lib.nz_batch_workspace_bytes.argtypes = [P, i32, P, ctypes.POINTER(ctypes.c_size_t)]
    lib.nz_canonical.argtypes = [P, i64, P, i64, P]
    lib.nz_smax_window.argtypes = [i32, u32, i32, u64, i64, i64, i64, i64, i64, P]
    return lib


def launches(lib):
    """(kernel, dynamic LDS, limit of its function) of every launch since fake_reset."""
    out = []
    for k in range(lib.fake_launches()):
        lds, limit = ctypes.c_size_t(), ctypes.c_size_t()
        name = lib.fake_launch(k, ctypes.byref(lds), ctypes.byref(limit)).decode()
        out.append((name, lds.value, limit.value))
    return out
