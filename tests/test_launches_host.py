"""The built library against the host-only HIP stand-in (no GPU, no kernel runs): refusals before any launch, the status of
every launch, and how many launches a call takes."""
from __future__ import annotations

import json
import os
import shutil
import subprocess
import sys
import textwrap

import pytest

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)
HOSTDIR = os.path.join(HERE, "host")
CLANGXX = "/opt/rocm/llvm/bin/clang++"

# Runs in a process of its own, with the stand-in's symbols ahead of the HIP runtime's.
PRELUDE = """
import ctypes, json, sys
vp, i32, f64 = ctypes.c_void_p, ctypes.c_int32, ctypes.c_double
lib, shim = ctypes.CDLL(sys.argv[1]), ctypes.CDLL(sys.argv[2])
lib.wolf_fit_forward.argtypes = [vp, i32, f64, f64, f64, f64, i32, vp, vp, vp, vp]
lib.wolf_fit_backward.argtypes = [vp, vp, i32, f64, f64, f64, f64, i32, vp, vp, vp, vp, vp]
lib.wolf_fit_sums_work_bytes.restype = ctypes.c_int64
lib.wolf_degree_of_coherence.argtypes = [vp, i32, i32, i32, i32, f64, vp, vp]
lib.wolf_propagate_padded.argtypes = [vp, vp, i32, i32, f64, f64, f64, i32, i32, i32, vp, vp, vp]
lib.wolf_last_error_message.restype = ctypes.c_char_p
stub = ctypes.CDLL(sys.argv[3])
stub.hipMalloc.argtypes = [ctypes.POINTER(vp), ctypes.c_size_t]
def alloc(n):
    p = vp()
    assert stub.hipMalloc(ctypes.byref(p), n) == 0
    return p.value
def launches(f, fail_at=0):
    shim.shim_reset(fail_at)
    status = f()
    return status, shim.shim_launches()
out = {}
"""


@pytest.fixture(scope="module")
def run(tmp_path_factory):
    if not os.path.exists(CLANGXX):
        pytest.skip("ROCm compilers not installed")
    import paper_2203_02734_amd as wolf
    if not os.path.exists(wolf.LIB_PATH):
        from paper_2203_02734_amd import build
        build.build()
    d = tmp_path_factory.mktemp("stand_in")
    libs = {}
    for name in ("launch_shim", "hip_stub"):
        libs[name] = str(d / f"lib{name}.so")
        subprocess.run([CLANGXX, "-shared", "-fPIC", "-std=c++17", "-D__HIP_PLATFORM_AMD__", "-I/opt/rocm/include", "-I", HOSTDIR,
                        "-o", libs[name], os.path.join(HOSTDIR, name + ".cpp")], check=True)

    def go(body):
        code = PRELUDE + textwrap.dedent(body) + "\nprint(json.dumps(out))\n"
        env = dict(os.environ, LD_PRELOAD=":".join([libs["launch_shim"], libs["hip_stub"]]))
        r = subprocess.run([sys.executable, "-c", code, wolf.LIB_PATH, libs["launch_shim"], libs["hip_stub"]],
                           capture_output=True, text=True, env=env, timeout=120)
        assert r.returncode == 0, r.stderr[-2000:]
        return json.loads(r.stdout)

    return go


FIT = """
n, nn = 16, 256
size = {"imap": 4 * nn, "corr": 16 * (n // 2 + 1) * n, "work": lib.wolf_fit_sums_work_bytes(n), "s": 8 * nn, "g": 8 * nn,
        "d_imap": 4 * nn, "d_sigma": 8}
def forward(b):
    return lib.wolf_fit_forward(b["imap"], n, 1e-5, 1e-4, 6e-7, 0.3, 0, b["work"], b["corr"], b["s"], None)
def backward(b):
    return lib.wolf_fit_backward(b["g"], b["imap"], n, 1e-5, 1e-4, 6e-7, 0.3, 0, b["corr"], b["work"], b["d_imap"], b["d_sigma"],
                                 None)
calls = {"forward": (forward, ["imap", "work", "corr", "s"]),
         "backward": (backward, ["g", "imap", "corr", "work", "d_imap", "d_sigma"])}
"""


def test_fit_refuses_overlapping_buffers(run):
    """Each pair of buffers of a call, sharing their first or their last bytes, and side by side in one allocation."""
    out = run(FIT + textwrap.dedent("""
        for name, (call, used) in calls.items():
            free = {k: alloc(size[k]) for k in used}
            out[name + " apart"] = launches(lambda: call(free))
            for i, x in enumerate(used):
                for y in used[:i]:
                    for how in ("first", "last", "beside"):
                        a, b = max(size[x], size[y]), min(size[x], size[y])
                        base = alloc(a + b)
                        big, small = (x, y) if size[x] >= size[y] else (y, x)
                        bufs = dict(free)
                        bufs[big] = base
                        bufs[small] = base + {"first": 0, "last": a - b, "beside": a}[how]
                        out["%s %s %s %s" % (name, x, y, how)] = launches(lambda: call(bufs))
    """))
    for what, (status, count) in out.items():
        if what.endswith(("apart", "beside")):
            assert status == 0 and count in (3, 4), what
        else:
            assert status == -1 and count == 0, what


def test_every_failed_launch_is_reported(run):
    """The difference sums of the fit, and S alone of a propagated source."""
    out = run(FIT + textwrap.dedent("""
        lib.wolf_propagate_density.argtypes = [vp, i32, f64, f64, f64, i32, i32, i32, vp, vp]
        size["w"] = 8 * nn * nn
        calls["density"] = (lambda b: lib.wolf_propagate_density(b["w"], n, 1e-5, 6e-7, 0.3, 0, 0, 0, b["s"], None), ["w", "s"])
        for name, (call, used) in calls.items():
            bufs = {k: alloc(size[k]) for k in used}
            count = launches(lambda: call(bufs))[1]
            out[name] = [launches(lambda: call(bufs), k + 1) for k in range(count)]
    """))
    assert [len(out[k]) for k in ("forward", "backward", "density")] == [3, 4, 3]
    for name, seen in out.items():
        for k, (status, count) in enumerate(seen):
            assert status == -4 and count == k + 1, (name, k)  # and nothing is launched after the failure


def test_mu_slice_in_one_launch_up_to_32(run):
    """Above, one workgroup's gather of N^2 lines takes longer than three launches."""
    out = run("""
        w, mu = alloc(16 * 66 ** 4), alloc(16 * 66 ** 2)
        for dtype in (0, 1):
            for n in (2, 16, 30, 32, 34, 48, 64, 66):
                out["%d %d" % (dtype, n)] = launches(lambda: lib.wolf_degree_of_coherence(w, n, dtype, 1, 1, 1e-3, mu, None))
    """)
    for what, (status, count) in out.items():
        assert status == 0 and count == (1 if int(what.split()[1]) <= 32 else 3), what


def test_padded_needs_no_work_buffer(run):
    """Four passes in place on the output, for lengths with an FFT split and without; a buffer that is given is still checked."""
    out = run("""
        n = 12
        size = 16 * n ** 4
        w, o, k = alloc(size), alloc(size), alloc(size)
        def call(w_in, w_out, work, nz, dtype):
            return launches(lambda: lib.wolf_propagate_padded(w_in, w_out, n, nz, 1e-5, 6e-7, 0.3, 0, 0, dtype, work, None, None))
        for dtype in (0, 1):
            for nz in (12, 13, 24, 30):
                out["%d %d none" % (dtype, nz)] = call(w, o, None, nz, dtype)
                out["%d %d none in place" % (dtype, nz)] = call(w, w, None, nz, dtype)
                out["%d %d given" % (dtype, nz)] = call(w, o, k, nz, dtype)
                out["%d %d input: refused" % (dtype, nz)] = call(w, o, w, nz, dtype)
                out["%d %d output: refused" % (dtype, nz)] = call(w, o, o, nz, dtype)
                out["%d %d small: refused" % (dtype, nz)] = call(w, o, k + size - 64, nz, dtype)
    """)
    for what, (status, count) in out.items():
        assert (status, count) == ((-1, 0) if "refused" in what else (0, 4)), what
