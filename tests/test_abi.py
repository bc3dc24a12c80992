"""The C-ABI library loads and exports every symbol the public header declares (no GPU needed)."""
import ctypes
import os
import re

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def declared_functions():
    text = open(os.path.join(ROOT, "include", "sparge.h")).read()
    text = re.sub(r"/\*.*?\*/", "", text, flags=re.S)
    return sorted(set(re.findall(r"\b(sparge_[a-z_]+)\s*\(", text)))


def test_header_declares_the_three_calls_of_the_boundary():
    names = declared_functions()
    for need in ("sparge_quantize", "sparge_predict", "sparge_attn", "sparge_forward", "sparge_workspace_bytes",
                 "sparge_last_error"):
        assert need in names


def test_library_exports_every_declared_symbol():
    import paper_2502_18137_amd as sp
    if not os.path.exists(sp.library_path()):
        from paper_2502_18137_amd.build import build_library
        build_library(verbose=False)
    lib = ctypes.CDLL(sp.library_path())
    for name in declared_functions():
        assert hasattr(lib, name), name
    assert sp.sparge_version() >= 100


def test_argument_validation_needs_no_gpu():
    import paper_2502_18137_amd as sp
    from paper_2502_18137_amd.binding import _Desc
    lib = sp.load_library()
    n = ctypes.c_size_t(0)
    good = _Desc(1, 2, 2048, 64, 0, 2 * 2048 * 64, 2048 * 64, 64)
    assert lib.sparge_workspace_bytes(ctypes.byref(good), sp.WS_FORWARD, ctypes.byref(n)) == 0
    assert n.value > 2 * 2048 * 64 * 2           # holds at least Q-hat and K-hat
    bad_d = _Desc(1, 2, 2048, 96, 0, 2 * 2048 * 96, 2048 * 96, 96)
    assert lib.sparge_workspace_bytes(ctypes.byref(bad_d), sp.WS_FORWARD, ctypes.byref(n)) == -2
    assert b"head dim" in lib.sparge_last_error()
    bad_n = _Desc(1, 2, 0, 64, 0, 0, 0, 64)
    assert lib.sparge_workspace_bytes(ctypes.byref(bad_n), sp.WS_FORWARD, ctypes.byref(n)) == -1
    too_long = _Desc(1, 1, 64 * 4096 + 1, 64, 1, 0, 0, 64)
    assert lib.sparge_workspace_bytes(ctypes.byref(too_long), sp.WS_ATTN, ctypes.byref(n)) == -2
    # NULL tensors / bad hyper-parameters are rejected before anything is enqueued
    tau = (ctypes.c_float * 2)(0.9, 1.5)
    theta = (ctypes.c_float * 2)(0.5, 0.5)
    rc = lib.sparge_predict(None, None, ctypes.byref(good), tau, theta, 0.0, 0, None, None, None, None, 0, None)
    assert rc == -1


@pytest.mark.parametrize("B,H,N,d", [(1, 2, 2048, 64), (3, 5, 1000, 128)])
def test_workspaces_hold_what_their_entry_points_use(B, H, N, d):
    """sparge_quantize and sparge_attn need K's block sums but no pooled Q and no similarities; the search needs per
    input a forward workspace and an output, and one more output."""
    import paper_2502_18137_amd as sp
    from paper_2502_18137_amd.binding import _Desc
    lib = sp.load_library()
    desc = _Desc(B, H, N, d, 1, H * N * d, N * d, d)
    def of(entry):
        n = ctypes.c_size_t(0)
        assert lib.sparge_workspace_bytes(ctypes.byref(desc), entry, ctypes.byref(n)) == 0
        return n.value
    up = lambda x: (x + 255) // 256 * 256
    BH, Tm, Tn = B * H, -(-N // 128), -(-N // 64)
    sums = up(BH * Tn * d * 8)
    assert of(sp.WS_QUANTIZE) == sums
    quant = up(BH * d * 4) + 2 * up(BH * N * d) + up(BH * Tm * 4) + up(BH * Tn * 4)
    tail = up(BH * Tn * d * 64 * 2) + 1024                     # V tiles, item counters
    assert of(sp.WS_ATTN) == sums + quant + tail
    stats = up(BH * Tm * d * 8) + up(BH * Tm * 8) + up(BH * Tn * 8)
    assert of(sp.WS_FORWARD) == sums + quant + tail + stats + up(BH * Tm * Tn * 8) + up(BH * Tm * Tn)
    assert of(sp.WS_PREDICT) == sums + stats + up(BH * Tm * Tn * 8)
    for inputs in (1, 3):
        n = ctypes.c_size_t(0)
        assert lib.sparge_tune_workspace_bytes(ctypes.byref(desc), inputs, ctypes.byref(n)) == 0
        assert n.value == inputs * (of(sp.WS_FORWARD) + up(BH * N * d * 2)) + up(BH * N * d * 2)


def test_search_without_host_memory_is_an_error_code():
    """The search's host tables are allocated before anything is enqueued; where they do not fit, the call returns
    SPARGE_ENOSPACE: no exception leaves the C entry.  (In a process of its own with its address space bounded, and
    without a GPU: the device pointers are made up.)"""
    import subprocess
    import sys
    code = """
import ctypes, resource
import paper_2502_18137_amd as sp
from paper_2502_18137_amd.binding import _Desc
lib = sp.load_library()
n = 1 << 20                                         # a table of 2 GiB at 128 heads
one, lam = (ctypes.c_float * 1)(0.5), (ctypes.c_float * n)(*[-1.0] * n)
res, ptr = (ctypes.c_float * 128)(), (ctypes.c_void_p * 1)(4096)
desc = _Desc(1, 128, 64, 64, 1, 128 * 64 * 64, 64 * 64, 64)
used = int(open("/proc/self/statm").read().split()[0]) * resource.getpagesize()
resource.setrlimit(resource.RLIMIT_AS, (used + (1 << 30),) * 2)
rc = lib.sparge_tune(ptr, ptr, ptr, 1, ctypes.byref(desc), one, 1, one, 1, lam, n, 0.1, 0.1, 0.0, 0, res, res, res, None, None, None,
                     None, ctypes.c_void_p(4096), 1 << 40, None)
assert rc == -3 and b"host memory" in lib.sparge_last_error(), (rc, lib.sparge_last_error())
"""
    env = dict(os.environ, HIP_VISIBLE_DEVICES="", PYTHONPATH=ROOT)
    r = subprocess.run([sys.executable, "-c", code], env=env, cwd=ROOT, capture_output=True, text=True, timeout=100)
    assert r.returncode == 0, r.stdout + r.stderr


def test_search_accepts_the_workspace_it_names():
    """sparge_tune_workspace_bytes is enough for every layout the library takes, overlapping batches and heads (stride 0)
    among them, and so is the batched size.  (The call gets past the workspace check and ends at its host tables, which do
    not fit: nothing is enqueued and no GPU is needed.)"""
    import subprocess
    import sys
    code = """
import ctypes, resource
import paper_2502_18137_amd as sp
from paper_2502_18137_amd.binding import _Desc
lib = sp.load_library()
one, ptr = (ctypes.c_float * 1)(0.5), (ctypes.c_void_p * 3)(4096, 4096, 4096)
shapes = [(B, H, N, d, pv, n) for B, H in ((1, 128), (4, 64)) for N in (1, 333, 1536, 8192) for d in (64, 128)
          for pv in (0, 1) for n in (1, 3)]
lams = {}
for H in (64, 128):
    m = (1 << 31) // (16 * H)                           # a table of 2 GiB
    lams[H] = (ctypes.c_float * m).from_buffer(bytearray(bytes([0, 0, 128, 191]) * m))
res = (ctypes.c_float * 128)()
used = int(open("/proc/self/statm").read().split()[0]) * resource.getpagesize()
resource.setrlimit(resource.RLIMIT_AS, (used + (1 << 30),) * 2)
def call(desc, n, H, size):
    rc = lib.sparge_tune(ptr, ptr, ptr, n, ctypes.byref(desc), one, 1, one, 1, lams[H], len(lams[H]), 0.1, 0.1, 0.0, 0, res, res, res,
                         None, None, None, None, ctypes.c_void_p(4096), size, None)
    return rc, lib.sparge_last_error()
for B, H, N, d, pv, n in shapes:
    for sb, sh, sn in ((H * N * d, N * d, d), (N * H * d, d, H * d), (0, N * d, d), (H * N * d, 0, d), (0, 0, d), (2 * H * N * d, N * d + 64, d)):
        desc = _Desc(B, H, N, d, 1, sb, sh, sn, pv, 0)
        for f in (lib.sparge_tune_workspace_bytes, lib.sparge_tune_workspace_batched_bytes):
            size = ctypes.c_size_t(0)
            assert f(ctypes.byref(desc), n, ctypes.byref(size)) == 0
            rc, err = call(desc, n, H, size.value)
            assert rc == -3 and b"host memory" in err, (B, H, N, d, pv, n, sb, sh, sn, rc, err)
        rc, err = call(desc, n, H, 1 << 10)
        assert rc == -3 and b"workspace has" in err, (rc, err)
"""
    env = dict(os.environ, HIP_VISIBLE_DEVICES="", PYTHONPATH=ROOT)
    r = subprocess.run([sys.executable, "-c", code], env=env, cwd=ROOT, capture_output=True, text=True, timeout=100)
    assert r.returncode == 0, r.stdout + r.stderr


def test_missing_library_fails_loudly(monkeypatch):
    import paper_2502_18137_amd.binding as b
    monkeypatch.setattr(b, "_LIB", None)
    monkeypatch.setattr(b, "library_path", lambda: "/nonexistent/libsparge.so")
    with pytest.raises(b.SpargeError):
        b.load_library()
