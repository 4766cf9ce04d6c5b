"""Workspaces of the loss path on the host: the library's own buffer under a capture and on a card with little room, and
workspaces smaller than the named one.  The library runs against a HIP runtime without a device (hip_stub.c), in a process
of its own."""
import json
import os
import subprocess
import sys

import pytest

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)

PRELUDE = """
import ctypes, json, os, sys
stub = ctypes.CDLL(sys.argv[1], mode=ctypes.RTLD_GLOBAL)
lib = ctypes.CDLL(sys.argv[2])
vp, ci, cf, sz = ctypes.c_void_p, ctypes.c_int, ctypes.c_float, ctypes.c_size_t
stub.stub_room.argtypes = [sz]
stub.stub_launches.restype = ctypes.c_char_p
for n in ("stub_used", "stub_peak"):
    getattr(stub, n).restype = sz
for n, k in (("gc_workspace_bytes", 4), ("gc_ntxent_workspace_bytes", 2), ("gc_bidirectional_workspace_bytes", 2), ("gc_bilinear_workspace_bytes", 3)):
    getattr(lib, n).restype, getattr(lib, n).argtypes = sz, [ci] * k
for n in ("gc_loss_and_rep_grad_f32", "gc_loss_and_rep_grad_bf16"):
    getattr(lib, n).argtypes = [vp, vp, vp, ci, ci, ci, cf, cf, vp, vp, vp, vp]
lib.gc_loss_and_rep_grad_ex.argtypes = [ci, vp, vp, vp, ci, ci, ci, cf, cf, ctypes.c_uint, vp, vp, vp, vp, vp, vp, sz, vp]
lib.gc_ntxent_loss_and_grad_bf16.argtypes = [vp, ci, ci, cf, vp, vp, vp, sz, vp]
lib.gc_bidirectional_loss_and_rep_grad_bf16.argtypes = [vp, vp, vp, ci, ci, cf, cf, vp, vp, vp, vp, sz, vp]
lib.gc_bilinear_loss_and_grads_bf16.argtypes = [vp, vp, vp, ci, ci, ci, vp, cf, cf, vp, vp, vp, vp, vp, sz, vp]
F32, BF16, MIB = 0, 1, 1 << 20
X = 1 << 20   # addresses that nothing reads
def plain(dt, B, P, d):
    return (lib.gc_loss_and_rep_grad_f32 if dt == F32 else lib.gc_loss_and_rep_grad_bf16)(X, X, X, B, P, d, 1.0, 1.0, X, X, X, None)
def ex(dt, B, P, d, n):
    return lib.gc_loss_and_rep_grad_ex(dt, X, X, X, B, P, d, 1.0, 1.0, 0, X, X, X, None, None, X, n, None)
def launched(name):
    return name in stub.stub_launches().decode()
def report(**k):
    print("RESULT " + json.dumps(k))
"""


@pytest.fixture(scope="module")
def stub(tmp_path_factory):
    out = str(tmp_path_factory.mktemp("hip") / "libhipstub.so")
    r = subprocess.run(["gcc", "-O1", "-shared", "-fPIC", "-o", out, os.path.join(HERE, "hip_stub.c")], capture_output=True, text=True)
    assert r.returncode == 0, r.stderr
    return out


def run(stub, body):
    from paper_2101_06983_amd import binding
    r = subprocess.run([sys.executable, "-c", PRELUDE + body, stub, binding.LIB_PATH], capture_output=True, text=True, timeout=120)
    assert r.returncode == 0, r.stdout + r.stderr
    return json.loads([l for l in r.stdout.splitlines() if l.startswith("RESULT ")][-1][7:])


def test_a_buffer_that_a_capture_has_recorded_is_kept_when_a_later_call_needs_a_larger_one(stub):
    """The replayed graph goes on using the recorded address: giving that memory back would be a use after free."""
    got = run(stub, """
first = plain(F32, 32, 64, 200)                 # the library's buffer: 1 MiB
stub.stub_capturing(1)
captured = plain(F32, 300, 500, 200)            # what fits it
general = launched("grad_generic_kernel") and stub.stub_last_error() == 0
stub.stub_capturing(0)
stub.stub_reset()
later = plain(F32, 300, 500, 200)               # the kernels that want more
report(first=first, captured=captured, general=general, later=later, mallocs=stub.stub_mallocs(), frees=stub.stub_frees(),
       again=plain(F32, 512, 1024, 768), frees_again=stub.stub_frees(), error=lib.gc_check_async_error(None))
""")
    assert got["first"] == got["captured"] == got["later"] == got["again"] == 0 and got["general"]
    assert got["mallocs"] == 1 and got["frees"] == 0
    assert got["frees_again"] == 1      # the second buffer was in no capture
    assert got["error"] == 0


@pytest.mark.parametrize("mib,kernel", [(45, "planes_grad_kernel"), (25, "planes_grad_kernel"), (1, "grad_generic_kernel")])
def test_first_call_on_a_device_with_little_room(stub, mib, kernel):
    """512 x 1024 x 768 in fp32 wants 40 MB for packed inputs and partial sums, a quarter more to grow, 22 MB with one split,
    and needs 0.2 MB of row statistics."""
    got = run(stub, """
stub.stub_room(%d * MIB)
rc = [plain(F32, 512, 1024, 768) for _ in range(3)]
report(rc=rc, names=stub.stub_launches().decode(), mallocs=stub.stub_mallocs(), frees=stub.stub_frees(), error=stub.stub_last_error(),
       none=plain(BF16, 4096, 8192, 768), none_error=stub.stub_last_error())
""" % mib)
    assert got["rc"] == [0, 0, 0] and kernel in got["names"]
    assert got["mallocs"] <= 2 and got["frees"] == 0 and got["error"] == 0
    assert got["none"] == -6 and got["none_error"] == 0      # no kernels of this width need that little


def test_a_buffer_that_cannot_grow_stays_in_use(stub):
    got = run(stub, """
first = plain(F32, 32, 64, 200)
stub.stub_room(stub.stub_used() + MIB // 2)
stub.stub_reset()
rc = [plain(F32, 512, 1024, 768) for _ in range(3)]
report(first=first, rc=rc, names=stub.stub_launches().decode(), mallocs=stub.stub_mallocs(), frees=stub.stub_frees(), error=stub.stub_last_error())
""")
    assert got["first"] == 0 and got["rc"] == [0, 0, 0] and "grad_generic_kernel" in got["names"]
    assert got["mallocs"] == 0 and got["frees"] == 0 and got["error"] == 0
