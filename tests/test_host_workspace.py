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


# a workspace smaller than the named one: row statistics only at fp32 and general widths, the splits of an equal share of the
# rows per compute unit at the widths of the bf16 kernels, and some bytes between (packed inputs with fewer splits)
SMALLER = [("f32", 512, 1024, 768, 205056), ("f32", 512, 1024, 768, 24 << 20), ("bf16", 300, 260, 1000, 66816), ("f32", 2000, 2500, 200, 249600),
           ("bf16", 128, 256, 768, 1185024), ("bf16", 690, 1792, 128, 5302528), ("bf16", 2018, 16468, 512, 67486208), ("bf16", 700, 900, 128, 2865152),
           ("ntxent", 300, 300, 200, 556032), ("ntxent", 1000, 1000, 256, 4169216), ("symmetric", 300, 300, 200, 1111040),
           ("symmetric", 300, 300, 200, 3 << 20), ("symmetric", 700, 700, 768, 12993280), ("bilinear", 300, 500, 256, 3034368)]


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


def test_a_workspace_smaller_than_the_named_one_is_taken_while_some_kernels_fit_it(stub):
    """These sizes were the named ones before the kernels that want more; they are what a program may have kept."""
    got = run(stub, """
from_list = json.loads(%r)
def call(kind, B, P, d, n):
    if kind == "ntxent":
        return lib.gc_ntxent_loss_and_grad_bf16(X, B, d, 0.1, X, X, X, n, None)
    if kind == "symmetric":
        return lib.gc_bidirectional_loss_and_rep_grad_bf16(X, X, X, B, d, 1.0, 1.0, X, X, X, X, n, None)
    if kind == "bilinear":
        return lib.gc_bilinear_loss_and_grads_bf16(X, X, X, B, P, d, X, 1.0, 1.0, X, X, X, X, X, n, None)
    return ex(F32 if kind == "f32" else BF16, B, P, d, n)
def named(kind, B, P, d):
    if kind == "ntxent":
        return lib.gc_ntxent_workspace_bytes(B, d)
    if kind == "symmetric":
        return lib.gc_bidirectional_workspace_bytes(B, d)
    if kind == "bilinear":
        return lib.gc_bilinear_workspace_bytes(B, P, d)
    return lib.gc_workspace_bytes(B, P, d, F32 if kind == "f32" else BF16)
out = []
for c in from_list:
    stub.stub_reset()
    out.append(dict(rc=call(*c), whole=call(*c[:4], named(*c[:4])), named=named(*c[:4]), little=call(*c[:4], 4096), error=stub.stub_last_error()))
report(out=out)
""" % json.dumps(SMALLER))
    for c, o in zip(SMALLER, got["out"]):
        assert o["rc"] == 0 and o["whole"] == 0 and o["little"] == -4 and o["error"] == 0, (c, o)
        assert o["named"] > c[4], (c, o)


def test_a_forward_needs_the_transposed_weights_and_two_activations_only(stub):
    """The named size also covers the fragments of a backward."""
    got = run(stub, """
class Params(ctypes.Structure):
    _fields_ = [(n, vp) for n in ("W1", "b1", "W2", "b2")] + [(n, ci) for n in ("din", "dh", "dout")]
lib.gc_mlp_workspace_bytes.restype, lib.gc_mlp_workspace_bytes.argtypes = sz, [ci, vp]
lib.gc_mlp_forward_nograd_bf16.argtypes = [vp, ci, vp, vp, vp, sz, vp]
out = []
for rows, din, dh, dout in ((1, 64, 128, 128), (200, 128, 256, 128), (2048, 1024, 3072, 768)):
    w = Params(X, X, X, X, din, dh, dout)
    need = (din * dh + dh * dout) * 2 + 2 * rows * dh * 4
    call = lambda n: lib.gc_mlp_forward_nograd_bf16(X, rows, ctypes.byref(w), X, X, n, None)
    out.append([call(need), call(need - 256), need < lib.gc_mlp_workspace_bytes(rows, ctypes.byref(w))])
report(out=out)
""")
    assert got["out"] == [[0, -4, True]] * 3


# (type, B, P, d, gradient kernel of the call): D and whether it merges the statistics itself; planes, owner blocks, column tiles, merge
FEW = [("bf16", 1, 1, 256, "grad_few_kernelILi256ELb0ELb1E"), ("bf16", 129, 257, 384, "grad_few_kernelILi384ELb0ELb1E"),
       ("bf16", 70, 9000, 512, "grad_few_kernelILi512ELb0ELb1E"), ("bf16", 9000, 70, 768, "grad_few_kernelILi768ELb0ELb0E"),
       ("bf16", 1021, 1000, 640, "grad_few_kernelILi640ELb0ELb1E"), ("bf16", 97, 4000, 768, "grad_few_kernelILi768ELb0ELb1E"),
       ("f32", 33, 31, 776, "planes_grad_kernelILi3ELi1ELi8ELb1E"), ("f32", 129, 257, 129, "planes_grad_kernelILi3ELi1ELi2ELb1E"),
       ("f32", 9000, 70, 520, "planes_grad_kernelILi3ELi1ELi6ELb0E"), ("f32", 200, 300, 2100, "planes_grad_kernelILi3ELi1ELi6ELb1E"),
       ("bf16", 512, 512, 400, "planes_grad_kernelILi1ELi1ELi4ELb1E"), ("bf16", 1000, 1040, 1000, "planes_grad_kernelILi1ELi1ELi8ELb0E")]


def test_few_scores_reach_the_kernels_that_their_parity_tests_mean(stub):
    got = run(stub, """
out = []
for dt, B, P, d, _ in json.loads(%r):
    stub.stub_reset()
    rc = ex(F32 if dt == "f32" else BF16, B, P, d, lib.gc_workspace_bytes(B, P, d, F32 if dt == "f32" else BF16))
    out.append([rc, stub.stub_launches().decode()])
report(out=out)
""" % json.dumps(FEW))
    for c, (rc, names) in zip(FEW, got["out"]):
        assert rc == 0 and c[4] in names, (c, names)


ENCODER = """
class Params(ctypes.Structure):
    _fields_ = [(n, vp) for n in ("W1", "b1", "W2", "b2")] + [(n, ci) for n in ("din", "dh", "dout")]
class Grads(ctypes.Structure):
    _fields_ = [(n, vp) for n in ("dW1", "db1", "dW2", "db2")]
lib.gc_mlp_workspace_bytes.restype, lib.gc_mlp_workspace_bytes.argtypes = sz, [ci, vp]
lib.gc_mlp_forward_nograd_bf16.argtypes = [vp, ci, vp, vp, vp, sz, vp]
lib.gc_chunk_surrogate_backward_bf16.argtypes = [vp, ci, vp, vp, vp, vp, sz, vp]
lib.gc_step_mlp_workspace_bytes.restype, lib.gc_step_mlp_workspace_bytes.argtypes = sz, [ci] * 4 + [vp]
lib.gc_step_mlp_bf16.argtypes = [vp, ci, vp, ci, vp, ci, ci, vp, cf, cf, vp, vp, vp, vp, vp, vp, vp, sz, vp]
G = Grads(X, X, X, X)
def of(call):
    stub.stub_reset()
    rc = call()
    return [rc, stub.stub_last_error(), [l.split()[0] for l in stub.stub_launches().decode().splitlines()], stub.stub_misaligned()]
def forward(rows, w, x=X):
    return of(lambda: lib.gc_mlp_forward_nograd_bf16(x, rows, ctypes.byref(w), X, X, lib.gc_mlp_workspace_bytes(rows, ctypes.byref(w)), None))
def backward(rows, w, x=X, u=X):
    return of(lambda: lib.gc_chunk_surrogate_backward_bf16(x, rows, ctypes.byref(w), u, ctypes.byref(G), X, lib.gc_mlp_workspace_bytes(rows, ctypes.byref(w)), None))
def step(B, P, w, xq=X, xp=X):
    return of(lambda: lib.gc_step_mlp_bf16(xq, B, xp, P, X, 32, 32, ctypes.byref(w), 1.0, 1.0, X, ctypes.byref(G), X, X, X, X, X,
                                           lib.gc_step_mlp_workspace_bytes(B, P, 32, 32, ctypes.byref(w)), None))
def bilinear(B, P, d, q=X, om=X):
    return of(lambda: lib.gc_bilinear_loss_and_grads_bf16(q, X, X, B, P, d, om, 1.0, 1.0, X, X, X, X, X, lib.gc_bilinear_workspace_bytes(B, P, d), None))
"""
RING = ("mlp_hidden_kernel", "mlp_output_kernel", "mlp_dh_tiled_kernel")


def test_operands_aligned_to_their_elements_only_are_copied_for_the_16_byte_loads(stub):
    """The ring's loads into LDS take 16 bytes at 16-byte addresses: an operand that lies elsewhere is copied once a call (rows: once a
    launch), and the kernels are those of aligned operands."""
    got = run(stub, ENCODER + """
w = lambda *s, **k: Params(*[X + 2 * k.get(n, 0) for n in ("W1", "b1", "W2", "b2")], *(s or (256, 2048, 256)))
out = dict(
    aligned=[forward(300, w()), backward(300, w()), step(200, 300, w()), bilinear(300, 600, 256), step(3000, 100, w())],
    forward=[forward(300, w(), X + 2), forward(300, w(W1=1)), forward(5000, w(W2=5)), forward(300, w(W1=1, W2=1), X + 2), forward(300, w(b1=1, b2=3))],
    backward=[backward(300, w(), X + 2), backward(300, w(W1=1)), backward(300, w(W1=1), X + 6), backward(300, w(W2=1)), backward(300, w(), X, X + 4)],
    step=[step(200, 300, w(W1=1)), step(200, 300, w(W2=1)), step(3000, 100, w(W1=1, W2=1))],
    inputs=[step(200, 300, w(), X + 2), step(200, 300, w(), X, X + 2), step(20, 30, w(), X + 2, X + 2), step(5000, 300, w(W1=3, W2=3), X + 2, X + 2)],
    halves=[forward(3000, w(2048, 512, 128), X + 2), backward(3000, w(2048, 512, 128), X + 2), backward(6000, w(2048, 128, 128), X + 2)], few=[forward(3000, w(1280, 128, 128), X + 2), forward(100, w(W1=1, W2=1), X + 2)],
    bilinear=[bilinear(300, 600, 256, X + 2), bilinear(300, 600, 256, X, X + 2), bilinear(300, 600, 256, X + 2, X + 6)])
report(**out)
""")
    named = lambda r, *k: [n for n in r[2] if any(x in n for x in k)]  # noqa: E731
    copies = lambda r: len(named(r, "copy_aligned_kernel"))  # noqa: E731
    rest = lambda r: [n for n in r[2] if "copy_aligned" not in n]  # noqa: E731
    for k in got:
        for r in got[k]:
            assert r[0] == 0 and r[1] == 0 and r[3] == 0, (k, r)
    fwd, bwd, st, bil, mixed = got["aligned"]
    assert len(named(fwd, *RING)) == 2 and len(named(bwd, *RING)) == 1 and len(named(st, *RING)) == 3 and not copies(st)
    assert [copies(r) for r in got["forward"]] == [1, 1, 1, 3, 0] and [copies(r) for r in got["backward"]] == [1, 1, 2, 0, 0]
    assert all(len(named(r, *RING)) == 2 and not named(r, "skinny") for r in got["forward"])
    assert all(rest(r) == bwd[2] for r in got["backward"])
    # (W2: of a backward only fragments are read.  3000 x 100: the copies for the anchors are over when the targets' fragments come)
    assert [copies(r) for r in got["step"]] == [1, 1, 3] and rest(got["step"][0]) == rest(got["step"][1]) == st[2] and rest(got["step"][2]) == mixed[2]
    one, other, few, many = got["inputs"]
    assert copies(one) == copies(other) == 2 and len(named(one, *RING)) == len(named(other, *RING)) == 6 and not named(one, "skinny")
    assert not copies(few) and named(few, "mlp_dh_skinny") and not named(few, *RING)
    assert copies(many) == 2 + 2 * 4 and len(named(many, "mlp_hidden")) == 4 and len(named(many, "mlp_dh_tiled")) == 4
    assert [copies(r) for r in got["halves"]] == [2, 2, 2] and [len(named(r, "mlp_hidden", "mlp_dh_tiled")) for r in got["halves"]] == [2, 2, 2]
    assert all(not copies(r) and not named(r, *RING) and named(r, "mlp_skinny") for r in got["few"])
    for r, n, ends in zip([bil] + got["bilinear"], (0, 1, 1, 2), (1, 2, 1, 2)):
        assert copies(r) == n and len(named(r, "bilinear_end_kernel")) == ends, r
        if n:
            assert "copy_aligned" in r[2][0] and "bilinear_project" in r[2][n]


# (rows, din, dh, dout): tiles in units of 64 of the hidden layer, the output layer, Act and dH, or None for the kernel for few rows; whether
# the parameter gradients take their kernel for few rows
TILES = [((31, 64, 128, 128), None, None, None, True), ((65, 128, 256, 256), None, None, None, True), ((129, 64, 128, 128), (1, 2), (1, 2), None, True),
         ((192, 320, 256, 128), (1, 2), (1, 2), None, True), ((193, 64, 384, 384), (1, 2), (1, 2), None, False),
         ((255, 192, 1408, 256), (1, 2), (1, 2), (1, 2), False), ((1000, 64, 2176, 128), (2, 2), (1, 2), (2, 2), False),
         ((1500, 128, 3200, 128), (2, 3), (1, 2), (2, 3), False), ((1024, 64, 3072, 768), (2, 2), (2, 2), (2, 2), False),
         ((2040, 64, 3072, 768), (2, 2), (2, 3), (2, 3), False)]
# (B, P, d): tiles of H and of u
BILINEAR = [((1, 3, 128), (1, 2), (1, 2)), ((1000, 100, 512), (1, 2), (1, 2)), ((2560, 40, 768), (1, 2), (2, 2)), ((4096, 64, 768), (2, 2), (2, 3)),
            ((5600, 40, 768), (2, 3), (2, 2))]


def test_sizes_reach_the_tiles_that_their_parity_tests_mean(stub):
    got = run(stub, ENCODER + """
out = []
for rows, din, dh, dout in json.loads(%r):
    w = Params(X, X, X, X, din, dh, dout)
    out.append([forward(rows, w), backward(rows, w)])
report(encoder=out, bilinear=[bilinear(*c) for c in json.loads(%r)])
""" % (json.dumps([t[0] for t in TILES]), json.dumps([t[0] for t in BILINEAR])))

    def has(r, kernel, tile):
        return any("%sILi%dELi%dE" % ((kernel,) + tile) in n for n in r[2])

    for (size, hidden, output, dh, few), (f, b) in zip(TILES, got["encoder"]):
        for r, kernel, tile, other in ((f, "mlp_hidden_kernel", hidden, "mlp_skinny"), (f, "mlp_output_kernel", output, "mlp_skinny"),
                                       (b, "mlp_dh_tiled_kernel", dh, "mlp_dh_skinny")):
            assert has(r, kernel, tile) if tile else any(other in n for n in r[2]), (size, kernel, r)
        assert any("mlp_grads_few_kernel" in n for n in b[2]) == few, (size, b)
    for (size, h, u), r in zip(BILINEAR, got["bilinear"]):
        assert has(r, "bilinear_project_kernel", h) and has(r, "bilinear_end_kernel", u), (size, r)
