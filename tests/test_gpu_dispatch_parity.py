"""GPU parity at the edges of the kernels' tiles and of the rules that choose between them, against the fp64 oracle."""
import numpy as np
import pytest
import torch

from paper_2101_06983_amd import binding as gc
from paper_2101_06983_amd import synth
from parity import TOL_BF16, TOL_F32, check, check_argmax, check_loss, oracle_loss, relerr, to_np
from test_host_workspace import SMALLER

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


@pytest.mark.parametrize("B,P,d,named", [(255, 40, 128, 40), (256, 9, 256, 1), (257, 700, 384, 5), (1021, 300, 128, 300),
                                         (2, 3, 768, 1)])
def test_targets_shared_by_several_anchors(B, P, d, named):
    """dP rows that sum the terms of several anchors: fewer, exactly and more anchors than one pass of the sum kernel
    looks at, a single target for all of them, rows that straddle two workgroups, rows nobody names."""
    q, p, _ = synth.dpr_batch(B, P, d, seed=4000 + B)
    r = torch.from_numpy(np.random.default_rng(B).integers(0, named, size=B).astype(np.int32))
    want = oracle_loss(q, p, r, 1.0, 0.3)
    out = gc.gc_loss_and_rep_grad_ex(q.to(DEV), p.to(DEV), r.to(DEV), 1.0, 0.3)
    torch.cuda.synchronize()
    check_loss("shared loss", out["loss"].item(), want["loss"], TOL_BF16)
    for k in ("dq", "dp"):
        check("shared %dx%dx%d %s" % (B, P, d, k), relerr(to_np(out[k]), want[k]), TOL_BF16)


def run_ex(q, p, r, scale, temp, flags=0):
    out = gc.gc_loss_and_rep_grad_ex(q, p, r, scale, temp, flags)
    torch.cuda.synchronize()
    assert gc.gc_check_async_error(out["workspace"]) == gc.GC_OK
    return out


# fp32 arithmetic whatever the storage: the fp32 tolerance also for bf16 inputs
def check_fp32_grade(label, out, want, q, p, alpha):
    check_loss(label + " loss", out["loss"].item(), want["loss"], TOL_F32, 1e-30)
    for k in ("dq", "dp", "lse"):
        check(label + " " + k, relerr(to_np(out[k]), want[k]), TOL_F32)
    assert check_argmax(to_np(out["argmax"]), want, synth.widen(q), synth.widen(p), alpha, 1e-5) <= max(1, len(want["argmax"]) // 500)


@pytest.mark.parametrize("dtype", [torch.float32, torch.bfloat16])
@pytest.mark.parametrize("B,P,d", [(31, 33, 65), (129, 127, 63), (128, 256, 64), (5, 700, 130), (700, 5, 97), (300, 260, 1025),
                                   (70, 90, 1023), (40, 257, 2112), (257, 129, 776), (33, 32, 520), (1, 600, 264), (520, 1, 1024)])
def test_any_width_in_fp32_grade(B, P, d, dtype):
    """Edges of the 32-row blocks, the 128-row steps, the 64-column padding, the column slices of 1024; widths whose
    rows are and are not whole 16-byte vectors; streams of one row."""
    q, p, _ = synth.dpr_batch(B, P, d, dtype, seed=4200 + B)
    r = torch.from_numpy(np.random.default_rng(B + P).integers(0, P, size=B).astype(np.int32))
    want = oracle_loss(q, p, r, 1.0, 0.5)
    check_fp32_grade("%dx%dx%d %s" % (B, P, d, dtype), run_ex(q.to(DEV), p.to(DEV), r.to(DEV), 1.0, 0.5), want, q, p, 2.0)


@pytest.mark.parametrize("B,P,d,dtype", [(4096, 4100, 64, torch.float32), (4100, 4096, 72, torch.bfloat16), (4096, 4096, 200, torch.float32)])
def test_any_width_large_batch(B, P, d, dtype):
    # (64 owner rows per workgroup from here on)
    q, p, r = synth.dpr_batch(B, P, d, dtype, seed=4300 + d, positive_mix=0.3)
    want = oracle_loss(q, p, r, 1.0, 0.25)
    check_fp32_grade("%dx%dx%d %s" % (B, P, d, dtype), run_ex(q.to(DEV), p.to(DEV), r.to(DEV), 1.0, 0.25), want, q, p, 4.0)


@pytest.mark.parametrize("dtype,shift", [(torch.float32, 1), (torch.bfloat16, 1), (torch.float32, 3), (torch.bfloat16, 5)])
def test_inputs_and_outputs_aligned_to_their_elements_only(dtype, shift):
    B, P, d = 70, 130, 136
    q, p, r = synth.dpr_batch(B, P, d, dtype, seed=4400)
    want = oracle_loss(q, p, r)

    def off(t):
        buf = torch.empty(t.numel() + shift, dtype=t.dtype, device=DEV)
        buf[shift:] = t.reshape(-1).to(DEV)
        return buf[shift:].view(t.shape)

    out = dict(dq=off(torch.zeros(B, d)), dp=off(torch.zeros(P, d)))
    got = gc.gc_loss_and_rep_grad_ex(off(q), off(p), r.to(DEV), out=out)
    torch.cuda.synchronize()
    check_fp32_grade("shifted by %d %s" % (shift, dtype), got, want, q, p, 1.0)


@pytest.mark.parametrize("n,d", [(66, 96), (300, 200)])
def test_masked_ntxent_and_symmetric_at_any_width(n, d):
    q, p, _ = synth.dpr_batch(n, n, d, seed=4500 + n, positive_mix=0.2)
    r = torch.arange(n, dtype=torch.int32) ^ 1
    want = oracle_loss(q, p, r, 1.0, 0.5, mask_self=True)
    check_fp32_grade("mask n=%d d=%d" % (n, d), run_ex(q.to(DEV), p.to(DEV), r.to(DEV), 1.0, 0.5, gc.GC_MASK_SELF), want, q, p, 2.0)
    z = synth.ntxent_views(n, d, seed=4510)
    want = oracle_loss(z, z, r, 1.0, 0.2, mask_self=True)
    loss, dz = gc.gc_ntxent_loss_and_grad_bf16(z.to(DEV), 0.2)
    torch.cuda.synchronize()
    check_loss("ntxent n=%d d=%d" % (n, d), loss.item(), want["loss"], TOL_F32)
    check("ntxent n=%d d=%d dz" % (n, d), relerr(to_np(dz), want["dq"] + want["dp"]), TOL_F32)
    perm = torch.from_numpy(np.random.default_rng(n).permutation(n).astype(np.int32))
    from oracle import gc_oracle as O
    want = O.bidirectional(synth.widen(q), synth.widen(p), perm.numpy(), 1.0, 0.5)
    out = gc.gc_bidirectional_loss_and_rep_grad_bf16(q.to(DEV), p.to(DEV), perm.to(DEV), 1.0, 0.5)
    torch.cuda.synchronize()
    check_loss("symmetric n=%d d=%d" % (n, d), out["loss"].item(), want["loss"], TOL_F32)
    for k in ("dq", "dp"):
        check("symmetric n=%d d=%d %s" % (n, d, k), relerr(to_np(out[k]), want[k]), TOL_F32)


@pytest.mark.parametrize("B,P,d", [(300, 500, 200), (512, 1024, 1000), (2000, 3000, 520), (3000, 4000, 520)])
def test_static_scratch_takes_every_width_it_took(B, P, d):
    """Where the packed inputs do not fit the fixed array beside the partials, fewer splits (the second and third shape) or
    the general kernels (the last) serve the call; the workspace-less entry point takes the same shapes with the room it
    wants."""
    q, p, r = synth.dpr_batch(B, P, d, seed=4600 + d, positive_mix=0.3)
    want = oracle_loss(q, p, r, 1.0, 0.5)
    for call in (gc.gc_loss_and_rep_grad_bf16_static, gc.gc_loss_and_rep_grad_bf16):
        loss, dq, dp = call(q.to(DEV), p.to(DEV), r.to(DEV), 1.0, 0.5)
        torch.cuda.synchronize()
        assert gc.gc_check_async_error() == gc.GC_OK
        check_loss("static %dx%dx%d" % (B, P, d), loss.item(), want["loss"], TOL_F32)
        check("static %dx%dx%d dq" % (B, P, d), relerr(to_np(dq), want["dq"]), TOL_F32)
        check("static %dx%dx%d dp" % (B, P, d), relerr(to_np(dp), want["dp"]), TOL_F32)


CAPTURE = """
import sys, torch
sys.path.insert(0, %r)
from paper_2101_06983_amd import binding as gc
g = torch.Generator(device="cuda").manual_seed(1)
mk = lambda n, d: torch.randn(n, d, generator=g, device="cuda") * d ** -0.5
gc.gc_loss_and_rep_grad_f32(mk(8, 64), mk(16, 64), torch.arange(8, device="cuda", dtype=torch.int32))   # the library's buffer: 1 MiB
q, p, r = mk(300, 200), mk(500, 200), torch.arange(300, device="cuda", dtype=torch.int32)
torch.cuda.synchronize()
graph = torch.cuda.CUDAGraph()
with torch.cuda.graph(graph):
    got = gc.gc_loss_and_rep_grad_f32(q, p, r)
for k in range(3):
    q.copy_(mk(300, 200))
    graph.replay()
    torch.cuda.synchronize()
    want = gc.gc_loss_and_rep_grad_ex(q, p, r, want=("loss", "dq", "dp"))
    torch.cuda.synchronize()
    for a, b in zip(got, (want["loss"], want["dq"], want["dp"])):
        assert (a - b).abs().max().item() <= 1e-5 * b.abs().max().item(), k
print("replays agree")
"""


def test_capture_with_the_library_buffer_too_small_for_the_packed_inputs():
    """A capture cannot grow the library's buffer: a width that needed little workspace is still served."""
    import os
    import subprocess
    import sys
    root = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
    r = subprocess.run([sys.executable, "-c", CAPTURE % root], capture_output=True, text=True, timeout=100)
    assert r.returncode == 0 and "replays agree" in r.stdout, r.stdout + r.stderr


@pytest.mark.parametrize("rows,din,dh,dout", [(33, 192, 128, 128), (96, 64, 384, 256), (127, 128, 256, 128), (128, 320, 256, 128),
                                              (129, 128, 256, 128), (300, 192, 384, 256), (1500, 64, 128, 128),
                                              (2731, 64, 3072, 128)])
def test_chunk_backward_row_edges(rows, din, dh, dout):
    """The 32-row, 64-row and 128-row tiles of the backward, whole and ragged; inputs of an odd number of 64 columns."""
    from oracle import gc_oracle as O
    x, _, _, params = synth.mlp_problem(rows, 1, din, dh, dout, seed=4700 + rows)
    u = torch.from_numpy((np.random.default_rng(rows).standard_normal((rows, dout)) * 1e-3).astype(np.float32))
    want = O.mlp_backward(synth.widen(x), {k: synth.widen(v) for k, v in params.items()}, synth.widen(u))
    dev = {k: v.to(DEV) for k, v in params.items()}
    grads = {k: torch.full(v.shape, 0.25, dtype=torch.float32, device=DEV) for k, v in params.items()}   # added to
    gc.gc_chunk_surrogate_backward_bf16(x.to(DEV), dev, u.to(DEV), grads)
    torch.cuda.synchronize()
    for k in ("W1", "b1", "W2", "b2"):
        got = to_np(grads[k]) - 0.25
        # 0.25 + g is stored in fp32: half an ulp of the sum beside the arithmetic
        check("backward rows=%d %dx%dx%d d%s" % (rows, din, dh, dout, k), max(0.0, np.abs(got - want[k]).max() - 2.0 ** -25),
              TOL_BF16 * np.abs(want[k]).max())


@pytest.mark.parametrize("dtype", [torch.float32, torch.bfloat16])
@pytest.mark.parametrize("B,P,d", [(1, 1, 1), (1, 17, 3), (17, 1, 5), (32, 64, 64), (70, 40, 33), (8, 32, 760), (3, 1000, 20), (1000, 3, 20)])
def test_a_handful_of_scores(B, P, d, dtype):
    """Calls that one workgroup serves whole, up to the line (32 x 64 x 64, 8 x 32 x 760; 768 in bf16 is one of the
    widths with bf16 coefficients and not of this path) and beyond a wave and a workgroup of rows and columns."""
    q, p, _ = synth.dpr_batch(B, P, d, dtype, seed=4800 + B)
    r = torch.from_numpy(np.random.default_rng(B + P).integers(0, P, size=B).astype(np.int32))
    want = oracle_loss(q, p, r, 1.0, 0.5)
    check_fp32_grade("tiny %dx%dx%d %s" % (B, P, d, dtype), run_ex(q.to(DEV), p.to(DEV), r.to(DEV), 1.0, 0.5), want, q, p, 2.0)
    if B >= 2:
        r[1] = P   # out of range: reported, and the other rows' statistics are unaffected
        out = gc.gc_loss_and_rep_grad_ex(q.to(DEV), p.to(DEV), r.to(DEV), 1.0, 0.5)
        torch.cuda.synchronize()
        assert gc.gc_check_async_error(out["workspace"]) == gc.GC_ERR_POS_IDX and torch.isnan(out["loss"]).all()
        check("tiny lse beside a bad positive", relerr(to_np(out["lse"]), want["lse"]), TOL_F32)


def test_a_handful_of_scores_masked_ntxent_and_symmetric():
    n, d = 30, 24
    q, p, _ = synth.dpr_batch(n, n, d, seed=4900, positive_mix=0.2)
    r = torch.arange(n, dtype=torch.int32) ^ 1
    want = oracle_loss(q, p, r, 1.0, 0.5, mask_self=True)
    check_fp32_grade("tiny mask", run_ex(q.to(DEV), p.to(DEV), r.to(DEV), 1.0, 0.5, gc.GC_MASK_SELF), want, q, p, 2.0)
    z = synth.ntxent_views(n, d, seed=4910)
    want = oracle_loss(z, z, r, 1.0, 0.2, mask_self=True)
    loss, dz = gc.gc_ntxent_loss_and_grad_bf16(z.to(DEV), 0.2)
    torch.cuda.synchronize()
    check_loss("tiny ntxent", loss.item(), want["loss"], TOL_F32)
    check("tiny ntxent dz", relerr(to_np(dz), want["dq"] + want["dp"]), TOL_F32)
    from oracle import gc_oracle as O
    perm = torch.from_numpy(np.random.default_rng(n).permutation(n).astype(np.int32))
    want = O.bidirectional(synth.widen(q), synth.widen(p), perm.numpy(), 1.0, 0.5)
    out = gc.gc_bidirectional_loss_and_rep_grad_bf16(q.to(DEV), p.to(DEV), perm.to(DEV), 1.0, 0.5)
    torch.cuda.synchronize()
    check_loss("tiny symmetric", out["loss"].item(), want["loss"], TOL_F32)
    for k in ("dq", "dp"):
        check("tiny symmetric " + k, relerr(to_np(out[k]), want[k]), TOL_F32)


@pytest.mark.parametrize("B,P", [(33, 70), (200, 130)])
def test_deep_distance_with_saturated_rows(B, P):
    """Pre-activations far beyond where 2^a 2^c can be formed from its factors, on some anchors and some targets (tiles with
    and without such rows, pairs whose large parts cancel): z has an error of some ulp of its largest part, 100 here, and
    so has tanh z where it is not saturated: 100 * 2^-22 = 2.4e-5, within the 1e-4 of the other cases."""
    from oracle import gc_oracle as O
    d = 128
    q, p, _ = synth.dpr_batch(B, P, d, torch.float32, seed=5000 + B)
    q[::3] *= 25.0
    p[5::7] *= 25.0
    p[40] = -q[3]
    q, p = q.to(torch.bfloat16), p.to(torch.bfloat16)
    om = synth.deep_omega(d)
    om["C"] = om["A"].clone()      # a_3 + c_40 = 0 although both are large
    r = torch.from_numpy(np.random.default_rng(B).integers(0, P, size=B).astype(np.int32))
    om64 = {k: synth.widen(v) for k, v in om.items()}
    assert np.abs(synth.widen(q) @ om64["A"].T).max() * 2 / np.log(2.0) > 120.0
    want = O.deep_distance(synth.widen(q), synth.widen(p), synth.widen(r), om64, 1.0, 0.5)
    out = gc.gc_deepdist_loss_and_grads_bf16(q.to(DEV), p.to(DEV), r.to(DEV), {k: v.to(DEV) for k, v in om.items()}, 1.0, 0.5)
    torch.cuda.synchronize()
    check_loss("saturated deep loss", out["loss"].item(), want["loss"], 1e-4)
    for k in ("u", "v", "dA", "dC", "dw"):
        check("saturated deep %dx%d %s" % (B, P, k), relerr(to_np(out[k]), want[k]), 1e-4)


def masked_batch(B, P, d, seed):
    """Features of one sign, so that a target with a large negative feature has a large negative logit for every anchor;
    the targets of `out` are masked (by the caller) and nobody's positive."""
    rng = np.random.default_rng(seed)
    q = torch.from_numpy((0.05 + rng.random((B, d))).astype(np.float32)) * (2.0 / d)
    p = torch.from_numpy((0.05 + rng.random((P, d))).astype(np.float32))
    out = rng.permutation(P)[:max(2, P // 16)]
    r = torch.from_numpy(rng.choice(np.setdiff1d(np.arange(P), out), size=B).astype(np.int32))
    return q, p, r, torch.from_numpy(out)


# one workgroup; few scores; the larger statistics kernel; 64 owner rows per workgroup
MASK_SHAPES = [(8, 24, 40), (64, 96, 200), (70, 130, 776), (1100, 1000, 96), (2100, 4100, 130)]


@pytest.mark.parametrize("lowest", [torch.finfo(torch.float32).min, -3.3961775e38, -3.39e38])
@pytest.mark.parametrize("B,P,d", MASK_SHAPES)
def test_targets_masked_by_the_types_lowest_value(B, P, d, lowest):
    """A feature (of some targets: every feature) at the lowest fp32 value, which rounds to minus infinity in bf16, at the
    first value that does, and at one just above: the target's weight is 0 and everything else is as if it were not there."""
    q, p, r, out = masked_batch(B, P, d, 5100 + B)
    p[out, 3] = lowest
    p[out[0]] = lowest
    want = oracle_loss(q, p, r, 1.0, 0.5)
    check_fp32_grade("lowest %dx%dx%d" % (B, P, d), run_ex(q.to(DEV), p.to(DEV), r.to(DEV), 1.0, 0.5), want, q, p, 2.0)


@pytest.mark.parametrize("dtype", [torch.float32, torch.bfloat16])
@pytest.mark.parametrize("B,P,d", MASK_SHAPES)
def test_targets_masked_by_an_infinite_feature(B, P, d, dtype):
    """Weight 0 times the infinity is NaN in that column of dq, as in any arithmetic; nothing else sees it."""
    q, p, r, out = masked_batch(B, P, d, 5200 + B)
    p[out, 3] = -torch.inf
    q, p = q.to(dtype), p.to(dtype)
    with np.errstate(invalid="ignore"):
        want = oracle_loss(q, p, r, 1.0, 0.5)
    got = run_ex(q.to(DEV), p.to(DEV), r.to(DEV), 1.0, 0.5)
    assert torch.isnan(got["dq"][:, 3]).all() and np.isnan(want["dq"][:, 3]).all()
    got["dq"][:, 3] = 0.0
    want["dq"][:, 3] = 0.0
    with np.errstate(invalid="ignore"):
        check_fp32_grade("infinite feature %dx%dx%d" % (B, P, d), got, want, q, p, 2.0)


@pytest.mark.parametrize("B,P,d", MASK_SHAPES)
def test_targets_masked_by_products_beyond_the_fp32_range(B, P, d):
    """Anchors with a large feature against masked targets: the product, and products of the remainders of the two factors
    with either sign, are beyond 3.4e38."""
    q, p, r, out = masked_batch(B, P, d, 5300 + B)
    q[:, 3] = 1e3 * (1.0 + q[:, 3] * d)
    p[:, 3] = 1e-6
    p[out, 3] = -3e38
    want = oracle_loss(q, p, r, 1.0, 0.5)
    check_fp32_grade("overflow %dx%dx%d" % (B, P, d), run_ex(q.to(DEV), p.to(DEV), r.to(DEV), 1.0, 0.5), want, q, p, 2.0)


def test_replay_after_the_library_has_grown_its_buffer():
    """The graph of a captured call goes on using the buffer it has recorded."""
    import os
    import subprocess
    import sys
    root = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
    grow = """
gc.gc_loss_and_rep_grad_f32(mk(300, 200), mk(500, 200), r)     # wants a larger buffer
full = torch.full((1 << 24,), float("nan"), device="cuda")     # where memory that was given back would show
for k in range(3):"""
    code = (CAPTURE % root).replace("\nfor k in range(3):", grow)
    assert "wants a larger" in code
    r = subprocess.run([sys.executable, "-c", code], capture_output=True, text=True, timeout=100)
    assert r.returncode == 0 and "replays agree" in r.stdout, r.stdout + r.stderr


@pytest.mark.parametrize("kind,B,P,d,nbytes", SMALLER)
def test_smaller_workspaces(kind, B, P, d, nbytes):
    """What serves a call whose workspace is smaller than the named one, and nothing written behind it."""
    from oracle import gc_oracle as O
    buf = torch.full((nbytes + 8192,), 0xA5, dtype=torch.uint8, device=DEV)
    assert buf.data_ptr() % 256 == 0
    ws = buf[:nbytes]
    q, p, r = synth.dpr_batch(B, P, d, torch.float32 if kind == "f32" else torch.bfloat16, seed=5400 + d, positive_mix=0.3)
    tol = TOL_F32 if kind == "f32" or d % 128 or d > 768 else TOL_BF16
    label = "%s %dx%dx%d in %d" % (kind, B, P, d, nbytes)
    if kind == "ntxent":
        z = synth.ntxent_views(B, d, seed=5400)
        want = oracle_loss(z, z, torch.arange(B, dtype=torch.int32) ^ 1, 1.0, 0.2, mask_self=True)
        want["dz"] = want["dq"] + want["dp"]
        loss, dz = gc.gc_ntxent_loss_and_grad_bf16(z.to(DEV), 0.2, ws)
        got = dict(loss=loss, dz=dz)
    elif kind == "symmetric":
        r = torch.from_numpy(np.random.default_rng(B).permutation(B).astype(np.int32))
        want = O.bidirectional(synth.widen(q), synth.widen(p), r.numpy(), 1.0, 0.5)
        got = gc.gc_bidirectional_loss_and_rep_grad_bf16(q.to(DEV), p.to(DEV), r.to(DEV), 1.0, 0.5, ws)
    elif kind == "bilinear":
        om = (torch.eye(d) + 0.5 * torch.randn(d, d, generator=torch.Generator().manual_seed(d)) * d ** -0.5).to(torch.bfloat16)
        whole = gc.gc_bilinear_loss_and_grads_bf16(q.to(DEV), p.to(DEV), r.to(DEV), om.to(DEV), 1.0, 0.5)
        got = gc.gc_bilinear_loss_and_grads_bf16(q.to(DEV), p.to(DEV), r.to(DEV), om.to(DEV), 1.0, 0.5, ws)
        want = {k: to_np(whole[k]) for k in ("loss", "u", "v", "domega")}   # (that one is held to the oracle elsewhere)
        want["loss"] = want["loss"][0]
    else:
        want = oracle_loss(q, p, r, 1.0, 0.5)
        got = gc.gc_loss_and_rep_grad_ex(q.to(DEV), p.to(DEV), r.to(DEV), 1.0, 0.5, 0, ("loss", "dq", "dp", "lse"), ws)
    torch.cuda.synchronize()
    check_loss(label + " loss", got["loss"].item(), want["loss"], tol)
    for k in ("dq", "dp", "dz", "lse", "u", "v", "domega"):
        if k in got and k in want:
            check(label + " " + k, relerr(to_np(got[k]), want[k]), tol)
    assert bool((buf[nbytes:] == 0xA5).all())


@pytest.mark.parametrize("rows", ["within", "one anchor", "one target", "every row"])
@pytest.mark.parametrize("B,P", [(33, 70), (200, 330)])
def test_deep_distance_where_the_powers_end(B, P, rows):
    """Scaled pre-activations up to the largest whose powers of two are normal numbers (126), and beyond on one anchor, one
    target or everywhere: workgroups that multiply powers beside workgroups that exponentiate sums.  Bound as above."""
    from oracle import gc_oracle as O
    d = 128
    q, p, _ = synth.dpr_batch(B, P, d, torch.float32, seed=5500 + B)
    om = synth.deep_omega(d)
    om["C"] = om["A"].clone()
    r = torch.from_numpy(np.random.default_rng(B).integers(0, P, size=B).astype(np.int32))
    scaled = lambda x: np.abs(synth.widen(x.to(torch.bfloat16)) @ synth.widen(om["A"]).T).max(axis=1) * 2 / np.log(2.0)  # noqa: E731
    q *= torch.from_numpy(100.0 / scaled(q)).float()[:, None]      # every row: largest entry 100 (bf16: within half a percent)
    p *= torch.from_numpy(100.0 / scaled(p)).float()[:, None]
    if rows == "one anchor":
        q[B - 2] *= 1.8
    if rows == "one target":
        p[P - 3] *= 1.8
    if rows == "every row":
        q *= 1.4
        p *= 1.4
    p[40] = -q[3]
    p[P - 1] = -q[B - 2]
    q, p = q.to(torch.bfloat16), p.to(torch.bfloat16)
    assert (max(scaled(q).max(), scaled(p).max()) < 126.0) == (rows == "within")
    om64 = {k: synth.widen(v) for k, v in om.items()}
    want = O.deep_distance(synth.widen(q), synth.widen(p), synth.widen(r), om64, 1.0, 0.5)
    out = gc.gc_deepdist_loss_and_grads_bf16(q.to(DEV), p.to(DEV), r.to(DEV), {k: v.to(DEV) for k, v in om.items()}, 1.0, 0.5)
    torch.cuda.synchronize()
    check_loss("deep %s loss" % rows, out["loss"].item(), want["loss"], 1e-4)
    for k in ("u", "v", "dA", "dC", "dw"):
        check("deep %s %dx%d %s" % (rows, B, P, k), relerr(to_np(out[k]), want[k]), 1e-4)


@pytest.mark.parametrize("dtype", [torch.float32, torch.bfloat16])
def test_few_scores_with_64_owner_rows(dtype):
    """A few anchors against so many targets that a workgroup owns 64 rows: the statistics of few scores, merged by a launch."""
    q, p, r = synth.dpr_batch(3, 100000, 24, dtype, seed=5500)
    want = oracle_loss(q, p, r, 1.0, 0.25)
    check_fp32_grade("3x100000x24 %s" % dtype, run_ex(q.to(DEV), p.to(DEV), r.to(DEV), 1.0, 0.25), want, q, p, 4.0)


@pytest.mark.parametrize("B,P,d,dtype", [(3000, 3100, 500, torch.float32), (3000, 3000, 768, torch.float32), (2800, 3000, 1000, torch.float32),
                                         (3000, 3100, 500, torch.bfloat16), (3000, 3000, 700, torch.bfloat16), (3000, 3000, 1000, torch.bfloat16),
                                         (2000, 2100, 1300, torch.bfloat16)])
def test_large_batches_of_larger_widths(B, P, d, dtype):
    """64 owner rows per workgroup with four, six and eight column tiles per wave, of which owner rows are staged in part; the
    larger statistics kernel with owner rows beyond what it stages (from 24 k-steps of fp32, 76 of bf16 on)."""
    q, p, r = synth.dpr_batch(B, P, d, dtype, seed=5600 + d, positive_mix=0.3)
    want = oracle_loss(q, p, r, 1.0, 0.25)
    check_fp32_grade("%dx%dx%d %s" % (B, P, d, dtype), run_ex(q.to(DEV), p.to(DEV), r.to(DEV), 1.0, 0.25), want, q, p, 4.0)


@pytest.mark.parametrize("n,d", [(1200, 130), (3000, 200)])
def test_masked_ntxent_and_symmetric_above_the_few_scores(n, d):
    """The larger statistics kernel, and the gradients with 32 and 64 owner rows per workgroup, with the diagonal masked."""
    from oracle import gc_oracle as O
    q, p, _ = synth.dpr_batch(n, n, d, torch.float32, seed=5700 + n, positive_mix=0.2)
    r = torch.arange(n, dtype=torch.int32) ^ 1
    want = oracle_loss(q, p, r, 1.0, 0.5, mask_self=True)
    check_fp32_grade("mask n=%d d=%d" % (n, d), run_ex(q.to(DEV), p.to(DEV), r.to(DEV), 1.0, 0.5, gc.GC_MASK_SELF), want, q, p, 2.0)
    z = synth.ntxent_views(n, d, seed=5710)
    want = oracle_loss(z, z, r, 1.0, 0.2, mask_self=True)
    loss, dz = gc.gc_ntxent_loss_and_grad_bf16(z.to(DEV), 0.2)
    torch.cuda.synchronize()
    check_loss("ntxent n=%d d=%d" % (n, d), loss.item(), want["loss"], TOL_F32)
    check("ntxent n=%d d=%d dz" % (n, d), relerr(to_np(dz), want["dq"] + want["dp"]), TOL_F32)
    q, p = q.to(torch.bfloat16), p.to(torch.bfloat16)
    perm = torch.from_numpy(np.random.default_rng(n).permutation(n).astype(np.int32))
    want = O.bidirectional(synth.widen(q), synth.widen(p), perm.numpy(), 1.0, 0.5)
    out = gc.gc_bidirectional_loss_and_rep_grad_bf16(q.to(DEV), p.to(DEV), perm.to(DEV), 1.0, 0.5)
    torch.cuda.synchronize()
    check_loss("symmetric n=%d d=%d" % (n, d), out["loss"].item(), want["loss"], TOL_F32)
    for k in ("dq", "dp"):
        check("symmetric n=%d d=%d %s" % (n, d, k), relerr(to_np(out[k]), want[k]), TOL_F32)


@pytest.mark.parametrize("dtype", [torch.float32, torch.bfloat16])
@pytest.mark.parametrize("B,P,d", [(64, 100, 200), (512, 1024, 776), (1500, 1600, 200), (2100, 2200, 96)])
def test_gradients_where_the_softmax_has_converged(B, P, d, dtype):
    """Aligned positives at temperature 0.1: p - 1 of the positive is the small difference of 2^(t - lse2) and 1.  t is part
    of lse2, so that the rounding of its sum cancels: what is left is that of lse2 (half a unit in its last place, another
    half for log2 and the sum) and of the exponential, times the largest entry of the row it multiplies."""
    g = torch.Generator().manual_seed(5800 + B)
    q = torch.nn.functional.normalize(torch.randn(B, d, generator=g), dim=1)
    p = torch.nn.functional.normalize(torch.randn(P, d, generator=g), dim=1)
    r = torch.randperm(P, generator=g)[:B]
    p[r] = torch.nn.functional.normalize(0.9 * q + 0.1 * p[r], dim=1)
    q, p, r = q.to(dtype), p.to(dtype), r.to(torch.int32)
    alpha = 10.0
    want = oracle_loss(q, p, r, 1.0, 1.0 / alpha)
    out = run_ex(q.to(DEV), p.to(DEV), r.to(DEV), 1.0, 1.0 / alpha)
    lse2 = np.abs(want["lse"]).max() / np.log(2.0)
    coeff = np.log(2.0) * 2.0 ** (np.floor(np.log2(lse2)) - 23) + 2.0 ** -23
    for k, other in (("dq", p), ("dp", q)):
        err = np.abs(to_np(out[k]) - want[k]).max()
        bound = alpha / B * coeff * float(other.float().abs().max()) + 2e-6 * np.abs(want[k]).max()
        check("converged %dx%dx%d %s %s" % (B, P, d, dtype, k), err, bound)


@pytest.mark.parametrize("dtype", [torch.float32, torch.bfloat16])
@pytest.mark.parametrize("B,P,d,masked", [(129, 200, 520, False), (33, 31, 700, False), (640, 640, 776, True), (300, 500, 1030, False),
                                          (1030, 1100, 1000, False), (257, 129, 1300, False)])
def test_scores_in_halves_of_the_width(B, P, d, masked, dtype):
    """More than 512 columns of 32 owner rows: eight waves, of which two share a score (of fp32 owner rows LDS holds 40 k-steps)."""
    q, p, r = synth.dpr_batch(B, P, d, dtype, seed=5900 + d, positive_mix=0.3)
    if masked:
        r = torch.arange(B, dtype=torch.int32) ^ 1
    want = oracle_loss(q, p, r, 1.0, 0.25, mask_self=masked)
    got = run_ex(q.to(DEV), p.to(DEV), r.to(DEV), 1.0, 0.25, *([gc.GC_MASK_SELF] if masked else []))
    check_fp32_grade("%dx%dx%d %s" % (B, P, d, dtype), got, want, q, p, 4.0)


@pytest.mark.parametrize("dtype", [torch.float32, torch.bfloat16])
@pytest.mark.parametrize("B,P,d,masked", [(33, 31, 776, False), (1, 300, 300, False), (300, 1, 520, False), (129, 257, 129, False),
                                          (129, 257, 257, False), (512, 512, 400, True), (70, 9000, 300, False), (9000, 70, 520, False),
                                          (200, 300, 2100, False), (1000, 1040, 1000, False)])
def test_few_scores_of_general_widths(B, P, d, masked, dtype):
    """Few scores in the named workspace and in one a little smaller (fewer splits, packed for the same kernels or not at all): one
    answer; and one gradient alone."""
    q, p, r = synth.dpr_batch(B, P, d, dtype, seed=6000 + d, positive_mix=0.3)
    if masked:
        r = torch.arange(B, dtype=torch.int32) ^ 1
    want = oracle_loss(q, p, r, 1.0, 0.25, mask_self=masked)
    flags = gc.GC_MASK_SELF if masked else 0
    dev = [x.to(DEV) for x in (q, p, r)]
    out = run_ex(*dev, 1.0, 0.25, flags)
    check_fp32_grade("%dx%dx%d %s" % (B, P, d, dtype), out, want, q, p, 4.0)
    need = gc.load().gc_workspace_bytes(B, P, d, gc.GC_F32 if dtype == torch.float32 else gc.GC_BF16)
    less = gc.gc_loss_and_rep_grad_ex(*dev, 1.0, 0.25, flags, workspace=gc.alloc_workspace(need - 4096, DEV))
    torch.cuda.synchronize()
    check_fp32_grade("... less workspace", less, want, q, p, 4.0)
    for k in ("dq", "dp"):
        one = gc.gc_loss_and_rep_grad_ex(*dev, 1.0, 0.25, flags, want=("loss", k))
        torch.cuda.synchronize()
        check_loss("... %s alone, loss" % k, one["loss"].item(), want["loss"], TOL_F32, 1e-30)
        check("... %s alone" % k, relerr(to_np(one[k]), want[k]), TOL_F32)


@pytest.mark.parametrize("B,P,d,masked", [(1, 1, 256, False), (33, 31, 768, False), (1, 300, 256, False), (300, 1, 640, False), (129, 257, 384, False),
                                          (512, 512, 768, True), (70, 9000, 512, False), (9000, 70, 768, False), (1000, 1040, 256, False),
                                          (1021, 1000, 640, False), (97, 4000, 768, False), (4000, 97, 384, False)])
def test_walks_of_few_scores(B, P, d, masked):
    """bf16, widths that are multiples of 128: in the named workspace and in one a little smaller (fewer splits), merged inside the
    gradient kernel or by a launch (many rows); and one gradient alone."""
    q, p, r = synth.dpr_batch(B, P, d, torch.bfloat16, seed=6100 + d + B, positive_mix=0.3)
    if masked:
        r = torch.arange(B, dtype=torch.int32) ^ 1
    want = oracle_loss(q, p, r, 1.0, 0.25, mask_self=masked)
    flags = gc.GC_MASK_SELF if masked else 0
    dev = [x.to(DEV) for x in (q, p, r)]
    need = gc.load().gc_workspace_bytes(B, P, d, gc.GC_BF16)
    for label, n, want_ in (("named workspace", need, None), ("less workspace", need - 4096, None), ("dq alone", need, ("loss", "dq")), ("dp alone", need, ("loss", "dp"))):
        kw = dict(want=want_) if want_ else {}
        if n < need and (B, P) in ((1, 1), (1000, 1040)):   # the named one is the least there is
            with pytest.raises(gc.GradCacheError):
                gc.gc_loss_and_rep_grad_ex(*dev, 1.0, 0.25, flags, workspace=gc.alloc_workspace(n, DEV))
            continue
        out = gc.gc_loss_and_rep_grad_ex(*dev, 1.0, 0.25, flags, workspace=gc.alloc_workspace(n, DEV), **kw)
        torch.cuda.synchronize()
        check_loss("few %s loss" % label, out["loss"].item(), want["loss"], TOL_F32, 1e-30)
        for k in ("dq", "dp"):
            if not want_ or k in want_:
                # With one target the softmax is 1 and the gradients are 0: what is left is the rounding of the positive's
                # coefficient 2^(t - lse2) - 1, by ulp(t) + ulp(lse2) <= 2^-22 |t|, times a row of the other side and alpha / B.
                other, t = (p if k == "dq" else q), 4.0 * np.log2(np.e) * np.abs(synth.widen(q) @ synth.widen(p).T).max()
                floor = 4.0 / B * float(other.float().abs().max()) * 2.0 ** -22 * (1.0 + t) * (B if k == "dp" else 1)
                err = np.abs(to_np(out[k]) - want[k]).max()
                check("few %dx%dx%d %s %s" % (B, P, d, label, k), err, TOL_BF16 * np.abs(want[k]).max() + floor)


@pytest.mark.parametrize("dtype,d", [(torch.bfloat16, 256), (torch.bfloat16, 768), (torch.float32, 300), (torch.float32, 768), (torch.bfloat16, 520), (torch.bfloat16, 1000)])
def test_no_scores_in_memory(dtype, d):
    """s_ij = 256 i + j, exact in either type and no two alike: after a call next to none of them, scaled or not, lies in the workspace
    (of the row statistics, the positives and the row maxima may)."""
    B, P = 128, 256
    q, p = torch.zeros(B, d), torch.zeros(P, d)
    q[:, 0], q[:, 1] = 256.0 * torch.arange(B), 1.0
    p[:, 0], p[:, 1] = 1.0, torch.arange(P).float()
    temp = 4096.0
    ws = gc.alloc_workspace(gc.load().gc_workspace_bytes(B, P, d, gc.GC_F32 if dtype == torch.float32 else gc.GC_BF16), DEV)
    ws.zero_()
    r = torch.arange(B, dtype=torch.int32)
    gc.gc_loss_and_rep_grad_ex(q.to(dtype).to(DEV), p.to(dtype).to(DEV), r.to(DEV), 1.0, temp, 0, workspace=ws)
    torch.cuda.synchronize()
    words = np.unique(ws.cpu().numpy()[:ws.numel() // 4 * 4].view(np.float32))
    words = words[np.isfinite(words)].astype(np.float64)
    scores = np.arange(1, B * P, dtype=np.float64)
    for mul in (1.0, 1.0 / temp, np.log2(np.e) / temp):
        at = np.clip(np.searchsorted(words, scores * mul), 1, len(words) - 1)
        near = np.minimum(np.abs(words[at] - scores * mul), np.abs(words[at - 1] - scores * mul))
        check("scores in memory (x %.1e)" % mul, float((near <= 2.0 ** -23 * scores * mul).mean()), 4 * (B + P) / (B * P))
