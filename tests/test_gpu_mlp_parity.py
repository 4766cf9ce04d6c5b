"""GPU parity of the stand-in encoder steps (graph-less forward, chunk surrogate
backward, whole Gradient Cache step) against the fp64 oracle."""
import math

import numpy as np
import pytest
import torch

from oracle import gc_oracle as O
from paper_2101_06983_amd import binding as gc
from paper_2101_06983_amd import synth
from parity import TOL_BF16, check, check_loss, relerr, to_np

pytestmark = pytest.mark.gpu
DEV = "cuda:0"
# A value stored in bf16 may land on the neighbouring bf16 number on the two sides: one ulp (2^-8)
# of the largest entry on top of the arithmetic tolerance.
TOL_STORED = TOL_BF16 + 2.0 ** -8
# End to end (Steps 1-3) the representations the loss sees are such stored values, so the scores of
# the two sides differ by more than arithmetic error alone.  Every stage is therefore held to TOL_BF16 on
# its own, AT FULL SIZE, by giving the oracle what the GPU's previous stage stored (stagewise() below);
# the chained result (oracle end to end against GPU end to end) is an extra, held to three times that:
# the only place in this suite where a bound wider than the stated tolerance remains.
TOL_CHAIN = 3 * TOL_BF16


def widen_params(params):
    return {k: synth.widen(v) for k, v in params.items()}


def dev_params(params):
    return {k: v.to(DEV) for k, v in params.items()}


def stagewise(label, out, xq, xp, r, params, cq, cp, scale=1.0, temp=1.0):
    """Steps 2 and 3 each against the oracle on the GPU's own stored inputs of that step (Step 1 is compared
    directly: its inputs are the caller's).  Step 2 (Eq. 1, 4-7): the oracle on the returned bf16 representations
    widened exactly, against the returned loss and cache.  Step 3 (Eq. 8-9): the oracle's per-sub-batch backward of
    the returned cache rows (fp32 widened exactly), summed over the sub-batches in index order, against the
    returned parameter gradients."""
    p64 = widen_params(params)
    want_q, want_p = O.mlp_forward(synth.widen(xq), p64), O.mlp_forward(synth.widen(xp), p64)
    check(label + " step1 q", relerr(to_np(out["q"]), want_q), TOL_STORED)
    check(label + " step1 p", relerr(to_np(out["p"]), want_p), TOL_STORED)
    s2 = O.loss_and_rep_grad(to_np(out["q"]), to_np(out["p"]), synth.widen(r), scale, temp)
    check_loss(label + " step2 loss", out["loss"].item(), s2["loss"], TOL_BF16)
    check(label + " step2 dq", relerr(to_np(out["dq"]), s2["dq"]), TOL_BF16)
    check(label + " step2 dp", relerr(to_np(out["dp"]), s2["dp"]), TOL_BF16)
    u, v = to_np(out["dq"]), to_np(out["dp"])
    x_q, x_p = synth.widen(xq), synth.widen(xp)
    acc = {k: 0.0 for k in ("W1", "b1", "W2", "b2")}
    for x, up, c in ((x_q, u, cq), (x_p, v, cp)):
        for a in range(0, len(x), c):
            g = O.mlp_backward(x[a:a + c], p64, up[a:a + c])
            for k in acc:
                acc[k] = acc[k] + g[k]
    for k in ("W1", "b1", "W2", "b2"):
        check(label + " step3 d" + k, relerr(to_np(out["grads"][k]), acc[k]), TOL_BF16)


def small_problem(B=48, P=96, din=128, dh=256, dout=128, seed=9):
    return synth.mlp_problem(B, P, din, dh, dout, seed=synth.SEED0 + seed)


# (from 128 rows on the forward runs as tiled GEMMs: whole tiles, ragged last tiles, one- and two-step contractions)
@pytest.mark.parametrize("rows,din,dh", [(1, 128, 256), (32, 128, 256), (40, 128, 256), (100, 128, 256), (128, 128, 256),
                                         (200, 128, 256), (1000, 128, 256), (130, 64, 128), (333, 192, 384)])
def test_forward_nograd(rows, din, dh):
    xq, _, _, params = small_problem(B=rows, din=din, dh=dh)
    want = O.mlp_forward(synth.widen(xq), widen_params(params))
    y = gc.gc_mlp_forward_nograd_bf16(xq.to(DEV), dev_params(params))
    torch.cuda.synchronize()
    check("forward rows=%d din=%d dh=%d" % (rows, din, dh), relerr(to_np(y), want), TOL_STORED)


@pytest.mark.parametrize("rows", [1, 16, 32, 45])
def test_chunk_surrogate_backward(rows):
    xq, _, _, params = small_problem(B=rows)
    g = np.random.default_rng(rows)
    u = torch.from_numpy((g.standard_normal((rows, 128)) * 1e-3).astype(np.float32))
    want = O.mlp_backward(synth.widen(xq), widen_params(params), synth.widen(u))
    dp = dev_params(params)
    grads = gc.zero_mlp_grads(dp)
    gc.gc_chunk_surrogate_backward_bf16(xq.to(DEV), dp, u.to(DEV), grads)
    torch.cuda.synchronize()
    for k in ("W1", "b1", "W2", "b2"):
        check("chunk backward rows=%d d%s" % (rows, k), relerr(to_np(grads[k]), want[k]), TOL_BF16)
    # accumulation (+=): a second call doubles the sums
    gc.gc_chunk_surrogate_backward_bf16(xq.to(DEV), dp, u.to(DEV), grads)
    torch.cuda.synchronize()
    for k in ("W1", "b1", "W2", "b2"):
        check("chunk backward twice rows=%d d%s" % (rows, k), relerr(to_np(grads[k]), 2 * want[k]), TOL_BF16)


@pytest.mark.parametrize("cq,cp", [(16, 16), (32, 32), (7, 24), (48, 96)])
def test_step_small_matches_fullbatch_oracle(cq, cp):
    xq, xp, r, params = small_problem()
    # the workload stores representations in bf16: the oracle rounds F, G the same way before Step 2
    want = O.mlp_fullbatch_grad(synth.widen(xq), synth.widen(xp), synth.widen(r), widen_params(params), 1.0, 0.05,
                                rep_dtype="bf16")
    out = gc.gc_step_mlp_bf16(xq.to(DEV), xp.to(DEV), r.to(DEV), cq, cp, dev_params(params), 1.0, 0.05, keep=True)
    torch.cuda.synchronize()
    stagewise("small step %d/%d" % (cq, cp), out, xq, xp, r, params, cq, cp, 1.0, 0.05)
    # extra: the chained result, oracle end to end
    check_loss("small step chained loss", out["loss"].item(), want["loss"], TOL_BF16)
    check("small step chained dq", relerr(to_np(out["dq"]), want["dq"]), TOL_CHAIN)
    check("small step chained dp", relerr(to_np(out["dp"]), want["dp"]), TOL_CHAIN)
    for k in ("W1", "b1", "W2", "b2"):
        check("small step chained d" + k, relerr(to_np(out["grads"][k]), want["grads"][k]), TOL_CHAIN)


def test_chunking_does_not_change_the_update():
    # the method's exactness claim (Sec. "Gradient Cache Technique", Step 3): any sub-batching gives the
    # full-batch gradient; on the GPU only the fp32 summation order differs
    xq, xp, r, params = small_problem()
    dp = dev_params(params)
    a = gc.gc_step_mlp_bf16(xq.to(DEV), xp.to(DEV), r.to(DEV), 48, 96, dp, 1.0, 0.05)
    b = gc.gc_step_mlp_bf16(xq.to(DEV), xp.to(DEV), r.to(DEV), 16, 8, dp, 1.0, 0.05)
    c = gc.gc_step_mlp_bf16(xq.to(DEV), xp.to(DEV), r.to(DEV), 16, 8, dp, 1.0, 0.05)
    torch.cuda.synchronize()
    assert a["loss"].item() == b["loss"].item()
    for k in ("W1", "b1", "W2", "b2"):
        assert relerr(to_np(b["grads"][k]), to_np(a["grads"][k])) <= 1e-5, k
        assert torch.equal(b["grads"][k], c["grads"][k]), k      # run-to-run reproducible


@pytest.mark.parametrize("B,P", [(100, 300), (130, 200)])
def test_step_with_the_tiled_forward(B, P):
    # (100, 300): B below and P above the row count from which the graph-less forward runs as tiled GEMMs (split
    # contraction in the second layer): both forward paths in one step.  (130, 200): both sides tiled and in the same
    # launches, a tile straddling the two inputs.  Ragged last sub-batches, and the same update for another chunking.
    xq, xp, r, params = small_problem(B=B, P=P, din=192, dh=384, dout=128, seed=11)
    dp = dev_params(params)
    out = gc.gc_step_mlp_bf16(xq.to(DEV), xp.to(DEV), r.to(DEV), 32, 64, dp, 1.0, 0.05, keep=True)
    torch.cuda.synchronize()
    stagewise("tiled step %d/%d 32/64" % (B, P), out, xq, xp, r, params, 32, 64, 1.0, 0.05)
    other = gc.gc_step_mlp_bf16(xq.to(DEV), xp.to(DEV), r.to(DEV), 24, 40, dp, 1.0, 0.05, keep=True)
    torch.cuda.synchronize()
    assert torch.equal(out["q"], other["q"]) and torch.equal(out["p"], other["p"])   # Step 1 does not depend on the chunking
    assert out["loss"].item() == other["loss"].item()
    for k in ("W1", "b1", "W2", "b2"):
        assert relerr(to_np(other["grads"][k]), to_np(out["grads"][k])) <= 1e-5, k


def test_step_with_a_large_batch_takes_the_online_walk():
    """B = P = 4096 with a small encoder (64-128-768): 2^24 scores, so Step 2 runs without a statistics pass; the
    parameter gradients still equal the full-batch ones."""
    xq, xp, r, params = synth.mlp_problem(B=4096, P=4096, din=64, dh=128, dout=768, seed=synth.SEED0 + 50)
    want = O.mlp_fullbatch_grad(synth.widen(xq), synth.widen(xp), synth.widen(r), widen_params(params), 1.0, 0.2,
                                rep_dtype="bf16")
    out = gc.gc_step_mlp_bf16(xq.to(DEV), xp.to(DEV), r.to(DEV), 256, 512, dev_params(params), 1.0, 0.2, keep=True)
    torch.cuda.synchronize()
    # every stage against the oracle on what the previous stage stored, at the stated tolerance
    stagewise("4096x4096 step", out, xq, xp, r, params, 256, 512, 1.0, 0.2)
    # extra: the chained result (oracle end to end).  A parameter gradient here is a sum over 8192 rows whose terms
    # largely cancel (the cached gradients of a batch sum to about zero: invariant I1), so its size is that of a few
    # terms while every row brings the difference of the two sides' stored representations: twice the chained bound
    check_loss("4096x4096 chained loss", out["loss"].item(), want["loss"], TOL_BF16)
    check("4096x4096 chained dq", relerr(to_np(out["dq"]), want["dq"]), TOL_CHAIN)
    check("4096x4096 chained dp", relerr(to_np(out["dp"]), want["dp"]), TOL_CHAIN)
    for k in ("W1", "b1", "W2"):
        check("4096x4096 chained d" + k, relerr(to_np(out["grads"][k]), want["grads"][k]), 2 * TOL_CHAIN)
    # db2 is the plain sum of all 8192 cached rows, of which the 4096 target rows sum to exactly zero in exact
    # arithmetic (I1): what is left is small against the terms, while the differences of the rows add like a
    # random walk.  Held to that: sqrt(rows) times the chained-tolerance error of one row (as for the other sums: twice).
    rows = 4096 + 4096
    row_scale = max(np.abs(want["dq"]).max(), np.abs(want["dp"]).max())
    check("4096x4096 chained db2 (absolute)", np.abs(to_np(out["grads"]["b2"]) - want["grads"]["b2"]).max(),
          2 * TOL_CHAIN * math.sqrt(rows) * row_scale)


def test_config5_full_size():
    xq, xp, r, params = synth.mlp_problem()
    want = O.mlp_chunked_grad(synth.widen(xq), synth.widen(xp), synth.widen(r), widen_params(params), 32, 32,
                              rep_dtype="bf16")
    out = gc.gc_step_mlp_bf16(xq.to(DEV), xp.to(DEV), r.to(DEV), 32, 32, dev_params(params), keep=True)
    torch.cuda.synchronize()
    # Steps 1, 2, 3 each at the stated tolerance: 48 sub-batches of 32 rows, every parameter gradient (Eq. 8-9)
    stagewise("config5", out, xq, xp, r, params, 32, 32)
    # extra: the chained result against the oracle's own Steps 1-3
    check_loss("config5 chained loss", out["loss"].item(), want["loss"], TOL_BF16)
    check("config5 chained dq", relerr(to_np(out["dq"]), want["dq"]), TOL_CHAIN)
    check("config5 chained dp", relerr(to_np(out["dp"]), want["dp"]), TOL_CHAIN)
    for k in ("W1", "b1", "W2", "b2"):
        check("config5 chained d" + k, relerr(to_np(out["grads"][k]), want["grads"][k]), TOL_CHAIN)
    # Step 3 runs as a software pipeline over the sub-batches: the accumulation order must not depend on timing
    again = gc.gc_step_mlp_bf16(xq.to(DEV), xp.to(DEV), r.to(DEV), 32, 32, dev_params(params), keep=True)
    torch.cuda.synchronize()
    for k in ("W1", "b1", "W2", "b2"):
        assert torch.equal(out["grads"][k], again["grads"][k]), k
    assert torch.equal(out["q"], again["q"]) and torch.equal(out["dp"], again["dp"])


@pytest.mark.parametrize("B,P,cq,cp,group", [(200, 330, 32, 64, 3), (96, 96, 16, 32, 8)])
def test_accumulate_group_is_accepted_and_changes_nothing(B, P, cq, cp, group):
    """Step 3 takes as many whole sub-batches at a time as the activation buffer of Step 1 holds, whatever the argument says."""
    xq, xp, r, params = synth.mlp_problem(B, P, 128, 256, 128, seed=synth.SEED0 + 70 + B)
    dp = dev_params(params)
    one = gc.gc_step_mlp_bf16(xq.to(DEV), xp.to(DEV), r.to(DEV), cq, cp, dp, keep=True)
    grp = gc.gc_step_mlp_bf16(xq.to(DEV), xp.to(DEV), r.to(DEV), cq, cp, dp, keep=True, accumulate_group=group)
    torch.cuda.synchronize()
    assert torch.equal(one["loss"], grp["loss"]) and float(one["grads"]["W1"].abs().max()) > 0
    for k in ("W1", "b1", "W2", "b2"):
        assert torch.equal(one["grads"][k], grp["grads"][k]), k


@pytest.mark.parametrize("B,P,dh,chunks", [(300, 4200, 128, [(24, 48), (500, 33), (300, 4200)]), (4200, 300, 256, [(48, 24), (2100, 64)]),
                                           (700, 1300, 4096, [(64, 64)])])
def test_step3_in_several_runs(B, P, dh, chunks):
    """A side above what the activation buffer holds (2048 rows, or 8 sub-batches) goes through Step 3 in runs that add to
    the gradients of the earlier ones: three and two runs of one side by the sub-batch size, one run with a single
    sub-batch; both sides in one run with the 128-row tiles (the last shape).  Gradients are added to what is there."""
    xq, xp, r, params = synth.mlp_problem(B, P, 64, dh, 128, seed=synth.SEED0 + 80 + dh)
    dp = dev_params(params)
    start = 2.0 ** -7
    first = None
    for cq, cp in chunks:
        grads = {k: torch.full(v.shape, start, dtype=torch.float32, device=DEV) for k, v in params.items()}
        out = gc.gc_step_mlp_bf16(xq.to(DEV), xp.to(DEV), r.to(DEV), cq, cp, dp, 1.0, 0.2, grads=grads, keep=True)
        torch.cuda.synchronize()
        for k in grads:
            grads[k] -= start
        stagewise("%dx%d step in %d/%d" % (B, P, cq, cp), out, xq, xp, r, params, cq, cp, 1.0, 0.2)
        if first is None:
            first = out
        for k in ("q", "p", "dq", "dp"):   # nothing before Step 3 depends on the sub-batches
            assert torch.equal(out[k], first[k]), k
        for k in grads:   # the same terms in the same order but for where a run ends: fp32 rounding of the sums
            check("%dx%d d%s, %d/%d" % (B, P, k, cq, cp), relerr(to_np(grads[k]), to_np(first["grads"][k])), 1e-5 + 2.0 ** -31 / float(grads[k].abs().max()))


def test_step_replayed_with_the_same_buffers_matches_the_first_call():
    # a call that repeats with the same buffers is recorded into a graph and replayed: every replay must
    # give the bits of the directly enqueued first call, with other GPU work in between
    xq, xp, r, params = small_problem()
    dp = dev_params(params)
    xq, xp, r = xq.to(DEV), xp.to(DEV), r.to(DEV)
    first = gc.gc_step_mlp_bf16(xq, xp, r, 16, 32, dp, 1.0, 0.05, keep=True)
    torch.cuda.synchronize()
    ref = {k: first["grads"][k].clone() for k in first["grads"]}
    ref_loss, ref_dq = first["loss"].clone(), first["dq"].clone()
    for rep in range(4):
        for k in first["grads"]:
            first["grads"][k].zero_()
        first["dq"].fill_(7.0)
        filler = torch.randn(1 << 20, device=DEV).sum()      # unrelated eager work between the replays
        out = gc.gc_step_mlp_bf16(xq, xp, r, 16, 32, dp, 1.0, 0.05, out=first)
        torch.cuda.synchronize()
        assert torch.isfinite(filler)
        assert torch.equal(out["loss"], ref_loss), rep
        assert torch.equal(out["dq"], ref_dq), rep
        for k in ref:
            assert torch.equal(out["grads"][k], ref[k]), (rep, k)


def test_step_with_a_workspace_that_leaves_the_loss_less_than_it_wants():
    """dout = 896 takes the loss kernels with packed inputs; without room for them the general kernels, in 0.1 MB."""
    import ctypes
    B, P, c = 300, 500, 32
    xq, xp, r, params = synth.mlp_problem(B, P, 64, 128, 896, seed=synth.SEED0 + 95)
    dp = dev_params(params)
    lib, w = gc.load(), gc.make_mlp_params(dp)
    named = lib.gc_step_mlp_workspace_bytes(B, P, c, c, ctypes.byref(w))
    nbytes = named - lib.gc_workspace_bytes(B, P, 896, gc.GC_BF16) + 120576   # row statistics
    buf = torch.full((nbytes + 8192,), 0xA5, dtype=torch.uint8, device=DEV)
    out = gc.gc_step_mlp_bf16(xq.to(DEV), xp.to(DEV), r.to(DEV), c, c, dp, 1.0, 0.2, keep=True, workspace=buf[:nbytes])
    torch.cuda.synchronize()
    stagewise("step in %d of %d" % (nbytes, named), out, xq, xp, r, params, c, c, 1.0, 0.2)
    assert bool((buf[nbytes:] == 0xA5).all())
    with pytest.raises(gc.GradCacheError):
        gc.gc_step_mlp_bf16(xq.to(DEV), xp.to(DEV), r.to(DEV), c, c, dp, 1.0, 0.2, workspace=buf[:nbytes - 256])


@pytest.mark.parametrize("rows,dh", [(33, 256), (200, 512), (200, 2048)])
def test_forward_in_the_bytes_it_uses(rows, dh):
    """The transposed weights and two activations (the second for the partial products of the narrow layer: all of it at
    dh = 512), nothing behind them."""
    xq, _, _, params = small_problem(B=rows, dh=dh)
    nbytes = (128 * dh + dh * 128) * 2 + 2 * rows * dh * 4
    buf = torch.full((nbytes + 8192,), 0xA5, dtype=torch.uint8, device=DEV)
    y = gc.gc_mlp_forward_nograd_bf16(xq.to(DEV), dev_params(params), workspace=buf[:nbytes])
    torch.cuda.synchronize()
    check("forward in %d bytes" % nbytes, relerr(to_np(y), O.mlp_forward(synth.widen(xq), widen_params(params))), TOL_STORED)
    assert bool((buf[nbytes:] == 0xA5).all())


@pytest.mark.parametrize("B,P,cq,cp", [(9, 2067, 190, 6), (2344, 31, 3, 110), (26, 2395, 85, 13)])
def test_step_with_sub_batches_that_fill_a_launch_differently(B, P, cq, cp):
    """The activation buffer holds whole sub-batches of the larger size: 1900, 1980 and 2040 rows here, where whole
    sub-batches of the other size come to 2046, 2046 and 2041.  Rows beyond the buffer would share memory with the partial
    products of the second layer."""
    xq, xp, r, params = synth.mlp_problem(B, P, 64, 512, 128, seed=synth.SEED0 + 96 + B)
    out = gc.gc_step_mlp_bf16(xq.to(DEV), xp.to(DEV), r.to(DEV), cq, cp, dev_params(params), 1.0, 0.2, keep=True)
    one = gc.gc_step_mlp_bf16(xq.to(DEV), xp.to(DEV), r.to(DEV), 32, 32, dev_params(params), 1.0, 0.2, keep=True)
    torch.cuda.synchronize()
    stagewise("%dx%d step in %d/%d" % (B, P, cq, cp), out, xq, xp, r, params, cq, cp, 1.0, 0.2)
    for k in ("q", "p", "dq", "dp", "loss"):
        assert torch.equal(out[k], one[k]), k


# The tiles of the encoder's products: 64 x 128 (few tiles), 128 x 128 (rows of 1000 at dh = 2176: 272 tiles of the first) and 128 x 192
# (1500 rows at dh = 3200, whose last tiles of columns and rows are part empty); one and several blocks of rows of the kernel for
# few rows and the line behind it; widths that leave half a tile of dW1 (din = 64, 192); the second layer in tiles of 128 x 128 (1024
# rows) and 128 x 192 (2040 rows, a full launch of Step 1) in three ranges.  Which kernels each size reaches is asserted on the host.
# The bound of the gradients: factors of two bf16 planes are off by up to 2^-17 of themselves, independently from term to term,
# so a sum is off by about that share of its size; largest of all entries over the largest entry: 2^-14.
@pytest.mark.parametrize("rows,din,dh,dout", [(31, 64, 128, 128), (64, 192, 384, 128), (65, 128, 256, 256), (129, 64, 128, 128),
                                              (192, 320, 256, 128), (193, 64, 384, 384), (255, 192, 1408, 256), (1000, 64, 2176, 128),
                                              (1500, 128, 3200, 128), (1024, 64, 3072, 768), (2040, 64, 3072, 768)])
def test_tiles_of_the_encoder(rows, din, dh, dout):
    xq, _, _, params = small_problem(B=rows, din=din, dh=dh, dout=dout)
    p64, dp = widen_params(params), dev_params(params)
    y = gc.gc_mlp_forward_nograd_bf16(xq.to(DEV), dp)
    g = np.random.default_rng(rows)
    u = torch.from_numpy((g.standard_normal((rows, dout)) * 1e-3).astype(np.float32))
    grads = gc.zero_mlp_grads(dp)
    gc.gc_chunk_surrogate_backward_bf16(xq.to(DEV), dp, u.to(DEV), grads)
    torch.cuda.synchronize()
    label = "tiles %dx%dx%dx%d " % (rows, din, dh, dout)
    check(label + "y", relerr(to_np(y), O.mlp_forward(synth.widen(xq), p64)), 2.0 ** -8)
    want = O.mlp_backward(synth.widen(xq), p64, synth.widen(u))
    for k in ("W1", "b1", "W2", "b2"):
        check(label + "d" + k, relerr(to_np(grads[k]), want[k]), 2.0 ** -14)


@pytest.mark.parametrize("B,P,dh", [(131, 190, 256), (517, 983, 3200)])
def test_two_inputs_in_the_tiles_of_the_encoder(B, P, dh):
    # the targets' rows begin at the next multiple of 32 behind the anchors', inside a tile
    xq, xp, r, params = small_problem(B=B, P=P, din=64, dh=dh, dout=128, seed=12)
    out = gc.gc_step_mlp_bf16(xq.to(DEV), xp.to(DEV), r.to(DEV), 32, 64, dev_params(params), 1.0, 0.2, keep=True)
    torch.cuda.synchronize()
    stagewise("tiles of two inputs %d/%d" % (B, P), out, xq, xp, r, params, 32, 64, 1.0, 0.2)


def test_gelu_far_out():
    # pre-activations from -60 to 60 and beyond: GELU(h) is h or 0 and its derivative 1 or 0, without a NaN
    rows, din, dh, dout = 40, 64, 128, 128
    params = dict(W1=torch.zeros(din, dh), b1=torch.linspace(-60.0, 60.0, dh), W2=torch.zeros(dh, dout), b2=torch.zeros(dout))
    params["b1"][0], params["b1"][-1] = -1e30, 1e30
    params["W2"][:, 0] = 1.0
    params["W2"][-1, 0] = 0.0
    params = {k: v.to(torch.bfloat16) for k, v in params.items()}
    for rows in (40, 300):
        x = torch.ones(rows, din).to(torch.bfloat16)
        y = gc.gc_mlp_forward_nograd_bf16(x.to(DEV), dev_params(params))
        u = torch.zeros(rows, dout)
        u[:, 0] = 1.0
        grads = gc.zero_mlp_grads(dev_params(params))
        gc.gc_chunk_surrogate_backward_bf16(x.to(DEV), dev_params(params), u.to(DEV), grads)
        torch.cuda.synchronize()
        check("gelu far out rows=%d y" % rows, relerr(to_np(y), O.mlp_forward(synth.widen(x), widen_params(params))), 2.0 ** -8)
        h = synth.widen(params["b1"])
        phi = np.array([0.5 * math.erfc(-t / math.sqrt(2.0)) for t in h])
        prime = phi + h * np.exp(-0.5 * np.minimum(h * h, 1e4)) / math.sqrt(2 * math.pi)
        check("gelu far out rows=%d db1" % rows, relerr(to_np(grads["b1"]), rows * prime * synth.widen(params["W2"])[:, 0]), 2.0 ** -14)


@pytest.mark.parametrize("rows", [1, 40, 300])
@pytest.mark.parametrize("sd", [0.1, 0.3, 1.0, 3.0])
def test_gelu_in_fp32(rows, sd):
    """db1 is GELU'(h) in fp32 where one row has dA = 1, dW2 GELU(h) in two bf16 planes; h = b1 + W1[0], two bf16 numbers.  GELU' is two
    or three values below 1 added up: each rounding up to 2^-25 off, 2^-25 / sqrt 3 in the mean, so 2^-25 root mean square."""
    din, dh, dout = 64, 8192, 128
    g = np.random.default_rng(int(100 * sd))
    params = dict(W1=torch.zeros(din, dh), b1=torch.from_numpy(g.standard_normal(dh) * sd), W2=torch.zeros(dh, dout), b2=torch.zeros(dout))
    params["W1"][0] = torch.from_numpy(g.standard_normal(dh) * sd / 512)
    params["W2"][:, 0] = 1.0
    params = {k: v.to(torch.bfloat16) for k, v in params.items()}
    x = torch.zeros(rows, din, dtype=torch.bfloat16)
    x[:, 0] = 1.0
    u = torch.zeros(rows, dout)
    u[0, 0] = 1.0
    grads = gc.zero_mlp_grads(dev_params(params))
    gc.gc_chunk_surrogate_backward_bf16(x.to(DEV), dev_params(params), u.to(DEV), grads)
    torch.cuda.synchronize()
    h = synth.widen(params["b1"]) + synth.widen(params["W1"])[0]
    h = h.astype(np.float32).astype(np.float64)
    phi = np.array([0.5 * math.erfc(-t / math.sqrt(2.0)) for t in h])
    prime = phi + h * np.exp(-0.5 * h * h) / math.sqrt(2 * math.pi)
    check("gelu' rows=%d s=%g" % (rows, sd), float(np.sqrt(((to_np(grads["b1"]) - prime) ** 2).mean())), 2.0 ** -25)
    some = (np.abs(h) > 1e-3) & (h > -13)   # (GELU itself: 8e-6 of its value down to -13)
    check("gelu rows=%d s=%g" % (rows, sd), float(np.abs(to_np(grads["W2"])[some, 0] / (h * phi)[some] - 1.0).max()), 2.0 ** -17 + 8e-6)


def shifted(t, by):
    """The same values `by` elements into a buffer: aligned to their elements only."""
    buf = torch.empty(t.numel() + by, dtype=t.dtype, device=DEV)
    buf[by:] = t.reshape(-1).to(DEV)
    return buf[by:].view(t.shape)


@pytest.mark.parametrize("rows", [31, 200])
@pytest.mark.parametrize("what", ["x", "W1", "W2", "b1", "all"])
def test_operands_aligned_to_their_elements_only(rows, what):
    # (200 rows at dh = 2048: tiles in the ring where everything is aligned)
    xq, xp, r, params = small_problem(B=rows, P=rows + 37, din=192, dh=2048, dout=256)
    p64 = widen_params(params)
    put = lambda name, t: shifted(t, 1 if name != "W2" else 5) if what in (name, "all") else t.to(DEV)  # noqa: E731
    dp = {k: put(k, v) for k, v in params.items()}
    x, other = put("x", xq), put("x", xp)
    y = gc.gc_mlp_forward_nograd_bf16(x, dp)
    u = torch.from_numpy((np.random.default_rng(rows).standard_normal((rows, 256)) * 1e-3).astype(np.float32))
    grads = gc.zero_mlp_grads(dp)
    gc.gc_chunk_surrogate_backward_bf16(x, dp, shifted(u, 1) if what == "all" else u.to(DEV), grads)
    torch.cuda.synchronize()
    check("shifted %s y" % what, relerr(to_np(y), O.mlp_forward(synth.widen(xq), p64)), 2.0 ** -8)
    want = O.mlp_backward(synth.widen(xq), p64, synth.widen(u))
    for k in ("W1", "b1", "W2", "b2"):
        check("shifted %s d%s" % (what, k), relerr(to_np(grads[k]), want[k]), 2.0 ** -14)
    out = gc.gc_step_mlp_bf16(x, other, r.to(DEV), 32, 64, dp, 1.0, 0.2, keep=True)
    torch.cuda.synchronize()
    stagewise("shifted %s step" % what, out, xq, xp, r, params, 32, 64, 1.0, 0.2)


@pytest.mark.parametrize("what", ["x", "W1", "W2", "all"])
@pytest.mark.parametrize("rows,din,dh,dout", [(700, 192, 2048, 256), (3000, 2048, 512, 128), (6000, 704, 128, 128)])
def test_copies_of_operands_that_are_not_aligned(rows, din, dh, dout, what):
    """The kernels are those of aligned operands, so are the bits; where the copy of x leaves room for half of the rows only (the second and
    third size), the gradients add up in another order: sums of at most `rows` terms in fp32."""
    xq, _, _, params = small_problem(B=rows, din=din, dh=dh, dout=dout)
    put = lambda name, t: shifted(t, 3) if what in (name, "all") else t.to(DEV)  # noqa: E731
    u = torch.from_numpy((np.random.default_rng(rows).standard_normal((rows, dout)) * 1e-3).astype(np.float32)).to(DEV)
    got = []
    for x, w in ((xq.to(DEV), dev_params(params)), (put("x", xq), {k: put(k, v) for k, v in params.items()})):
        grads = gc.zero_mlp_grads(w)
        gc.gc_chunk_surrogate_backward_bf16(x, w, u, grads)
        got.append((gc.gc_mlp_forward_nograd_bf16(x, w), grads))
    torch.cuda.synchronize()
    (y, want), (y2, grads) = got
    assert torch.equal(y, y2)
    for k in want:
        if rows >= 3000 and what in ("x", "all"):
            check("copies %s %d rows d%s" % (what, rows, k), relerr(to_np(grads[k]), to_np(want[k])), 2.0 ** -24 * math.sqrt(rows))
        else:
            assert torch.equal(grads[k], want[k]), k


def test_bias_gradient_of_many_rows():
    """db1 sums dA over every row, so that a bias of dA far below its rounding shows.  Beside what the two bf16 planes of U leave only the
    additions of 2048 block sums in a row: each up to 2^-24 of the sum so far off, independently, 2^-24 / sqrt 3 in the mean; 7 % for two standard
    deviations of a norm over 384 entries."""
    rows, din, dh, dout = 65536, 64, 384, 128
    g = torch.Generator().manual_seed(9)
    normal = lambda *s: torch.randn(*s, generator=g)  # noqa: E731
    params = {k: (normal(*s) * 0.02).to(torch.bfloat16).to(DEV) for k, s in (("W1", (din, dh)), ("b1", (dh,)), ("W2", (dh, dout)), ("b2", (dout,)))}
    x, u = normal(rows, din).to(torch.bfloat16).to(DEV), (normal(rows, dout) * 1e-3).to(DEV)
    grads = gc.zero_mlp_grads(params)
    gc.gc_chunk_surrogate_backward_bf16(x, params, u, grads)
    torch.cuda.synchronize()
    h = x.double() @ params["W1"].double() + params["b1"].double()
    prime = 0.5 * (1.0 + torch.erf(h / math.sqrt(2.0))) + h * torch.exp(-0.5 * h * h) / math.sqrt(2.0 * math.pi)
    db1 = lambda v: ((v @ params["W2"].double().T) * prime).sum(0)  # noqa: E731
    hi = u.bfloat16().double()
    two = hi + (u.double() - hi).bfloat16().double()
    want = db1(u.double())
    off = lambda got: float((got.double() - want).norm() / want.norm())  # noqa: E731
    check("db1 of %d rows" % rows, off(grads["b1"]), 1.07 * math.hypot(off(db1(two)), 2.0 ** -24 / math.sqrt(3.0) * math.sqrt(rows / 32 / 2)))
