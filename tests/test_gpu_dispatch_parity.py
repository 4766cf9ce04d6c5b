"""GPU parity at the edges of the kernels' tiles and of the rules that choose between them, against the fp64 oracle."""
import numpy as np
import pytest
import torch

from paper_2101_06983_amd import binding as gc
from paper_2101_06983_amd import synth
from parity import TOL_BF16, TOL_F32, check, check_argmax, check_loss, oracle_loss, relerr, to_np

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
