"""Precision of the automatic choice between sparse and dense kernels.  Below the density where the dense kernels are
the rule for a shape, every product keeps its fp32 operands in full (24 bits), whichever kernels the modelled
times pick; two bfloat16 parts per operand (16 bits) show as errors of 3e-6 to 1e-5 of the largest output.  Shapes on
both sides of the choice: whole tiles of the two-part kernels in short batches, and layers that only some of those
kernels' tiles divide."""
import numpy as np
import pytest

import paper_2408_11746_amd as mst
import synth
from oracle import products as opr

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
from gpu_util import Rig, DEV, dev, rel_err  # noqa: E402

FULL = 2e-6          # max error over max value of fp32 sums of up to a few thousand terms


@pytest.mark.parametrize("act,T,I,O,density", [
    ("f32", 1024, 768, 3072, 0.149), ("f32", 1024, 3072, 768, 0.149), ("f32", 512, 1024, 4096, 0.149), ("f32", 1792, 1280, 2560, 0.12),
    ("f32", 512, 640, 320, 0.28), ("f32", 256, 320, 576, 0.299),
    ("bf16", 256, 768, 3072, 0.25), ("bf16", 256, 768, 2304, 0.299), ("bf16", 1792, 1280, 2560, 0.2), ("bf16", 4096, 1056, 5120, 0.12)])
def test_automatic_products_keep_fp32_operands_in_full(act, T, I, O, density):
    print("case", act, T, I, O, density, flush=True)
    a = mst.MST_F32 if act == "f32" else mst.MST_BF16
    W, M = synth.make_layer(33, 1, I, O, density)
    W = (W * np.exp2(synth.normal(33, 8, W.shape))).astype(np.float32)
    if act == "f32":
        X, dY = synth.make_activations(33, 1, T, I, O)
        Xd, dYd = dev(X), dev(dY)
    else:
        X, dY, xb, yb = synth.make_activations(33, 1, T, I, O, "bf16")
        Xd, dYd = dev(xb.view(np.int16)), dev(yb.view(np.int16))
    rig = Rig(W, M, T, cap=int(M.sum()))
    L = rig.layer
    new = lambda *s: torch.full(s, float("nan"), dtype=torch.float32, device=DEV)  # noqa: E731
    Y, dX, dW, dX2, dW2 = new(T, O), new(T, I), new(L.nnz), new(T, I), new(L.nnz)
    mst.mst_sparse_fc_fwd(L, Xd, Y, T, a)
    mst.mst_sparse_fc_bwd_input(L, dYd, dX, T, a)
    mst.mst_sparse_fc_bwd_weight(L, dYd, Xd, dW, T, rig.ws, a)
    mst.mst_sparse_fc_bwd(L, dYd, Xd, dX2, dW2, T, rig.ws, a)
    torch.cuda.synchronize()
    print("dense: Y and dX, dW, one call:", [L.uses_dense(a, T, k) for k in (0, 1, 2)], flush=True)
    Yr, dXr, dWr = opr.fc_fwd(X, W, M), opr.fc_bwd_input(dY, W, M), opr.fc_bwd_weight(dY, X, M)
    errs = [rel_err(g.cpu().numpy(), r) for g, r in ((Y, Yr), (dX, dXr), (dW, dWr), (dX2, dXr), (dW2, dWr))]
    print("errors Y / dX / dW / one call:", ["%.2g" % e for e in errs], flush=True)
    assert max(errs) <= FULL
