"""Infinite and NaN activations on the sparse path: an output has one only if a weight that is active meets it.  The
views pad a row's entries with zero weights at the first index of a chunk, so those indices are the ones that
could reach outputs they have no business in.  Against float64 sums over the active positions alone."""
import numpy as np
import pytest

import paper_2408_11746_amd as mst
import synth

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
from gpu_util import Rig, DEV, dev, rel_err  # noqa: E402

FP32 = 2e-6          # max error over max value of an fp32 sum of up to 2000 terms
CHUNK = 4            # chunks start at multiples of four indices


def _special(A, rng):
    """an infinity or NaN at chunk starts and elsewhere, a few tokens each"""
    T, K = A.shape
    for k in sorted({0, K - 1} | set(range(0, K, CHUNK)) & set(rng.integers(0, K, 40).tolist()) | {c for c in (128, 432, 512, 640, 644) if c < K}):
        A[rng.integers(0, T), k] = rng.choice([np.inf, -np.inf, np.nan])


def _product(A, S):
    """A S^T over the entries of S (dense array, active where mask) with nothing from inactive positions"""
    W, M = S
    clean = np.where(np.isfinite(A), A, 0.0).astype(np.float64) @ (W * M).astype(np.float64).T
    with np.errstate(invalid="ignore"):
        for t, k in zip(*np.nonzero(~np.isfinite(A))):
            rows = np.flatnonzero(M[:, k])
            clean[t, rows] += A[t, k].astype(np.float64) * W[rows, k]
    return clean


def _same(got, ref, tag):
    finite = np.isfinite(ref)
    assert np.array_equal(np.isnan(got), np.isnan(ref)), tag
    inf = np.isinf(ref)
    assert np.array_equal(got[inf], ref[inf].astype(np.float32)), tag
    assert rel_err(got[finite], ref[finite]) <= FP32, tag


@pytest.mark.parametrize("O,I,T,mask,act", [(260, 1279, 70, "uniform", "f32"), (515, 1283, 130, "uniform", "f32"), (131, 433, 65, "uniform", "bf16"),
                                            (400, 700, 129, "spread", "f32"), (642, 1290, 66, "spread", "bf16")])
def test_infinite_activations_reach_the_outputs_of_active_weights_only(O, I, T, mask, act):
    print("case", O, I, T, mask, act, flush=True)
    rng = np.random.default_rng(O)
    if mask == "uniform":
        W, M = synth.make_layer(970 + O, 1, I, O, 0.06)
    else:                                                    # a few full rows among empty ones: rows spread over an octet
        M = (rng.random((O, I)) < 0.03).astype(np.uint8)
        M[rng.random(O) < 0.7] = 0
        M[rng.random(O) < 0.04] = 1
        W = (synth.normal(O, 5, (O, I), 0.02) * M).astype(np.float32)
    W = W.copy()
    W[M != 0] = np.where(rng.random(int(M.sum())) < 0.01, 0.0, W[M != 0])      # active weights that are zero (as grown ones are)
    X, dY = (a.copy() for a in synth.make_activations(970 + O, 1, T, I, O))
    for a in (X, dY):
        a.view(np.uint32)[...] &= 0xFFFF0000                 # (exact in bfloat16)
        _special(a, rng)
    a = mst.MST_F32 if act == "f32" else mst.MST_BF16
    send = (lambda v: dev(v)) if act == "f32" else (lambda v: dev((v.view(np.uint32) >> 16).astype(np.int16)))
    Xd, dYd = send(X), send(dY)
    rig = Rig(W, M, T)
    L = rig.layer
    L.set_path(mst.MST_PATH_SPARSE)
    Yr, dXr = _product(X, (W, M)), _product(dY, (W.T, M.T))
    assert (~np.isfinite(Yr)).any() and np.isfinite(Yr).mean() > 0.5
    new = lambda *s: torch.full(s, 7.0, dtype=torch.float32, device=DEV)  # noqa: E731
    Y, dX, dW, dX2, dW2 = new(T, O), new(T, I), new(L.nnz), new(T, I), new(L.nnz)
    for shape in [(0, 0), (128, 2), (64, 8)]:
        try:
            mst.mst_spmm_force_shape(*shape)
            mst.mst_sparse_fc_fwd(L, Xd, Y, T, a)
            mst.mst_sparse_fc_bwd_input(L, dYd, dX, T, a)
            torch.cuda.synchronize()
        finally:
            mst.mst_spmm_force_shape(0, 0)
        _same(Y.cpu().numpy(), Yr, ("Y", shape))
        _same(dX.cpu().numpy(), dXr, ("dX", shape))
    mst.mst_sparse_fc_bwd(L, dYd, Xd, dX2, dW2, T, rig.ws, a)
    mst.mst_sparse_fc_bwd_weight(L, dYd, Xd, dW, T, rig.ws, a)
    torch.cuda.synchronize()
    _same(dX2.cpu().numpy(), dXr, "dX of the one-call backward")
    with np.errstate(invalid="ignore"):
        G = np.where(np.isfinite(dY), dY, 0.0).astype(np.float64).T @ np.where(np.isfinite(X), X, 0.0).astype(np.float64)
        for t, o in zip(*np.nonzero(~np.isfinite(dY))):
            G[o] += dY[t, o].astype(np.float64) * X[t]
        for t, i in zip(*np.nonzero(~np.isfinite(X))):
            G[:, i] += np.where(np.isfinite(dY[t]), dY[t].astype(np.float64) * X[t, i], 0.0)
    for tag, got in (("dW", dW), ("dW of the one-call backward", dW2)):
        _same(got.cpu().numpy(), G[M != 0], tag)
