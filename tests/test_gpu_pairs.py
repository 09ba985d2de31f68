"""Y and dX on the sparse matrix instructions, pinned: token tiles and their remainders, bands of 256 rows and parts of
one, one and more k steps, masks whose quads overflow nowhere, here and there and everywhere, and every way in which the
weights change.  Against the oracle (App. Eq. (1) and its gradient); two bfloat16 parts per fp32 operand leave at most 3 * 2^-18 of a
term (one operand in parts: 2^-17), the bound of the dense kernels that share this arithmetic."""
import numpy as np
import pytest

import paper_2408_11746_amd as mst
import synth
from oracle import products as opr

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
from gpu_util import Rig, DEV, dev, rel_err  # noqa: E402

PARTS = 2e-5
PAIRS = 24


@pytest.fixture(autouse=True)
def pinned():
    mst.mst_gemm_force_fp32_mfma(PAIRS)
    yield
    mst.mst_gemm_force_fp32_mfma(0)


def _layer(T, I, O, density, dtype, mask="uniform", seed=71):
    W, M = synth.make_layer(seed, 1, I, O, density, mask)
    if dtype == "bf16":
        X, dY, xb, yb = synth.make_activations(seed, 2, T, I, O, "bf16")
        ops = xb.view(np.int16), yb.view(np.int16)
    else:
        X, dY = synth.make_activations(seed, 2, T, I, O)
        ops = X, dY
    rig = Rig(W, M, T, cap=O * I)
    rig.layer.set_path(mst.MST_PATH_DENSE)
    return rig, W, M, X, dY, ops, mst.MST_BF16 if dtype == "bf16" else mst.MST_F32


def _check(rig, ops, act, Y, dX, what):
    assert rel_err(rig.fwd(ops[0], act), Y) <= PARTS, what
    assert mst.mst_gemm_last_tile() == PAIRS, what
    assert rel_err(rig.bwd_input(ops[1], act), dX) <= PARTS, what
    assert mst.mst_gemm_last_tile() == PAIRS, what


# the pinned token tile of bfloat16 goes by T mod 3: 128, 192, 256
@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("T,I,O,density", [
    (1, 64, 64, 0.1), (127, 64, 256, 0.02), (128, 128, 320, 0.1), (129, 192, 64, 0.3), (191, 320, 192, 0.1), (192, 256, 512, 0.12),
    (193, 448, 256, 1.0), (257, 768, 832, 0.1), (700, 576, 640, 0.15), (300, 1088, 64, 0.6), (385, 64, 1344, 0.0)])
def test_products(T, I, O, density, dtype):
    print("case", T, I, O, density, dtype, flush=True)
    rig, W, M, X, dY, ops, act = _layer(T, I, O, density, dtype)
    _check(rig, ops, act, opr.fc_fwd(X, W, M), opr.fc_bwd_input(dY, W, M), "uniform")


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
def test_full_rows_and_columns(dtype):
    """A power-law mask: rows that fill every quad beside empty ones."""
    T, I, O = 260, 512, 768
    rig, W, M, X, dY, ops, act = _layer(T, I, O, 0.05, dtype, "powerlaw")
    _check(rig, ops, act, opr.fc_fwd(X, W, M), opr.fc_bwd_input(dY, W, M), "power law")


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
def test_packed_weights_follow_the_layer(dtype):
    T, I, O = 260, 320, 512
    rig, W, M, X, dY, ops, act = _layer(T, I, O, 0.1, dtype)
    L = rig.layer
    Y1, dX1 = opr.fc_fwd(X, W, M), opr.fc_bwd_input(dY, W, M)
    _check(rig, ops, act, Y1, dX1, "first")
    L.values().mul_(2.0)
    L.sync_values()
    _check(rig, ops, act, 2.0 * Y1, 2.0 * dX1, "handed over")
    L.values()[::3] = 0.0                                    # weights of zero hold no slot
    L.sync_values()
    torch.cuda.synchronize()
    W2, M2 = rig.export()
    _check(rig, ops, act, opr.fc_fwd(X, W2, M2), opr.fc_bwd_input(dY, W2, M2), "zeros")
    L.load_dense(dev(W), dev(M), rig.ws)
    L.values().mul_(2.0)
    L.sync_values()                                          # (no dense copy in use)
    _check(rig, ops, act, 2.0 * Y1, 2.0 * dX1, "loaded anew")
    for density, views in ((0.12, False), (0.02, True), (0.5, False), (0.08, False)):
        L.set_path(mst.MST_PATH_SPARSE if views else mst.MST_PATH_DENSE)
        mst.mst_mask_update(L, dev(ops[1]), dev(ops[0]), T, density, 0.3, 0.25, 5, rig.ws, act)
        L.set_path(mst.MST_PATH_DENSE)
        L.values().add_(0.01)                                # grown weights take part
        L.sync_values()
        torch.cuda.synchronize()
        W2, M2 = rig.export()
        _check(rig, ops, act, opr.fc_fwd(X, W2, M2), opr.fc_bwd_input(dY, W2, M2), density)


@pytest.mark.parametrize("warm", [True, False])
def test_recorded_products_and_handovers(warm):
    """A step recorded with and without products before it, replayed between eager work; every replay against the oracle."""
    T, I, O = 200, 256, 320
    rig, W, M, X, dY, ops, act = _layer(T, I, O, 0.1, "f32")
    L, side = rig.layer, torch.cuda.Stream()
    Y1, dX1 = opr.fc_fwd(X, W, M), opr.fc_bwd_input(dY, W, M)
    if warm:
        _check(rig, ops, act, Y1, dX1, "eager")
    Xd, dYd = dev(X), dev(dY)
    Y, dX = (torch.zeros((T, n), dtype=torch.float32, device=DEV) for n in (O, I))
    graph = torch.cuda.CUDAGraph()
    torch.cuda.synchronize()
    with torch.cuda.graph(graph, stream=side):
        mst.mst_sparse_fc_fwd(L, Xd, Y, T, act, side)
        mst.mst_sparse_fc_bwd_input(L, dYd, dX, T, act, side)
        L.values().mul_(2.0)
        L.sync_values(side)
    scale = 1.0
    for k in range(3):
        graph.replay()
        torch.cuda.synchronize()
        assert rel_err(Y.cpu().numpy(), scale * Y1) <= PARTS, k
        assert rel_err(dX.cpu().numpy(), scale * dX1) <= PARTS, k
        scale *= 2.0
        assert rel_err(rig.fwd(X, act), scale * Y1) <= PARTS, k
        L.values().mul_(0.5)
        L.sync_values()
        torch.cuda.synchronize()
        scale *= 0.5
        assert rel_err(rig.fwd(X, act), scale * Y1) <= PARTS, k


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
def test_automatic_choice(dtype):
    """Whole tiles at a density of a tenth go there, half-dense ones do not, nor Y of a mask with full rows, whose every step goes a second time."""
    mst.mst_gemm_force_fp32_mfma(0)
    T, I, O = 8192, 768, 3072
    for density, mask, want in ((0.1, "uniform", True), (0.5, "uniform", False), (0.1, "powerlaw", False)):
        W, M = synth.make_layer(5, 1, I, O, density, mask)
        rig = Rig(W, M, T)
        X = torch.randn((T, I), dtype=torch.float32, device=DEV)
        x = X.to(torch.bfloat16) if dtype == "bf16" else X
        Y = torch.empty((T, O), dtype=torch.float32, device=DEV)
        mst.mst_sparse_fc_fwd(rig.layer, x, Y, T, mst.MST_BF16 if dtype == "bf16" else mst.MST_F32)
        torch.cuda.synchronize()
        assert (mst.mst_gemm_last_tile() == PAIRS) == want, (density, mask)
        ref = x[:64].double() @ torch.from_numpy((W * M).astype(np.float64)).to(DEV).T
        assert rel_err(Y[:64].cpu().numpy(), ref.cpu().numpy()) <= PARTS, (density, mask)


def test_recordings_side_by_side():
    """Two recordings that each make the packed weights, replayed on two streams at once: what one makes again the other may be
    reading (masks of second steps included), so it has to stay what it is throughout."""
    T, I, O = 1024, 512, 832
    rig, W, M, X, dY, ops, act = _layer(T, I, O, 0.3, "f32")
    mst.mst_gemm_force_fp32_mfma(0)
    rig.fwd(ops[0], act)                                     # the dense copy, and no packed weights
    mst.mst_gemm_force_fp32_mfma(PAIRS)
    L, Xd, dYd = rig.layer, dev(X), dev(dY)
    sides = [torch.cuda.Stream() for _ in range(2)]
    outs = [(torch.zeros((T, O), dtype=torch.float32, device=DEV), torch.zeros((T, I), dtype=torch.float32, device=DEV)) for _ in sides]
    graphs = []
    for side, (Y, dX) in zip(sides, outs):
        torch.cuda.synchronize()
        graph = torch.cuda.CUDAGraph()
        with torch.cuda.graph(graph, stream=side):
            for _ in range(4):
                mst.mst_sparse_fc_fwd(L, Xd, Y, T, act, side)
                mst.mst_sparse_fc_bwd_input(L, dYd, dX, T, act, side)
        graphs.append(graph)
    Yr, dXr = opr.fc_fwd(X, W, M), opr.fc_bwd_input(dY, W, M)
    for k in range(4):
        torch.cuda.synchronize()
        for graph, side, (Y, dX) in zip(graphs, sides, outs):
            with torch.cuda.stream(side):
                Y.zero_()
                dX.zero_()
                graph.replay()
        torch.cuda.synchronize()
        for Y, dX in outs:
            assert rel_err(Y.cpu().numpy(), Yr) <= PARTS, k
            assert rel_err(dX.cpu().numpy(), dXr) <= PARTS, k


# Workgroups that form more tiles than one, whose steps follow each other without a break: one, two and odd numbers of steps a tile, three
# kinds of token tiles (by T mod 3), a cut-off last band and last token tile, tiles for some workgroups of an XCD only.
@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("density", [0.07, 0.13])
@pytest.mark.parametrize("T,I,O", [(16385, 64, 1280), (16386, 128, 960), (16384, 192, 1024), (20000, 320, 832), (10020, 64, 2880), (9001, 448, 1856)])
def test_tiles_in_a_row(T, I, O, density, dtype):
    print("case", T, I, O, density, dtype, flush=True)
    g = torch.Generator(device=DEV)
    g.manual_seed(T + I)
    act, td = (mst.MST_BF16, torch.bfloat16) if dtype == "bf16" else (mst.MST_F32, torch.float32)
    W, M = synth.make_layer(5, 1, I, O, density)
    X = torch.randn(T, I, generator=g, device=DEV).to(td)
    dY = torch.randn(T, O, generator=g, device=DEV).to(td)
    rig = Rig(W, M, 64, cap=O * I)
    rig.layer.set_path(mst.MST_PATH_DENSE)
    Wd = dev(W).double() * dev(M)
    Y = torch.full((T, O), float("nan"), device=DEV)
    dX = torch.full((T, I), float("nan"), device=DEV)
    mst.mst_sparse_fc_fwd(rig.layer, X, Y, T, act)
    assert mst.mst_gemm_last_tile() == PAIRS
    mst.mst_sparse_fc_bwd_input(rig.layer, dY, dX, T, act)
    assert mst.mst_gemm_last_tile() == PAIRS
    for got, ref in ((Y, X.double() @ Wd.t()), (dX, dY.double() @ Wd)):
        assert float((got.double() - ref).abs().max()) <= PARTS * float(ref.abs().max())
