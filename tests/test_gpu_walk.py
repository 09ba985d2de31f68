"""The walk kernels at the edges of their tiles: one index more or less than a chunk of 640, a block of
128 rows, a tile of 64 tokens, a sub-chunk; rows of an odd number of bfloat16; octets without
entries between others; rows spread over an octet; chunks split over workgroups; token ranges and
the slot kernel of the call without a workspace.  Against the oracle (App. Eq. (1) and its
gradients)."""
import numpy as np
import pytest

import paper_2408_11746_amd as mst
import synth
from oracle import products as opr

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
from gpu_util import Rig, DEV, dev, rel_err  # noqa: E402

# max error over max value.  Sums of n <= 1300 fp32 products in a fixed order: rounding errors of random sign add up to
# about sqrt(n) 2^-24 = 2.1e-6 of a sum of that many terms at the worst, and no output here has more than 160 (a full
# row of the spread test: 1300 in eight lane groups, a weight gradient: 1100 tokens in tiles of 64), so 7.5e-7.  Observed 2e-7.
TOL = 2e-6
HEAVY = 2e-5         # Y where rows are kept out of the row view: two bfloat16 parts per operand, 3 * 2^-18 = 1.1e-5 of a product

SPMM = [(0, 0), (128, 2), (128, 3), (128, 4), (64, 4), (64, 6), (64, 8)]     # 1 .. 6 row blocks per workgroup
BOTH = [(16, 1), (16, 2), (8, 4), (8, 5)]


def _check(W, M, X, dY, act=mst.MST_F32, Xd=None, dYd=None):
    T = X.shape[0]
    rig = Rig(W, M, T, cap=max(1, int(M.sum())))
    rig.layer.set_path(mst.MST_PATH_SPARSE)
    Xd, dYd = (dev(X), dev(dY)) if Xd is None else (Xd, dYd)
    nnz = rig.layer.nnz
    Yr, dXr, dWr = opr.fc_fwd(X, W, M), opr.fc_bwd_input(dY, W, M), opr.fc_bwd_weight(dY, X, M)
    new = lambda *shape: torch.full(shape, float("nan"), dtype=torch.float32, device=DEV)  # noqa: E731
    ys, dxs, dws = [], [], []
    try:
        for shape in SPMM:
            mst.mst_spmm_force_shape(*shape)
            Y, dX = new(T, rig.O), new(T, rig.I)
            mst.mst_sparse_fc_fwd(rig.layer, Xd, Y, T, act)
            mst.mst_sparse_fc_bwd_input(rig.layer, dYd, dX, T, act)
            ys.append(Y.cpu().numpy())
            dxs.append(dX.cpu().numpy())
        for shape in [(0, 0)] + BOTH:
            mst.mst_bwd_force_shape(*shape)
            dX, dW = new(T, rig.I), new(max(nnz, 1))
            mst.mst_sparse_fc_bwd(rig.layer, dYd, Xd, dX, dW, T, rig.ws, act)
            assert rel_err(dX.cpu().numpy(), dXr) <= TOL, shape
            if shape != (0, 0):
                dxs.append(dX.cpu().numpy())
            dws.append(dW.cpu().numpy()[:nnz])
    finally:
        mst.mst_spmm_force_shape(0, 0)
        mst.mst_bwd_force_shape(0, 0)
    dW = new(max(nnz, 1))
    mst.mst_sparse_fc_bwd_weight(rig.layer, dYd, Xd, dW, T, rig.ws, act)
    dW = dW.cpu().numpy()[:nnz]
    heavy = rig.layer.format_stats()["heavy_rows"] > 0
    assert rel_err(ys[0], Yr) <= (HEAVY if heavy else TOL) and rel_err(dxs[0], dXr) <= TOL
    if nnz:
        assert rel_err(dws[0], dWr) <= TOL and rel_err(dW, dWr) <= TOL
    for group in (ys, dxs, dws):
        for other in group[1:]:
            np.testing.assert_array_equal(other, group[0])
    return rig, Xd, dYd, dW


@pytest.mark.parametrize("O,I", [(127, 639), (128, 640), (129, 641), (1, 1281), (1283, 3), (260, 1279), (769, 515)])
@pytest.mark.parametrize("T", [1, 63, 64, 65, 193])
def test_edges_of_chunks_blocks_and_token_tiles(O, I, T):
    print("case", O, I, T, flush=True)
    W, M = synth.make_layer(900 + O, 1, I, O, 0.06)
    X, dY = synth.make_activations(900 + O, 1, T, I, O)
    _check(W, M, X, dY)


@pytest.mark.parametrize("O,I,T", [(131, 129, 70), (130, 257, 65), (257, 642, 33)])
def test_bfloat16_rows_of_odd_and_even_length(O, I, T):
    print("case", O, I, T, flush=True)
    W, M = synth.make_layer(950 + O, 1, I, O, 0.08)
    X, dY, xb, yb = synth.make_activations(950 + O, 1, T, I, O, "bf16")
    _check(W, M, X, dY, mst.MST_BF16, dev(xb.view(np.int16)), dev(yb.view(np.int16)))


@pytest.mark.parametrize("O,I,T", [(400, 700, 129), (1030, 1300, 66)])
def test_empty_octets_and_spread_rows(O, I, T):
    """Blocks with a few full rows among empty ones (spread over whole octets), blocks with nothing, and
    columns that leave whole chunks of the other view empty."""
    print("case", O, I, T, flush=True)
    rng = np.random.default_rng(O)
    M = (rng.random((O, I)) < 0.03).astype(np.uint8)
    M[rng.random(O) < 0.7] = 0
    M[128:256] = 0
    M[rng.random(O) < 0.04] = 1
    M[:, I // 3: I // 3 + 200] = 0
    W = (synth.normal(O, 5, (O, I), 0.02) * M).astype(np.float32)
    X, dY = synth.make_activations(960 + O, 1, T, I, O)
    _check(W, M, X, dY)


def test_weight_gradient_without_a_workspace_in_token_ranges_and_by_slots():
    """More token tiles than the library's array has planes for (taken in ranges), and a layer whose
    capacity leaves not one plane (taken slot by slot): the bits of the call with a workspace."""
    for O, I, T, cap in ((768, 1536, 1100, 220000), (4112, 4112, 40, 2300000)):
        print("case", O, I, T, cap, flush=True)
        W, M = synth.make_layer(970 + O, 1, I, O, 0.02 if O < 4000 else 0.002)
        X, dY = synth.make_activations(970 + O, 1, T, I, O)
        rig = Rig(W, M, T, cap=cap)
        rig.layer.set_path(mst.MST_PATH_SPARSE)
        want = rig.bwd_weight(dY, X)
        got = torch.full((rig.layer.nnz,), float("nan"), dtype=torch.float32, device=DEV)
        mst.mst_sparse_fc_bwd_weight_static(rig.layer, dev(dY), dev(X), got, T)
        torch.cuda.synchronize()
        np.testing.assert_array_equal(got.cpu().numpy(), want)
        assert rel_err(want, opr.fc_bwd_weight(dY, X, M)) <= TOL


@pytest.mark.parametrize("O,I,T,density,cap", [(1526, 2380, 1016, 0.03, 434108), (1679, 1110, 1247, 0.053, 396120),
                                               (937, 1424, 1559, 0.0635, 169342), (3317, 5118, 117, 0.0021, 2707830)])
def test_weight_gradient_without_a_workspace_walks_the_view_of_the_whole_batch(O, I, T, density, cap):
    """Layers whose token ranges by themselves (or whose slots, where no plane fits) would be driven by the other
    view than the whole batch: its lane groups add the tokens of a tile in another order."""
    print("case", O, I, T, density, cap, flush=True)
    W, M = synth.make_layer(975, 1, I, O, density)
    X, dY = synth.make_activations(975, 1, T, I, O)
    rig = Rig(W, M, T, cap=cap)
    rig.layer.set_path(mst.MST_PATH_SPARSE)
    want = rig.bwd_weight(dY, X)
    got = torch.full((rig.layer.nnz,), float("nan"), dtype=torch.float32, device=DEV)
    mst.mst_sparse_fc_bwd_weight_static(rig.layer, dev(dY), dev(X), got, T)
    torch.cuda.synchronize()
    np.testing.assert_array_equal(got.cpu().numpy(), want)


def test_values_reach_views_that_no_product_has_walked_yet():
    O, I, T = 300, 500, 70
    W, M = synth.make_layer(980, 1, I, O, 0.05)
    X, dY = synth.make_activations(980, 1, T, I, O)
    rig = Rig(W, M, T)
    L = rig.layer
    L.set_path(mst.MST_PATH_SPARSE)
    L.values().mul_(2.0)
    L.sync_values()                                   # before any walk
    assert rel_err(rig.fwd(X), opr.fc_fwd(X, 2 * W, M)) <= TOL
    L.values().mul_(2.0)
    L.sync_values()                                   # the row view has been walked, the col view has not
    assert rel_err(rig.fwd(X), opr.fc_fwd(X, 4 * W, M)) <= TOL
    assert rel_err(rig.bwd_input(dY), opr.fc_bwd_input(dY, 4 * W, M)) <= TOL


@pytest.mark.parametrize("T", [100, 384])
def test_values_changed_before_a_views_first_walk(T):
    """A view that nothing has walked takes changed values with its first walk: a recording that comes first must
    not count as one, other streams see them as soon as the call is back, and a recorded walk goes on
    seeing new values after the view was built anew."""
    I, O = 640, 512
    W, M = synth.make_layer(95, 1, I, O, 0.5)
    X, _ = synth.make_activations(95, 2, T, I, O)
    rig = Rig(W, M, T, cap=int(M.sum()))
    L, Xd = rig.layer, dev(X)
    new = lambda: torch.full((T, O), float("nan"), dtype=torch.float32, device=DEV)  # noqa: E731
    ref = opr.fc_fwd(X, W, M)
    L.set_path(mst.MST_PATH_SPARSE)
    L.values().mul_(2.0)
    L.sync_values()
    torch.cuda.synchronize()
    Yg, graph, side = new(), torch.cuda.CUDAGraph(), torch.cuda.Stream()
    with torch.cuda.graph(graph, stream=side):
        mst.mst_sparse_fc_fwd(L, Xd, Yg, T, mst.MST_F32, side)
    Y0, Y1 = new(), new()
    mst.mst_sparse_fc_fwd(L, Xd, Y0, T, mst.MST_F32, torch.cuda.current_stream())
    mst.mst_sparse_fc_fwd(L, Xd, Y1, T, mst.MST_F32, side)
    torch.cuda.synchronize()
    assert rel_err(Y0.cpu().numpy(), 2.0 * ref) <= TOL
    assert torch.equal(Y0, Y1)
    for k in range(3):                                       # replays with eager work and other values between them
        graph.replay()
        torch.cuda.synchronize()
        assert rel_err(Yg.cpu().numpy(), 2.0 ** (1 + k) * ref) <= TOL
        L.values().mul_(2.0)
        L.sync_values()
    W2 = (W * 16.0).astype(np.float32)
    L.load_dense(dev(W2), dev(M.astype(np.uint8)), rig.ws)    # views built anew, walked by nothing but the graph
    L.values().mul_(0.25)
    L.sync_values()
    graph.replay()
    torch.cuda.synchronize()
    assert rel_err(Yg.cpu().numpy(), 4.0 * ref) <= TOL
