"""mst_layer_sync_values and the views that no product has walked yet: handed over inside a recorded step,
whose replays come between eager products, and outside of one.  Against the oracle (App. Eq. (1) and its
gradient) at every point."""
import numpy as np
import pytest

import paper_2408_11746_amd as mst
import synth
from oracle import products as opr

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
from gpu_util import Rig, TOL, DEV, dev, rel_err  # noqa: E402


def _layer(mask, T=96, I=640, O=512):
    W, M = synth.make_layer(97, 1, I, O, 0.1, mask)
    X, dY = synth.make_activations(97, 1, T, I, O)
    mst.mst_heavy_rows(2 if mask == "powerlaw" else 1)      # (then dense rows beside the row view as well)
    try:
        rig = Rig(W, M, T)
    finally:
        mst.mst_heavy_rows(1)
    assert (rig.layer.format_stats()["heavy_rows"] > 0) == (mask == "powerlaw")
    return rig, X, dY, opr.fc_fwd(X, W, M), opr.fc_bwd_input(dY, W, M)


def _dense_copy_in_use(rig, X):
    rig.layer.set_path(mst.MST_PATH_DENSE)
    rig.fwd(X)


@pytest.mark.parametrize("mask", ["uniform", "powerlaw"])
def test_replays_of_a_recorded_handover_reach_views_walked_between_them(mask):
    """A step on the dense products is recorded with its hand-over before anything has walked a view; the
    sparse kernels then walk both views between its replays."""
    rig, X, dY, Y1, dX1 = _layer(mask)
    L = rig.layer
    _dense_copy_in_use(rig, X)
    Xd, Yg = dev(X), torch.empty((X.shape[0], rig.O), dtype=torch.float32, device=DEV)
    graph, side = torch.cuda.CUDAGraph(), torch.cuda.Stream()
    torch.cuda.synchronize()
    with torch.cuda.graph(graph, stream=side):
        mst.mst_sparse_fc_fwd(L, Xd, Yg, X.shape[0], mst.MST_F32, side)
        L.values().mul_(2.0)
        L.sync_values(side)
    for k in range(4):
        graph.replay()
        torch.cuda.synchronize()
        assert rel_err(Yg.cpu().numpy(), 2.0 ** k * Y1) <= TOL
        L.set_path(mst.MST_PATH_SPARSE)
        assert rel_err(rig.fwd(X), 2.0 ** (k + 1) * Y1) <= TOL, k
        if k > 0:                                            # the col view's first walk comes a replay later
            assert rel_err(rig.bwd_input(dY), 2.0 ** (k + 1) * dX1) <= TOL, k
        L.set_path(mst.MST_PATH_DENSE)


@pytest.mark.parametrize("mask", ["uniform", "powerlaw"])
def test_a_recorded_handover_that_has_not_run_leaves_views_to_be_refreshed(mask):
    """Views that missed a change of the values, walked first by a recording with a hand-over in it: products
    before the first replay see the values all the same, and so do the replays."""
    rig, X, dY, Y1, dX1 = _layer(mask)
    L, T = rig.layer, X.shape[0]
    _dense_copy_in_use(rig, X)
    L.values().mul_(2.0)
    L.sync_values()
    L.set_path(mst.MST_PATH_SPARSE)
    Xd, dYd = dev(X), dev(dY)
    Yg = torch.empty((T, rig.O), dtype=torch.float32, device=DEV)
    dXg = torch.empty((T, rig.I), dtype=torch.float32, device=DEV)
    graph, side = torch.cuda.CUDAGraph(), torch.cuda.Stream()
    torch.cuda.synchronize()
    with torch.cuda.graph(graph, stream=side):
        mst.mst_sparse_fc_fwd(L, Xd, Yg, T, mst.MST_F32, side)
        mst.mst_sparse_fc_bwd_input(L, dYd, dXg, T, mst.MST_F32, side)
        L.sync_values(side)
    assert rel_err(rig.fwd(X), 2.0 * Y1) <= TOL
    assert rel_err(rig.bwd_input(dY), 2.0 * dX1) <= TOL
    for k in range(3):
        graph.replay()
        torch.cuda.synchronize()
        assert rel_err(Yg.cpu().numpy(), 2.0 ** (k + 1) * Y1) <= TOL, k
        assert rel_err(dXg.cpu().numpy(), 2.0 ** (k + 1) * dX1) <= TOL, k
        L.values().mul_(2.0)
        L.sync_values()
        assert rel_err(rig.fwd(X), 2.0 ** (k + 2) * Y1) <= TOL, k


@pytest.mark.parametrize("mask", ["uniform", "powerlaw"])
def test_a_views_first_walk_sees_what_was_handed_over(mask):
    """Values changed after the last hand-over stay out of every product until the next one, whichever view is
    walked, and for the first time or not."""
    rig, X, dY, Y1, dX1 = _layer(mask)
    L = rig.layer
    _dense_copy_in_use(rig, X)
    L.values().mul_(2.0)
    L.sync_values()                                          # no view has been walked: left out
    L.values().mul_(2.0)                                     # not handed over
    assert rel_err(rig.fwd(X), 2.0 * Y1) <= TOL              # the dense product
    L.set_path(mst.MST_PATH_SPARSE)
    assert rel_err(rig.fwd(X), 2.0 * Y1) <= TOL
    assert rel_err(rig.bwd_input(dY), 2.0 * dX1) <= TOL
    L.sync_values()
    assert rel_err(rig.fwd(X), 4.0 * Y1) <= TOL
    assert rel_err(rig.bwd_input(dY), 4.0 * dX1) <= TOL
    W, M = rig.export()
    rig.layer.load_dense(dev(W), dev(M), rig.ws)             # no dense copy in use: every built view is refreshed
    L.values().mul_(2.0)
    L.sync_values()
    L.values().mul_(2.0)
    assert rel_err(rig.fwd(X), 8.0 * Y1) <= TOL
    assert rel_err(rig.bwd_input(dY), 8.0 * dX1) <= TOL


def test_a_recorded_first_walk_outlives_the_dense_copy_it_was_recorded_beside():
    """A recording that takes the refresh of a view with it, replayed while the dense copy holds the values
    handed over last and after the layer was loaded anew (the copy then holds old ones)."""
    rig, X, dY, Y1, dX1 = _layer("uniform")
    L, T = rig.layer, X.shape[0]
    _dense_copy_in_use(rig, X)
    L.values().mul_(2.0)
    L.sync_values()
    L.set_path(mst.MST_PATH_SPARSE)
    Xd, Yg = dev(X), torch.empty((T, rig.O), dtype=torch.float32, device=DEV)
    graph, side = torch.cuda.CUDAGraph(), torch.cuda.Stream()
    torch.cuda.synchronize()
    with torch.cuda.graph(graph, stream=side):
        mst.mst_sparse_fc_fwd(L, Xd, Yg, T, mst.MST_F32, side)

    def replayed():
        graph.replay()
        torch.cuda.synchronize()
        return Yg.cpu().numpy()

    L.values().mul_(2.0)                                     # not handed over
    assert rel_err(replayed(), 2.0 * Y1) <= TOL
    L.sync_values()
    assert rel_err(replayed(), 4.0 * Y1) <= TOL
    W, M = rig.export()
    L.load_dense(dev(4.0 * W), dev(M), rig.ws)
    assert rel_err(replayed(), 16.0 * Y1) <= TOL
    L.values().mul_(2.0)
    L.sync_values()
    L.values().mul_(2.0)                                     # not handed over
    assert rel_err(replayed(), 32.0 * Y1) <= TOL
    assert rel_err(rig.fwd(X), 32.0 * Y1) <= TOL
