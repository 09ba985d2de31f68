"""A layer whose first dense product is recorded: the recording forms the dense copy of the weights when it is replayed.  Eager calls that
come before the first replay, or instead of any, find weights all the same.  Against the oracle (App. Eq. (1) and its gradient)."""
import numpy as np
import pytest

import paper_2408_11746_amd as mst
import synth
from oracle import products as opr

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
from gpu_util import Rig, TOL, DEV, dev, rel_err  # noqa: E402


def _recorded(T, I, O, dtype):
    W, M = synth.make_layer(53, 1, I, O, 0.4)
    X, dY, xb, yb = synth.make_activations(53, 2, T, I, O, "bf16")
    ops, act = ((xb.view(np.int16), yb.view(np.int16)), mst.MST_BF16) if dtype == "bf16" else ((X, dY), mst.MST_F32)
    rig = Rig(W, M, T, cap=O * I)
    L, side, graph = rig.layer, torch.cuda.Stream(), torch.cuda.CUDAGraph()
    L.buf.fill_(0xFF)                                        # (NaN wherever nothing was written)
    L.load_dense(dev(W), dev(M), rig.ws)
    L.set_path(mst.MST_PATH_DENSE)
    Xd, Yg = dev(ops[0]), torch.zeros((T, O), dtype=torch.float32, device=DEV)
    torch.cuda.synchronize()
    with torch.cuda.graph(graph, stream=side):
        mst.mst_sparse_fc_fwd(L, Xd, Yg, T, act, side)
    rig.held = Xd                                            # (the recording reads it)
    return rig, W, M, X, dY, ops, act, graph, Yg


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("T,I,O", [(256, 256, 512), (77, 130, 90)])
def test_eager_products_before_the_first_replay(T, I, O, dtype):
    rig, W, M, X, dY, ops, act, graph, Yg = _recorded(T, I, O, dtype)
    L, Y, dX = rig.layer, opr.fc_fwd(X, W, M), opr.fc_bwd_input(dY, W, M)
    L.sync_values()                                          # (the active positions alone)
    assert rel_err(rig.fwd(ops[0], act), Y) <= TOL
    assert rel_err(rig.bwd_input(ops[1], act), dX) <= TOL
    for k in range(3):
        graph.replay()
        torch.cuda.synchronize()
        assert rel_err(Yg.cpu().numpy(), 2.0 ** k * Y) <= TOL, k
        L.values().mul_(2.0)
        L.sync_values()
        assert rel_err(rig.fwd(ops[0], act), 2.0 ** (k + 1) * Y) <= TOL, k


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
def test_an_update_before_the_first_replay(dtype):
    T, I, O = 256, 256, 512
    rig, W, M, X, dY, ops, act, graph, Yg = _recorded(T, I, O, dtype)
    L = rig.layer
    mst.mst_mask_update(L, dev(ops[1]), dev(ops[0]), T, 0.3, 0.3, 0.25, 5, rig.ws, act)      # (in place: the views stay unbuilt)
    L.values().add_(0.01)
    L.sync_values()
    torch.cuda.synchronize()
    W2, M2 = rig.export()
    assert rel_err(rig.fwd(ops[0], act), opr.fc_fwd(X, W2, M2)) <= TOL
    assert rel_err(rig.bwd_input(ops[1], act), opr.fc_bwd_input(dY, W2, M2)) <= TOL


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
def test_views_that_only_a_recording_has_built(dtype):
    """An update leaves the views unbuilt and a recorded backward builds them; eager calls before its first replay."""
    T, I, O = 256, 320, 512
    W, M = synth.make_layer(59, 1, I, O, 0.4)
    X, dY, xb, yb = synth.make_activations(59, 2, T, I, O, "bf16")
    ops, act = ((xb.view(np.int16), yb.view(np.int16)), mst.MST_BF16) if dtype == "bf16" else ((X, dY), mst.MST_F32)
    rig = Rig(W, M, T, cap=O * I)
    L, side, graph = rig.layer, torch.cuda.Stream(), torch.cuda.CUDAGraph()
    L.set_path(mst.MST_PATH_DENSE)
    rig.fwd(ops[0], act)
    mst.mst_mask_update(L, dev(ops[1]), dev(ops[0]), T, 0.2, 0.5, 0.25, 5, rig.ws, act)
    L.values().add_(0.01)
    L.sync_values()
    L.set_path(mst.MST_PATH_SPARSE)
    torch.cuda.synchronize()
    W, M = rig.export()
    Y, dX = opr.fc_fwd(X, W, M), opr.fc_bwd_input(dY, W, M)
    Xd, dYd = dev(ops[0]), dev(ops[1])
    dXg, dWg = torch.zeros((T, I), dtype=torch.float32, device=DEV), torch.zeros(L.nnz, dtype=torch.float32, device=DEV)
    torch.cuda.synchronize()
    with torch.cuda.graph(graph, stream=side):
        mst.mst_sparse_fc_bwd(L, dYd, Xd, dXg, dWg, T, rig.ws, act, side)
    assert rel_err(rig.fwd(ops[0], act), Y) <= TOL
    assert rel_err(rig.bwd_input(ops[1], act), dX) <= TOL
    dW = rig.bwd_weight(ops[1], ops[0], act)                 # (builds them)
    assert rel_err(rig.fwd(ops[0], act), Y) <= TOL
    scale = 1.0
    for k in range(3):
        graph.replay()
        torch.cuda.synchronize()
        assert rel_err(dXg.cpu().numpy(), scale * dX) <= TOL, k
        assert rel_err(dWg.cpu().numpy(), dW) <= 1e-5, k
        assert rel_err(rig.fwd(ops[0], act), scale * Y) <= TOL, k
        L.values().mul_(2.0)
        L.sync_values()
        scale *= 2.0
