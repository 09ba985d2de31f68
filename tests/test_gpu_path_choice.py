"""Y and dX choose between the sparse and the dense kernels each for itself: layers that are wide on one side only,
where the two products have their cross-over at different densities.  Which kernels ran shows in the bits."""
import numpy as np
import pytest

import paper_2408_11746_amd as mst
import synth
from oracle import products as opr

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
from gpu_util import Rig, TOL, DEV, dev, rel_err  # noqa: E402


# (modelled times of the slower kernels are 1.4 to 1.9 times those of the faster ones, either way round)
@pytest.mark.parametrize("act,T,I,O,density,y_dense", [("f32", 504, 3392, 448, 0.09, True), ("f32", 320, 369, 4224, 0.059, False),
                                                       ("f32", 573, 256, 2560, 0.068, False), ("bf16", 126, 4684, 559, 0.025, True)])
def test_y_and_dx_choose_for_themselves(act, T, I, O, density, y_dense):
    print("case", act, T, I, O, density, flush=True)
    a = mst.MST_F32 if act == "f32" else mst.MST_BF16
    W, M = synth.make_layer(34, 1, I, O, density)
    if act == "f32":
        X, dY = synth.make_activations(34, 1, T, I, O)
        Xd, dYd = X, dY
    else:
        X, dY, xb, yb = synth.make_activations(34, 1, T, I, O, "bf16")
        Xd, dYd = xb.view(np.int16), yb.view(np.int16)
    rig = Rig(W, M, T)
    L = rig.layer
    got = {}
    for path in (mst.MST_PATH_AUTO, mst.MST_PATH_SPARSE, mst.MST_PATH_DENSE):
        L.set_path(path)
        got[path] = (rig.fwd(Xd, a), rig.bwd_input(dYd, a))
    L.set_path(mst.MST_PATH_AUTO)
    assert L.uses_dense(a, T, 0) == y_dense and L.uses_dense(a, T, 3) != y_dense
    for k, (dense, ref) in enumerate(((y_dense, opr.fc_fwd(X, W, M)), (not y_dense, opr.fc_bwd_input(dY, W, M)))):
        auto, sparse, full = (got[p][k] for p in (mst.MST_PATH_AUTO, mst.MST_PATH_SPARSE, mst.MST_PATH_DENSE))
        assert rel_err(auto, ref) <= TOL and not np.array_equal(sparse, full)
        assert np.array_equal(auto, full if dense else sparse)
