"""mst_mask_update_from_scores_multi with layers that share a stream: their chains run in launches that take several layers.
Masks, weights, index sets and counts bit for bit as the oracle's (Algorithm 1) per layer, and the products on the
rebuilt views or dense copies; more layers than one launch takes, streams that repeat out of order, and in one call
layers that keep their views, stay dense, have heavy rows, another prune score, nothing to prune, to grow or to move."""
import numpy as np
import pytest

import paper_2408_11746_amd as mst
import synth
from oracle import mixed_growing as omg
from oracle import products as opr

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
from gpu_util import Rig, TOL, dev, rel_err  # noqa: E402

# O, I, density now, targets of the two updates, mask, path, prune score
LAYERS = [(300, 520, 0.08, (0.08, 0.05), "uniform", mst.MST_PATH_AUTO, 0.0),
          (64, 2100, 0.03, (0.03, 0.04), "powerlaw", mst.MST_PATH_AUTO, 0.0),          # heavy rows
          (256, 384, 0.5, (0.4, 0.4), "uniform", mst.MST_PATH_DENSE, 0.0),             # no views afterwards
          (129, 333, 0.2, (0.1, 0.2), "uniform", mst.MST_PATH_SPARSE, 0.5),
          (70, 65, 0.0, (0.0, 0.3), "uniform", mst.MST_PATH_AUTO, 0.0),                # nothing moves, then growth alone
          (700, 131, 0.3, (0.0, 0.0), "uniform", mst.MST_PATH_AUTO, 0.0),              # pruned away, then nothing left
          (96, 1030, 0.9, (1.0, 0.6), "uniform", mst.MST_PATH_DENSE, 0.0),
          (33, 47, 0.1, (0.1, 0.1), "uniform", mst.MST_PATH_AUTO, 0.0),
          (640, 641, 0.05, (0.05, 0.02), "uniform", mst.MST_PATH_SPARSE, 0.0),
          (1, 900, 0.2, (0.25, 0.2), "uniform", mst.MST_PATH_AUTO, 0.0),
          (1100, 768, 0.04, (0.04, 0.1), "uniform", mst.MST_PATH_DENSE, 0.25)]
STREAMS = {"all on one": [0] * 11, "in turn on two": [j % 2 for j in range(11)], "a run, then others": [0, 0, 0, 1, 1, 2, 0, 0, 1, 3, 0],
           "nine on the second": [0] + [1] * 9 + [0]}


@pytest.mark.parametrize("R", [0.25, 0.0, 1.0])
@pytest.mark.parametrize("share", list(STREAMS))
def test_layers_that_share_a_stream(share, R):
    T = 70
    rigs, state, XY = [], [], []
    for j, (O, I, d, _, mask, path, lam) in enumerate(LAYERS):
        W, M = synth.make_layer(41, j + 1, I, O, d, mask)
        mst.mst_heavy_rows(2 if mask == "powerlaw" else 1)
        try:
            rigs.append(Rig(W, M, T, cap=O * I))
        finally:
            mst.mst_heavy_rows(1)
        rigs[j].layer.set_path(path)
        rigs[j].layer.set_prune_lambda(lam)
        X, dY = synth.make_activations(41, j + 1, T, I, O)
        state.append((W, M))
        XY.append((X, dY))
        rigs[j].fwd(X)                                       # (the next update asks which path served the last call)
    assert rigs[1].layer.format_stats()["heavy_rows"] > 0
    pool = [torch.cuda.Stream() for _ in range(4)]
    for update in range(2):
        G = [synth.normal(43 + update, j + 1, W.shape) for j, (W, _) in enumerate(state)]
        seeds, targets = [900 + 20 * update + j for j in range(len(rigs))], [x[3][update] for x in LAYERS]
        Gd = [dev(g) for g in G]
        torch.cuda.synchronize()
        sts = mst.mst_mask_update_from_scores_multi([r.layer for r in rigs], Gd, targets, 0.3, R, seeds, [r.ws for r in rigs],
                                                    [pool[u] for u in STREAMS[share]])
        torch.cuda.synchronize()
        for j, rig in enumerate(rigs):
            print("layer", j, "update", update, share, R, flush=True)
            W, M = state[j]
            ref = omg.update(W, M, G[j], targets[j], 0.3, R, seeds[j], prune_lambda=float(np.float32(LAYERS[j][6])))
            c = ref["counts"]
            assert (sts[j]["n_prune"], sts[j]["n_grad"], sts[j]["n_rand"]) == (c["n_prune"], c["n_grad"], c["n_rand"])
            assert sts[j]["nnz_after"] == c["nnz_target"] == rig.layer.nnz
            We, Me = rig.export()
            np.testing.assert_array_equal(Me, ref["M"])
            np.testing.assert_array_equal(We, ref["W"])
            np.testing.assert_array_equal(rig.indices(), np.flatnonzero(ref["M"].reshape(-1)))
            vals = rig.layer.values()
            vals.add_(0.01)                                  # grown weights take part in products and in the next update
            rig.layer.sync_values()
            W = np.where(ref["M"] != 0, ref["W"] + np.float32(0.01), np.float32(0)).astype(np.float32)
            state[j] = (W, ref["M"])
            X, dY = XY[j]
            for path in (LAYERS[j][5], mst.MST_PATH_SPARSE):
                rig.layer.set_path(path)
                assert rel_err(rig.bwd_weight(dY, X), opr.fc_bwd_weight(dY, X, ref["M"])) <= TOL      # (builds views that are not there)
                assert rel_err(rig.fwd(X), opr.fc_fwd(X, W, ref["M"])) <= TOL
                assert rel_err(rig.bwd_input(dY), opr.fc_bwd_input(dY, W, ref["M"])) <= TOL
            rig.layer.set_path(LAYERS[j][5])
