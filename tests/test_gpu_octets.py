"""Which rows of the index views share an octet: by total length, or halved by their lengths in the parts of the chunks,
whichever stores fewer pairs.  The stored slots of both views against a plain model of the two orders, and the products against
the oracle (App. Eq. (1) and its gradients), over views of one to nine chunks, cut-off row blocks, empty rows, rows of very
different lengths and rows that lie in one chunk alone."""
import numpy as np
import pytest

import paper_2408_11746_amd as mst
import synth
from oracle import products as opr

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
from gpu_util import Rig, dev, rel_err  # noqa: E402

# fixed-order fp32 sums of at most 600 terms of random sign: about sqrt(600) 2^-24 = 1.5e-6 of such a sum (see test_gpu_walk.py)
TOL = 2e-6


def _chunk(K):
    """contraction indices of a chunk"""
    n = -(-K // 640)
    per = -(-K // n)
    sub = -(-per // 128)
    return sub * (-(-(-(-per // sub)) // 4) * 4)


def _pairs(L, order):
    groups = L[order].reshape(16, 8, -1)
    return int(((groups.max(axis=1) + 1) // 2).sum())


def _halved(L):
    """rows in the order of their octets"""
    n = L.shape[1]
    if n == 2:
        keys, sizes = [L[:, 0], L[:, 1]], [32, 8]
    elif n == 3:
        keys, sizes = [L[:, 0], L[:, 1], L[:, 2], L.sum(axis=1)], [64, 32, 16, 8]
    else:
        part = 4 * np.arange(n) // n
        keys, sizes = [L[:, part == q].sum(axis=1) for q in range(4)], [64, 32, 16, 8]
    groups = [np.arange(128)]
    for key, size in zip(keys, sizes):
        split = []
        for g in groups:
            g = g[np.lexsort((g, -key[g]))]
            split += [g[i:i + size] for i in range(0, g.size, size)]
        groups = split
    return np.concatenate(groups)


def _slots(M):
    """stored entry slots of the view of rows of M, no row of it spread"""
    R, K = M.shape
    KC, total = _chunk(K), 0
    n = -(-K // KC)
    P = np.zeros((-(-R // 128) * 128, n * KC), dtype=np.int64)
    P[:R, :K] = M
    for block in P.reshape(-1, 128, n, KC).sum(axis=3):
        ranked = _pairs(block, np.lexsort((np.arange(128), -block.sum(axis=1))))
        total += min(ranked, _pairs(block, _halved(block))) if n > 1 else ranked
    return 16 * total


@pytest.mark.parametrize("O,I,T,density,kind", [
    (128, 640, 64, 0.05, "uniform"), (129, 1280, 65, 0.02, "uniform"), (300, 1281, 70, 0.05, "uniform"),
    (131, 2560, 64, 0.03, "uniform"), (1285, 3300, 40, 0.02, "uniform"), (77, 5120, 64, 0.02, "uniform"),
    (640, 641, 64, 0.04, "steep"), (256, 3000, 64, 0.05, "steep"), (256, 1920, 64, 0.04, "banded"),
])
def test_octets(O, I, T, density, kind):
    rng = np.random.default_rng([O, I])
    p = np.full((O, I), density)
    if kind == "steep":                       # some entries everywhere (an empty row may let another one spread), a few long rows
        p *= np.geomspace(4.0, 0.25, O)[rng.permutation(O)][:, None]
    if kind == "banded":                      # every row in one third of the indices
        p = 3 * density * (np.arange(I)[None, :] * 3 // I == rng.integers(0, 3, O)[:, None])
    M = (rng.random((O, I)) < p).astype(np.uint8)
    M[np.arange(O), rng.integers(0, I, O)] = 1
    M[rng.integers(0, O, I), np.arange(I)] = 1
    W = (rng.standard_normal((O, I)) * 0.02).astype(np.float32) * M
    X, dY = synth.make_activations(1, O, T, I, O)
    rig = Rig(W, M, T, cap=int(M.sum()))
    rig.layer.set_path(mst.MST_PATH_SPARSE)
    st = rig.layer.format_stats()
    # (empty rows past the end of the last block let a row of it spread where that is shorter)
    want = {"row_view_slots": _slots(M), "col_view_slots": _slots(M.T)}
    for name, rows in (("row_view_slots", O), ("col_view_slots", I)):
        exact = rows % 128 == 0 or rows % 128 > 121
        assert (st[name] == want[name]) if exact else (st[name] <= 1.1 * want[name]), (name, st, want)
    assert rel_err(rig.fwd(X), opr.fc_fwd(X, W, M)) <= TOL
    assert rel_err(rig.bwd_input(dY), opr.fc_bwd_input(dY, W, M)) <= TOL
    assert rel_err(rig.bwd_weight(dY, X), opr.fc_bwd_weight(dY, X, M)) <= TOL
