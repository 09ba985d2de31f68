"""Y and dX of bfloat16 activations on whole 256 x 256 tiles, which read the weights' two bfloat16 parts from planes kept
beside the dense copy: at one, two and more k steps, and after every way in which the weights change.  Against the oracle
(App. Eq. (1) and its gradient); two parts leave at most 2^-17 of a term (rel_err measures against the largest output)."""
import numpy as np
import pytest

import paper_2408_11746_amd as mst
import synth
from oracle import products as opr

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
from gpu_util import Rig, DEV, dev, rel_err  # noqa: E402

PARTS = 2e-5


@pytest.fixture(autouse=True)
def whole_tiles():
    mst.mst_gemm_force_fp32_mfma(256)                        # (products this small would go to other kernels)
    yield
    mst.mst_gemm_force_fp32_mfma(0)


def _layer(T, I, O, seed=31):
    W, M = synth.make_layer(seed, 1, I, O, 0.4, "uniform")
    Xf, dYf, xb, yb = synth.make_activations(seed, 2, T, I, O, "bf16")
    rig = Rig(W, M, T, cap=O * I)
    rig.layer.set_path(mst.MST_PATH_DENSE)
    return rig, xb.view(np.int16), yb.view(np.int16), opr.fc_fwd(Xf, W, M), opr.fc_bwd_input(dYf, W, M), (Xf, dYf)


def _check(rig, X, dY, Y1, dX1, scale, what):
    assert rel_err(rig.fwd(X, mst.MST_BF16), scale * Y1) <= PARTS, what
    assert (mst.mst_gemm_last_tile() == 256) == (rig.O % 256 == 0), what
    assert rel_err(rig.bwd_input(dY, mst.MST_BF16), scale * dX1) <= PARTS, what
    assert (mst.mst_gemm_last_tile() == 256) == (rig.I % 256 == 0), what


@pytest.mark.parametrize("T,I,O", [(256, 32, 256), (256, 64, 512), (512, 544, 256), (256, 256, 96), (768, 512, 768)])
def test_products_of_whole_tiles(T, I, O):
    print("case", T, I, O, flush=True)
    rig, X, dY, Y1, dX1, _ = _layer(T, I, O)
    _check(rig, X, dY, Y1, dX1, 1.0, "first")
    _check(rig, X, dY, Y1, dX1, 1.0, "second")


def test_planes_follow_the_weights():
    T, I, O = 256, 256, 512
    rig, X, dY, Y1, dX1, (Xf, dYf) = _layer(T, I, O)
    L = rig.layer
    _check(rig, X, dY, Y1, dX1, 1.0, "first")
    L.values().mul_(2.0)
    L.sync_values()
    _check(rig, X, dY, Y1, dX1, 2.0, "handed over")
    W, M = rig.export()
    L.load_dense(dev(2.0 * W), dev(M), rig.ws)
    L.values().mul_(2.0)
    L.sync_values()                                          # (no dense copy in use)
    _check(rig, X, dY, Y1, dX1, 8.0, "loaded anew")
    for density, views in ((0.6, False), (0.02, True), (0.5, False)):
        L.set_path(mst.MST_PATH_SPARSE if views else mst.MST_PATH_DENSE)
        mst.mst_mask_update(L, dev(dY), dev(X), T, density, 0.3, 0.25, 5, rig.ws, mst.MST_BF16)
        L.set_path(mst.MST_PATH_DENSE)
        L.values().add_(0.01)                                # grown weights take part
        L.sync_values()
        torch.cuda.synchronize()
        W, M = rig.export()
        _check(rig, X, dY, opr.fc_fwd(Xf, W, M), opr.fc_bwd_input(dYf, W, M), 1.0, density)


def test_replays_of_a_recorded_handover_reach_planes_read_between_them():
    """A hand-over recorded while only the dense copy is in use; products read the planes for the first time between its
    replays.  And a recorded product sees values loaded anew once the dense copy has been made from them."""
    T, I, O = 256, 256, 256
    rig, X, dY, Y1, dX1, _ = _layer(T, I, O)
    L = rig.layer
    rig.fwd(X[:100], mst.MST_BF16)                           # a batch of no whole tiles: the dense copy alone
    graph, side = torch.cuda.CUDAGraph(), torch.cuda.Stream()
    torch.cuda.synchronize()
    with torch.cuda.graph(graph, stream=side):
        L.values().mul_(2.0)
        L.sync_values(side)
    for k in range(3):
        graph.replay()
        torch.cuda.synchronize()
        if k == 0:
            assert rel_err(rig.fwd(X, mst.MST_BF16), 2.0 * Y1) <= PARTS
        else:
            _check(rig, X, dY, Y1, dX1, 2.0 ** (k + 1), k)
    Xd, Yg = dev(X), torch.empty((T, O), dtype=torch.float32, device=DEV)
    product = torch.cuda.CUDAGraph()
    with torch.cuda.graph(product, stream=side):
        mst.mst_sparse_fc_fwd(L, Xd, Yg, T, mst.MST_BF16, side)
    for scale in (1.0, 4.0):
        W, M = rig.export()
        L.load_dense(dev(scale / 8.0 * W if scale == 1.0 else 4.0 * W), dev(M), rig.ws)
        rig.fwd(X[:100], mst.MST_BF16)
        product.replay()
        torch.cuda.synchronize()
        assert rel_err(Yg.cpu().numpy(), scale * Y1) <= PARTS, scale


@pytest.mark.parametrize("first", ["recorded", "eager"])
def test_products_of_two_streams_find_whole_planes(first):
    """The planes are made by a product on a busy stream; a product on another stream, issued after that call returned and
    ordered after the loading of the weights alone, reads them.  Also where the very first product was recorded only."""
    T, I, O = 256, 512, 512
    rig, X, dY, Y1, dX1, _ = _layer(T, I, O)
    L, a, b = rig.layer, torch.cuda.Stream(), torch.cuda.Stream()
    rig.fwd(X[:100], mst.MST_BF16)                           # the dense copy alone
    L.buf[-8 * O * I:].fill_(0xFF)                           # the planes, two arrays at the end of the buffer: NaN until they are made
    Xd, dYd = dev(X), dev(dY)
    Y, dX = (torch.full((T, n), 7.0, dtype=torch.float32, device=DEV) for n in (O, I))
    Yg, graph = torch.full((T, O), 7.0, dtype=torch.float32, device=DEV), torch.cuda.CUDAGraph()
    torch.cuda.synchronize()
    if first == "recorded":
        with torch.cuda.graph(graph, stream=a):
            mst.mst_sparse_fc_fwd(L, Xd, Yg, T, mst.MST_BF16, a)
    with torch.cuda.stream(a):
        torch.cuda._sleep(100_000_000)                       # (some 50 ms)
    mst.mst_sparse_fc_fwd(L, Xd, Y, T, mst.MST_BF16, a)
    mst.mst_sparse_fc_bwd_input(L, dYd, dX, T, mst.MST_BF16, b)
    torch.cuda.synchronize()
    assert rel_err(dX.cpu().numpy(), dX1) <= PARTS
    assert rel_err(Y.cpu().numpy(), Y1) <= PARTS
    if first == "recorded":
        for _ in range(2):
            graph.replay()
            torch.cuda.synchronize()
            assert rel_err(Yg.cpu().numpy(), Y1) <= PARTS


def test_a_handover_recorded_for_fp32_activations_leaves_the_planes_alone():
    """A layer that works on fp32 activations records its hand-over without the planes.  Products of bfloat16 activations that
    come after all, eager and recorded, see the values of every replay and of every eager hand-over."""
    T, I, O = 256, 512, 512
    rig, X, dY, Y1, dX1, (Xf, _) = _layer(T, I, O)
    L, side = rig.layer, torch.cuda.Stream()
    assert rel_err(rig.fwd(Xf), Y1) <= 1e-4                  # the dense copy alone
    L.buf[-8 * O * I:].fill_(0xFF)
    handover, product = torch.cuda.CUDAGraph(), torch.cuda.CUDAGraph()
    torch.cuda.synchronize()
    with torch.cuda.graph(handover, stream=side):
        L.values().mul_(2.0)
        L.sync_values(side)
    for _ in range(2):
        handover.replay()
        torch.cuda.synchronize()
    L.sync_values()
    torch.cuda.synchronize()
    assert bool((L.buf[-8 * O * I:] == 0xFF).all())
    assert rel_err(rig.fwd(Xf), 4.0 * Y1) <= 1e-4
    _check(rig, X, dY, Y1, dX1, 4.0, "first")
    Xd, Yg = dev(X), torch.empty((T, O), dtype=torch.float32, device=DEV)
    torch.cuda.synchronize()
    with torch.cuda.graph(product, stream=side):
        mst.mst_sparse_fc_fwd(L, Xd, Yg, T, mst.MST_BF16, side)
    for k, scale in ((3, 8.0), (4, 16.0)):
        handover.replay()
        product.replay()
        torch.cuda.synchronize()
        assert rel_err(Yg.cpu().numpy(), scale * Y1) <= PARTS, k
        _check(rig, X, dY, Y1, dX1, scale, k)
        L.values().mul_(0.5)
        L.sync_values()
        product.replay()
        torch.cuda.synchronize()
        assert rel_err(Yg.cpu().numpy(), 0.5 * scale * Y1) <= PARTS, k
        _check(rig, X, dY, Y1, dX1, 0.5 * scale, k)
        L.values().mul_(2.0)
        L.sync_values()


def test_products_of_two_streams_find_the_planes_of_weights_loaded_anew():
    """As above for planes that products have read before: the first product after a loading makes them again together with
    the dense copy."""
    T, I, O = 256, 512, 512
    rig, X, dY, Y1, dX1, _ = _layer(T, I, O)
    L, a, b = rig.layer, torch.cuda.Stream(), torch.cuda.Stream()
    _check(rig, X, dY, Y1, dX1, 1.0, "first")
    W, M = rig.export()
    L.load_dense(dev(4.0 * W), dev(M), rig.ws)
    Xd, dYd = dev(X), dev(dY)
    Y, dX = (torch.full((T, n), 7.0, dtype=torch.float32, device=DEV) for n in (O, I))
    torch.cuda.synchronize()
    with torch.cuda.stream(a):
        torch.cuda._sleep(100_000_000)                       # (some 50 ms)
    mst.mst_sparse_fc_fwd(L, Xd, Y, T, mst.MST_BF16, a)
    mst.mst_sparse_fc_bwd_input(L, dYd, dX, T, mst.MST_BF16, b)
    torch.cuda.synchronize()
    assert rel_err(dX.cpu().numpy(), 4.0 * dX1) <= PARTS
    assert rel_err(Y.cpu().numpy(), 4.0 * Y1) <= PARTS


def test_a_recorded_product_makes_the_planes_once():
    """The first product after a loading makes the planes together with the dense copy where a product has read them before,
    by themselves otherwise; recorded, it has as many nodes either way, and its replays see the values loaded."""
    import ctypes
    hip = ctypes.CDLL(next(line.split()[-1] for line in open("/proc/self/maps") if "libamdhip64" in line))     # (the one in use)
    T, I, O = 256, 256, 512
    nodes = []
    for read_before in (False, True):
        rig, X, dY, Y1, dX1, _ = _layer(T, I, O)
        L, side = rig.layer, torch.cuda.Stream()
        if read_before:
            _check(rig, X, dY, Y1, dX1, 1.0, "first")
            W, M = rig.export()
            L.load_dense(dev(W), dev(M), rig.ws)
        Xd, Y = dev(X), torch.empty((T, O), dtype=torch.float32, device=DEV)
        graph = torch.cuda.CUDAGraph(keep_graph=True)
        torch.cuda.synchronize()
        with torch.cuda.graph(graph, stream=side):
            mst.mst_sparse_fc_fwd(L, Xd, Y, T, mst.MST_BF16, side)
        n = ctypes.c_size_t()
        assert hip.hipGraphGetNodes(ctypes.c_void_p(graph.raw_cuda_graph()), None, ctypes.byref(n)) == 0
        nodes.append(n.value)
        for _ in range(3):
            graph.replay()
            torch.cuda.synchronize()
            assert rel_err(Y.cpu().numpy(), Y1) <= PARTS
    assert nodes[0] == nodes[1]
