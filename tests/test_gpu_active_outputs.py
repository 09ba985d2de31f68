"""The weight gradient on the dense matrix cores that writes the active positions alone (dW of App. Eq. (1)'s gradients): every tile, one
and several partial outputs, rows that end inside a word of 32 columns, tiles past the last row and column, empty and full rows, few and
all positions.  Small whole numbers, whose products and sums are exact in every kernel: the result has to be the exact one."""
import threading

import numpy as np
import pytest

import paper_2408_11746_amd as mst

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
from gpu_util import Rig, DEV  # noqa: E402


@pytest.fixture(autouse=True)
def automatic():
    yield
    mst.mst_gemm_force_fp32_mfma(0)


def _numbers(T, n, act, seed):
    gen = torch.Generator(device=DEV)
    gen.manual_seed(seed)
    return torch.randint(-3, 4, (T, n), generator=gen, device=DEV).to(torch.bfloat16 if act == mst.MST_BF16 else torch.float32).contiguous()


def _mask(O, I, density, seed):
    M = (np.random.default_rng(seed).random((O, I)) < density).astype(np.uint8)
    M[O // 2] = 0
    M[O - 1] = 0
    M[0] = 1
    M[1, :33] = 1
    M[2, I - 1] = 1
    return M


def _check(rig, dY, X, act, dW=None):
    if dW is None:
        dW = torch.full((rig.layer.nnz + 64,), 7.0, device=DEV)
        mst.mst_sparse_fc_bwd_weight(rig.layer, dY, X, dW, X.shape[0], rig.ws, act)
    G = dY.double().cpu().numpy().T @ X.double().cpu().numpy()
    dW = dW.cpu().numpy()
    n = rig.layer.nnz
    assert np.array_equal(dW[:n], G.ravel()[rig.indices()])
    assert np.all(dW[n:] == 7.0)


def _rig(O, I, T, density, seed=5):
    M = _mask(O, I, density, seed)
    rig = Rig(M * np.float32(0.5), M, T, cap=O * I)
    rig.layer.set_path(mst.MST_PATH_DENSE)
    return rig


@pytest.mark.parametrize("density", [0.01, 0.2, 1.0])
@pytest.mark.parametrize("O,I,T,act,tile", [
    (256, 256, 64, "f32", 256), (512, 256, 2048, "f32", 256), (3072, 768, 1024, "f32", 256), (2560, 2560, 1024, "f32", 256),
    (128, 128, 64, "f32", 128), (256, 384, 96, "f32", 128), (384, 1152, 2048, "f32", 128),
    (8, 16, 1, "bf16", 256), (264, 272, 33, "bf16", 256), (520, 48, 2049, "bf16", 256), (1288, 1040, 3000, "bf16", 256), (2048, 1040, 97, "bf16", 256),
    (264, 264, 96, "bf16", 256), (264, 264, 33, "f32", 1128), (130, 40, 1, "f32", 1128), (1300, 520, 2048, "f32", 1128), (2500, 1000, 3001, "f32", 1128),
    (2500, 1000, 130, "f32", 1128), (300, 270, 64, "f32", 0), (96, 80, 64, "bf16", 64)])
def test_exact_gradient(O, I, T, act, tile, density):
    print("case", O, I, T, act, tile, density, flush=True)
    kind = mst.MST_BF16 if act == "bf16" else mst.MST_F32
    mst.mst_gemm_force_fp32_mfma(tile)
    rig = _rig(O, I, T, density)
    X, dY = _numbers(T, I, kind, 1), _numbers(T, O, kind, 2)
    _check(rig, dY, X, kind)


def _writes_active(rig, dY, X, act):
    """Did the product write active positions alone?  By what it leaves in the workspace: whole outputs (one or several partial ones, or the
    one that is gathered from), or no more than the active positions of the partial ones."""
    ws = rig.ws[:rig.ws.numel() & ~3].view(torch.int32)
    ws.fill_(0x5A5A5A5A)
    dW = torch.full((rig.layer.nnz + 64,), 7.0, device=DEV)
    mst.mst_sparse_fc_bwd_weight(rig.layer, dY, X, dW, X.shape[0], rig.ws, act)
    _check(rig, dY, X, act, dW)
    written, n, nnz = int((ws != 0x5A5A5A5A).sum()), rig.O * rig.I, rig.layer.nnz
    assert nnz < n and (written % nnz == 0 and written // nnz <= 8 or written % n == 0 and 1 <= written // n <= 8), (written, nnz, n)
    return written == 0 or written % n != 0


@pytest.mark.parametrize("density", [0.01, 0.2, 1.0])
@pytest.mark.parametrize("O,I,T,act,tile", [
    (256, 256, 64, "f32", 256), (512, 256, 2048, "f32", 256), (3072, 768, 1024, "f32", 256), (2560, 2560, 1024, "f32", 256),
    (128, 128, 64, "f32", 128), (256, 384, 192, "f32", 128), (384, 1152, 2048, "f32", 128), (1664, 1280, 128, "f32", 128),
    (64, 64, 1, "bf16", 256), (264, 272, 33, "bf16", 256), (520, 48, 2049, "bf16", 256), (2048, 1040, 97, "bf16", 256), (40, 52432, 33, "bf16", 256),
    (264, 264, 33, "f32", 1128), (130, 40, 1, "f32", 1128), (2500, 1000, 3001, "f32", 1128), (256, 384, 96, "f32", 128), (300, 270, 64, "f32", 0), (96, 80, 64, "bf16", 64)])
def test_which_products_write_the_active_positions(O, I, T, act, tile, density):
    """Small layers with many active weights stay on whole outputs, and so do rows of no whole eights, the streaming kernels and batches that
    are no whole steps of the pinned kernel; the others write the active positions alone."""
    print("case", O, I, T, act, tile, density, flush=True)
    kind = mst.MST_BF16 if act == "bf16" else mst.MST_F32
    mst.mst_gemm_force_fp32_mfma(tile)
    rig = _rig(O, I, T, density)
    X, dY = _numbers(T, I, kind, 1), _numbers(T, O, kind, 2)
    can, nnz = tile in (256, 1128) or (tile == 128 and T % 64 == 0), rig.layer.nnz
    assert _writes_active(rig, dY, X, kind) == (can and (4 * nnz <= O * I or O * I >= 1 << 21))


def test_infinite_operands_of_the_full_precision_kernel():
    """the positions that full fp32 sums make infinite or no number, and the others as the whole dense gradient has them"""
    O, I, T, act = 264, 264, 64, mst.MST_F32
    mst.mst_gemm_force_fp32_mfma(1128)
    rig = _rig(O, I, T, 0.2)
    X, dY = _numbers(T, I, act, 1), _numbers(T, O, act, 2)
    X[5, 0], X[6, 0], X[7, 33], dY[9, 2] = float("inf"), float("-inf"), float("inf"), float("nan")
    dW, G = torch.full((rig.layer.nnz + 64,), 7.0, device=DEV), torch.empty((O, I), device=DEV)
    mst.mst_sparse_fc_bwd_weight(rig.layer, dY, X, dW, T, rig.ws, act)
    mst.mst_dense_grad(dY, X, G, T, O, I, act, rig.ws)
    want, dW = G.cpu().numpy().ravel()[rig.indices()], dW.cpu().numpy()
    assert np.isnan(want).any() and np.isinf(want).any()
    assert np.array_equal(dW[:-64], want, equal_nan=True) and np.all(dW[-64:] == 7.0)


@pytest.mark.parametrize("path", [mst.MST_PATH_DENSE, mst.MST_PATH_AUTO])
@pytest.mark.parametrize("O,I,kind", [(1024, 256, "f32"), (776, 272, "bf16"), (1048, 224, "bf16")])
@pytest.mark.parametrize("read_before", [True, False])
def test_updates_take_the_words_along(read_before, O, I, kind, path):
    """Eager and recorded products before and behind eager and recorded updates of the active set, updates that rebuild the views and
    updates that do not."""
    T, act = 512, mst.MST_BF16 if kind == "bf16" else mst.MST_F32
    mst.mst_gemm_force_fp32_mfma(256)
    rig = _rig(O, I, T, 0.1)
    rig.layer.set_path(path)
    L, side = rig.layer, torch.cuda.Stream()
    X, dY = _numbers(T, I, act, 1), _numbers(T, O, act, 2)
    score = torch.randn(O, I, device=DEV)
    density = L.nnz / (O * I)
    if read_before:
        _check(rig, dY, X, act)
    mst.mst_mask_update_from_scores(L, score, density, 0.3, 0.25, 11, rig.ws)
    if read_before:
        _check(rig, dY, X, act)
    update, product = torch.cuda.CUDAGraph(), torch.cuda.CUDAGraph()
    dW = torch.full((L.nnz + 64,), 7.0, device=DEV)
    torch.cuda.synchronize()
    with torch.cuda.graph(update, stream=side):
        mst.mst_mask_update_from_scores(L, score, density, 0.3, 0.25, 12, rig.ws, side)
    with torch.cuda.graph(product, stream=side):
        mst.mst_sparse_fc_bwd_weight(L, dY, X, dW, T, rig.ws, act, side)
    for _ in range(3):
        update.replay()
        torch.cuda.synchronize()
        _check(rig, dY, X, act)
        dW.fill_(7.0)
        product.replay()
        torch.cuda.synchronize()
        _check(rig, dY, X, act, dW)
    mst.mst_mask_update_from_scores(L, score, density, 0.3, 0.25, 13, rig.ws)
    _check(rig, dY, X, act)
    product.replay()
    torch.cuda.synchronize()
    _check(rig, dY, X, act, dW)


def test_two_streams_behind_an_update_that_left_the_words():
    O, I, T, act = 1024, 256, 512, mst.MST_F32
    mst.mst_gemm_force_fp32_mfma(256)
    rig = _rig(O, I, T, 0.1)
    L, a, b = rig.layer, torch.cuda.Stream(), torch.cuda.Stream()
    X, dY = _numbers(T, I, act, 1), _numbers(T, O, act, 2)
    mst.mst_mask_update_from_scores(L, torch.randn(O, I, device=DEV), L.nnz / (O * I), 0.3, 0.25, 11, rig.ws)
    out = [torch.full((L.nnz + 64,), 7.0, device=DEV) for _ in range(2)]
    ws = torch.empty_like(rig.ws)
    torch.cuda.synchronize()
    with torch.cuda.stream(a):
        torch.cuda._sleep(10_000_000)
    mst.mst_sparse_fc_bwd_weight(L, dY, X, out[0], T, rig.ws, act, a)
    mst.mst_sparse_fc_bwd_weight(L, dY, X, out[1], T, ws, act, b)
    torch.cuda.synchronize()
    for dW in out:
        _check(rig, dY, X, act, dW)


def test_two_threads_behind_an_update_that_left_the_words():
    """The words are said to be there once they are: a product of another thread that comes while the first one waits for them does not read
    those of the mask before."""
    O, I, T, act = 1024, 256, 512, mst.MST_F32
    mst.mst_gemm_force_fp32_mfma(256)
    rig = _rig(O, I, T, 0.1)
    L, a, b = rig.layer, torch.cuda.Stream(), torch.cuda.Stream()
    X, dY = _numbers(T, I, act, 1), _numbers(T, O, act, 2)
    mst.mst_mask_update_from_scores(L, torch.randn(O, I, device=DEV), L.nnz / (O * I), 0.3, 0.25, 11, rig.ws)
    out = [torch.full((L.nnz + 64,), 7.0, device=DEV) for _ in range(2)]
    ws = torch.empty_like(rig.ws)
    begun = torch.cuda.Event()
    torch.cuda.synchronize()
    with torch.cuda.stream(a):
        torch.cuda._sleep(1_000_000_000)                 # (0.4 s)
        begun.record()
    first = threading.Thread(target=mst.mst_sparse_fc_bwd_weight, args=(L, dY, X, out[0], T, rig.ws, act, a))
    first.start()
    first.join(0.02)
    assert not begun.query()                                  # (the first thread's words are still to be made)
    mst.mst_sparse_fc_bwd_weight(L, dY, X, out[1], T, ws, act, b)
    first.join()
    torch.cuda.synchronize()
    for dW in out:
        _check(rig, dY, X, act, dW)


@pytest.mark.parametrize("O,I", [(1024, 256), (776, 272)])
@pytest.mark.parametrize("updates", [1, 8, 9, 20])
def test_updates_that_make_the_words_for_nobody(updates, O, I):
    """Behind eight updates that nothing read the words of, an update leaves them to the next product.  A recorded product, which cannot make
    them, shows which: it writes active positions alone where they are there.  Then it is read by its replays, and every update makes them."""
    T, act, side = 512, mst.MST_BF16, torch.cuda.Stream()
    mst.mst_gemm_force_fp32_mfma(256)
    rig = _rig(O, I, T, 0.1)
    L = rig.layer
    X, dY = _numbers(T, I, act, 1), _numbers(T, O, act, 2)
    score = torch.randn(O, I, device=DEV)
    density = L.nnz / (O * I)
    assert _writes_active(rig, dY, X, act)
    for k in range(updates):
        mst.mst_mask_update_from_scores(L, score, density, 0.3, 0.25, 20 + k, rig.ws)
    dW = torch.full((L.nnz + 64,), 7.0, device=DEV)
    ws = rig.ws[:rig.ws.numel() & ~3].view(torch.int32)

    def record():
        graph = torch.cuda.CUDAGraph()
        torch.cuda.synchronize()
        with torch.cuda.graph(graph, stream=side):
            mst.mst_sparse_fc_bwd_weight(L, dY, X, dW, T, rig.ws, act, side)
        return graph

    def replay(graph):
        ws.fill_(0x5A5A5A5A)
        dW.fill_(7.0)
        graph.replay()
        torch.cuda.synchronize()
        _check(rig, dY, X, act, dW)
        written = int((ws != 0x5A5A5A5A).sum())
        return written == 0 or written % (O * I) != 0

    graph = record()
    for _ in range(3):
        assert replay(graph) == (updates <= 8)
    assert _writes_active(rig, dY, X, act)                    # (an eager one makes them)
    graph = record()
    for k in range(12):                                       # (the recorded product has read them)
        assert replay(graph)
        mst.mst_mask_update_from_scores(L, score, density, 0.3, 0.25, 50 + k, rig.ws)
    assert replay(graph) and _writes_active(rig, dY, X, act)


@pytest.mark.parametrize("O,I", [(512, 512), (1280, 320), (64, 2048)])
def test_a_handover_that_packs(O, I):
    """Values handed over, eagerly and by a recording, before and behind an update, while products read the packed weights: those, the
    dense copy (products pinned to a kernel that reads it) and a view that is walked for the first time later all hold them."""
    T, act, side = 4096, mst.MST_F32, torch.cuda.Stream()
    rig = _rig(O, I, T, 0.08)
    L = rig.layer
    X = _numbers(T, I, act, 1)
    Y = torch.empty((T, O), device=DEV)
    fill = torch.empty(O * I, device=DEV)                     # whole numbers that three and two bfloat16 parts hold

    def product(tile, path=mst.MST_PATH_DENSE):
        L.set_path(path)
        mst.mst_gemm_force_fp32_mfma(tile)
        Y.fill_(7.0)
        mst.mst_sparse_fc_fwd(L, X, Y, T, act)
        torch.cuda.synchronize()
        return Y.double()

    def check(values):
        W = torch.zeros(O * I, dtype=torch.float64, device=DEV)
        W[torch.from_numpy(rig.indices()).to(DEV).long()] = values.double()
        want = X.double() @ W.view(O, I).T
        assert torch.equal(product(24), want)
        assert mst.mst_gemm_last_tile() == 24
        assert torch.equal(product(128 if O % 128 == 0 and I % 128 == 0 else 1032), want)
        return want

    def hand_over(scale):
        n = L.nnz
        L.values().copy_((torch.arange(n, device=DEV) % 15 - 7) * scale)
        L.sync_values()
        return L.values().clone()

    hand_over(1.0)
    product(24)                                               # packed from now on
    check(hand_over(2.0))
    graph = torch.cuda.CUDAGraph()
    torch.cuda.synchronize()
    with torch.cuda.graph(graph, stream=side):
        L.values().copy_(fill[:L.nnz])
        L.sync_values(side)
    for k in range(3):
        fill.copy_((torch.arange(O * I, device=DEV) + k) % 13 - 6)
        graph.replay()
        torch.cuda.synchronize()
        check(fill[:L.nnz])
        check(hand_over(1.0 + k))
    mst.mst_mask_update_from_scores(L, torch.randn(O, I, device=DEV), L.nnz / (O * I), 0.3, 0.25, 11, rig.ws)
    product(24)
    check(hand_over(4.0))
    fill.copy_(torch.arange(O * I, device=DEV) % 11 - 5)
    graph.replay()
    torch.cuda.synchronize()
    check(fill[:L.nnz])
    want = check(hand_over(3.0))
    L.values().zero_()                                        # (not handed over)
    assert torch.equal(product(0, mst.MST_PATH_SPARSE), want)
