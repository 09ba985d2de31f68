"""The dense products of any shape at full fp32 precision (three bfloat16 parts per fp32 operand): Y, dX
and the dense gradient of a dense layer at the edges of the 32 x 32, 64 x 64 and 128 x 128 tiles and of the k steps
of 16, 32 and 64, staged through LDS and streamed into registers, fp32 and bfloat16 activations, and the
bfloat16 dense gradient on rows that are no multiple of anything.  Against the oracle (App. Eq. (1) and its
gradients) at the precision of fp32 sums, far inside what two parts per operand would reach."""
import numpy as np
import pytest

import paper_2408_11746_amd as mst
import synth
from oracle import products as opr

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
from gpu_util import Rig, DEV, dev, rel_err  # noqa: E402

FP32 = 2e-6          # max error over max value of an fp32 sum of up to 2000 terms
SHAPES = [(1, 1, 1), (63, 65, 127), (64, 64, 64), (129, 33, 130), (130, 257, 63), (200, 191, 321), (257, 2000, 66), (2000, 66, 129)]


@pytest.mark.parametrize("T,I,O", SHAPES)
@pytest.mark.parametrize("mode", [1032, 1064, 1096, 1128])
def test_fp32_operands_of_any_shape(T, I, O, mode):
    print("case", T, I, O, mode, flush=True)
    X, dY = synth.make_activations(61, 2, T, I, O)
    X = (X * np.exp2(synth.normal(61, 7, X.shape) * 3)).astype(np.float32)       # all three parts matter
    W = synth.normal(61, 3, (O, I), 0.02)
    M = np.ones((O, I), np.uint8)
    rig = Rig(W, M, T, cap=O * I)
    rig.layer.set_path(mst.MST_PATH_DENSE)
    G = torch.full((O, I), float("nan"), dtype=torch.float32, device=DEV)
    try:
        mst.mst_gemm_force_fp32_mfma(mode)
        Y, dX = rig.fwd(X), rig.bwd_input(dY)
        mst.mst_dense_grad(dev(dY), dev(X), G, T, O, I, mst.MST_F32, rig.ws)      # with room to split the token range
        torch.cuda.synchronize()
        G0 = torch.full((O, I), float("nan"), dtype=torch.float32, device=DEV)
        mst.mst_dense_grad(dev(dY), dev(X), G0, T, O, I, mst.MST_F32, None)
        torch.cuda.synchronize()
    finally:
        mst.mst_gemm_force_fp32_mfma(0)
    assert rel_err(Y, opr.fc_fwd(X, W, M)) <= FP32
    assert rel_err(dX, opr.fc_bwd_input(dY, W, M)) <= FP32
    assert rel_err(G.cpu().numpy(), opr.dense_grad(dY, X)) <= FP32
    assert rel_err(G0.cpu().numpy(), opr.dense_grad(dY, X)) <= FP32


@pytest.mark.parametrize("T,I,O", SHAPES)
@pytest.mark.parametrize("mode", [1032, 1064, 1096, 1128])
def test_bfloat16_activations_of_any_shape(T, I, O, mode):
    print("case", T, I, O, mode, flush=True)
    Xf, dYf, xb, yb = synth.make_activations(62, 2, T, I, O, "bf16")
    W = synth.normal(62, 3, (O, I), 0.02)
    W = (W * np.exp2(synth.normal(62, 8, W.shape) * 3)).astype(np.float32)
    M = np.ones((O, I), np.uint8)
    rig = Rig(W, M, T, cap=O * I)
    rig.layer.set_path(mst.MST_PATH_DENSE)
    try:
        mst.mst_gemm_force_fp32_mfma(mode)
        Y, dX = rig.fwd(xb.view(np.int16), mst.MST_BF16), rig.bwd_input(yb.view(np.int16), mst.MST_BF16)
    finally:
        mst.mst_gemm_force_fp32_mfma(0)
    assert rel_err(Y, opr.fc_fwd(Xf, W, M)) <= FP32
    assert rel_err(dX, opr.fc_bwd_input(dYf, W, M)) <= FP32


@pytest.mark.parametrize("T,I,O", SHAPES + [(1027, 513, 255), (1984, 257, 320)])
@pytest.mark.parametrize("mode", [64, 128, 256])
def test_bfloat16_dense_gradient_of_any_shape(T, I, O, mode):
    print("case", T, I, O, mode, flush=True)
    Xf, dYf, xb, yb = synth.make_activations(62, 2, T, I, O, "bf16")
    X, dY = dev(xb.view(np.int16)), dev(yb.view(np.int16))
    ws = torch.empty(16 * O * I * 4 + 256, dtype=torch.uint8, device=DEV)
    ref = opr.dense_grad(dYf, Xf)
    try:
        mst.mst_gemm_force_fp32_mfma(mode)
        for area in (ws, None):                              # with room to split the token range, and without
            G = torch.full((O, I), float("nan"), dtype=torch.float32, device=DEV)
            mst.mst_dense_grad(dY, X, G, T, O, I, mst.MST_BF16, area)
            torch.cuda.synchronize()
            assert rel_err(G.cpu().numpy(), ref) <= FP32
    finally:
        mst.mst_gemm_force_fp32_mfma(0)


@pytest.mark.parametrize("act", [mst.MST_F32, mst.MST_BF16])
@pytest.mark.parametrize("mode", [1032, 1064, 1096, 1128])
def test_infinite_operands_as_fp32_products_give_them(mode, act):
    """The parts of an infinite value are NaN; the outputs are what fp32 products give: infinities, or NaN where
    two of opposite sign or an infinity and a zero meet, and every other output as without it."""
    T, I, O = 130, 190, 97
    print("case", T, I, O, mode, act, flush=True)
    X = synth.normal(63, 1, (T, I)).astype(np.float32)
    X.view(np.uint32)[...] &= 0xFFFF0000                     # (exact in bfloat16)
    W = synth.normal(63, 3, (O, I), 0.02).astype(np.float32)
    X[3, 7], X[129, 189], X[40, 5], X[40, 6], X[50, 9] = np.inf, -np.inf, np.inf, -np.inf, np.nan
    X[60, 11], W[5, 11] = np.inf, 0.0
    W[96, 100] = -np.inf
    rig = Rig(W, np.ones((O, I), np.uint8), T, cap=O * I)
    rig.layer.set_path(mst.MST_PATH_DENSE)
    try:
        mst.mst_gemm_force_fp32_mfma(mode)
        Y = rig.fwd(X if act == mst.MST_F32 else (X.view(np.uint32) >> 16).astype(np.int16), act)
    finally:
        mst.mst_gemm_force_fp32_mfma(0)
    with np.errstate(invalid="ignore"):
        ref = X.astype(np.float64) @ W.T.astype(np.float64)
    finite = np.isfinite(ref)
    assert 400 < (~finite).sum() < ref.size // 10 and np.isinf(ref).any() and np.isnan(ref).any()
    assert np.array_equal(np.isnan(Y), np.isnan(ref))
    assert np.array_equal(Y[np.isinf(ref)], ref[np.isinf(ref)].astype(np.float32))
    assert rel_err(Y[finite], ref[finite]) <= FP32


@pytest.mark.parametrize("act", [mst.MST_F32, mst.MST_BF16])
@pytest.mark.parametrize("mode", [1032, 1064, 1096, 1128])
def test_infinite_operands_of_the_input_gradient_and_the_dense_gradient(mode, act):
    """The same for dX and G, whose operands lie the other way (contraction index along the columns of one or
    both): infinities in dY, X and W at the edges of tiles and k steps."""
    T, I, O = 130, 97, 190
    print("case", T, I, O, mode, act, flush=True)
    X, dY = synth.normal(67, 1, (T, I)).astype(np.float32), synth.normal(67, 2, (T, O)).astype(np.float32)
    W = synth.normal(67, 3, (O, I), 0.02).astype(np.float32)
    dY[3, 7], dY[129, 189], dY[40, 5], dY[40, 6], dY[50, 9] = np.inf, -np.inf, np.inf, -np.inf, np.nan
    X[129, 96], X[64, 0], X[60, 11], dY[60, 12] = np.inf, -np.inf, np.inf, 0.0
    W[189, 64], W[11, 5], dY[61, 11] = -np.inf, np.inf, 0.0
    for a in (X, dY):
        a.view(np.uint32)[...] &= 0xFFFF0000                 # (exact in bfloat16; infinities and the NaN stay what they are)
    send = (lambda a: a) if act == mst.MST_F32 else (lambda a: (a.view(np.uint32) >> 16).astype(np.int16))
    rig = Rig(W, np.ones((O, I), np.uint8), T, cap=O * I)
    rig.layer.set_path(mst.MST_PATH_DENSE)
    G = {}
    try:
        mst.mst_gemm_force_fp32_mfma(mode)
        dX = rig.bwd_input(send(dY), act)
        for area in (rig.ws, None):                          # with room to split the token range, and without
            g = torch.full((O, I), 7.0, dtype=torch.float32, device=DEV)
            mst.mst_dense_grad(dev(send(dY)), dev(send(X)), g, T, O, I, act, area)
            torch.cuda.synchronize()
            G["G with" if area is not None else "G without"] = g.cpu().numpy()
    finally:
        mst.mst_gemm_force_fp32_mfma(0)
    with np.errstate(invalid="ignore"):
        refs = {"dX": dY.astype(np.float64) @ W.astype(np.float64)}
        refs["G with"] = refs["G without"] = dY.astype(np.float64).T @ X.astype(np.float64)
    for name, got in dict(G, dX=dX).items():
        ref = refs[name]
        finite = np.isfinite(ref)
        assert 300 < (~finite).sum() < ref.size // 4 and np.isinf(ref).any() and np.isnan(ref).any(), name
        assert np.array_equal(np.isnan(got), np.isnan(ref)), name
        assert np.array_equal(got[np.isinf(ref)], ref[np.isinf(ref)].astype(np.float32)), name
        assert rel_err(got[finite], ref[finite]) <= FP32, name


@pytest.mark.parametrize("mode", [1032, 1064, 1096, 1128])
def test_positive_operands_of_full_mantissas_leave_no_one_sided_error(mode):
    """Terms of one sign and 24 significant bits: whatever a product drops must not point one way, or it adds up over
    k.  Error in units of 2^-24 of the exact output.  Bounds: what the order of the fp32 sums leaves, about
    sqrt(additions in a row) of random sign with a small mean from the matrix cores' alignment; measured mean 0.3 on the
    streaming kernels (16 or 8 sums) and 1.4 through LDS (one sum), rms 1.7 and 10.  (Truncated parts: mean 0.8 and
    194; fp32 matrix instructions: rms 16.)"""
    T, I, O = 129, 4099, 130
    print("case", T, I, O, mode, flush=True)
    rng = np.random.default_rng(64)
    X, W = (1.0 + rng.random((T, I))).astype(np.float32), (1.0 + rng.random((O, I))).astype(np.float32)
    dY = (1.0 + rng.random((T, O))).astype(np.float32)
    rig = Rig(W, np.ones((O, I), np.uint8), T, cap=O * I)
    rig.layer.set_path(mst.MST_PATH_DENSE)
    G = torch.full((O, I), float("nan"), dtype=torch.float32, device=DEV)
    try:
        mst.mst_gemm_force_fp32_mfma(mode)
        Y, dX = rig.fwd(X), rig.bwd_input(dY)
        mst.mst_dense_grad(dev(dY), dev(X), G, T, O, I, mst.MST_F32, None)
        torch.cuda.synchronize()
    finally:
        mst.mst_gemm_force_fp32_mfma(0)
    X, W, dY = X.astype(np.float64), W.astype(np.float64), dY.astype(np.float64)
    mean, rms = (0.5, 2.5) if mode in (1032, 1096) else (3.0, 16.0)
    for name, got, ref in (("Y", Y, X @ W.T), ("dX", dX, dY @ W), ("G", G.cpu().numpy(), dY.T @ X)):
        e = (got / ref - 1.0) * 2.0 ** 24
        print(name, "mean %.2f rms %.2f" % (e.mean(), np.sqrt((e * e).mean())), flush=True)
        assert abs(e.mean()) <= mean and np.sqrt((e * e).mean()) <= rms, name


@pytest.mark.parametrize("mode", [1032, 1064, 1096, 1128])
def test_values_next_to_the_largest_finite_one(mode):
    """Their first part rounds to an infinity; the products are what fp32 gives."""
    T, I, O = 65, 100, 70
    print("case", T, I, O, mode, flush=True)
    X = synth.normal(65, 1, (T, I)).astype(np.float32)
    W = synth.normal(65, 3, (O, I), 0.02).astype(np.float32)
    X[3, 7], X[64, 99] = np.finfo(np.float32).max, -np.finfo(np.float32).max
    rig = Rig(W, np.ones((O, I), np.uint8), T, cap=O * I)
    rig.layer.set_path(mst.MST_PATH_DENSE)
    try:
        mst.mst_gemm_force_fp32_mfma(mode)
        Y = rig.fwd(X)
    finally:
        mst.mst_gemm_force_fp32_mfma(0)
    ref = X.astype(np.float64) @ W.T.astype(np.float64)
    for rows in ([3, 64], [t for t in range(T) if t not in (3, 64)]):
        assert rel_err(Y[rows], ref[rows]) <= FP32


@pytest.mark.parametrize("M,N,K", [(5000, 2040, 37), (5000, 2500, 37), (2561, 3970, 70), (12700, 1025, 33)])
def test_two_and_three_workgroups_on_a_cu(M, N, K):
    """128 x 128 tiles: 80, 100, 84 and 113 of them an XCD, in rounds of 96 or of 64, whichever is the shorter way; Y, dX and the dense
    gradient as M x N products over K."""
    g = torch.Generator(device=DEV).manual_seed(M)
    A, B = torch.randn(M, K, generator=g, device=DEV), torch.randn(N, K, generator=g, device=DEV)
    ref = A.double() @ B.double().t()
    new = lambda: torch.full((M, N), float("nan"), device=DEV)  # noqa: E731
    Y, dX, G = new(), new(), new()
    try:
        mst.mst_gemm_force_fp32_mfma(1128)
        for O, I, W, out, call in ((N, K, B, Y, mst.mst_sparse_fc_fwd), (K, N, B.t().contiguous(), dX, mst.mst_sparse_fc_bwd_input)):
            L = mst.Layer(O, I, O * I, DEV)
            ws = torch.empty(mst.mst_workspace_bytes(O, I, O * I, 1), dtype=torch.uint8, device=DEV)
            L.load_dense(W, torch.ones((O, I), dtype=torch.uint8, device=DEV), ws)
            L.set_path(mst.MST_PATH_DENSE)
            call(L, A, out, M, mst.MST_F32)
        mst.mst_dense_grad(A.t().contiguous(), B.t().contiguous(), G, K, M, N, mst.MST_F32, None)
        torch.cuda.synchronize()
    finally:
        mst.mst_gemm_force_fp32_mfma(0)
    for got in (Y, dX, G):
        assert float((got.double() - ref).abs().max()) <= FP32 * float(ref.abs().max())
