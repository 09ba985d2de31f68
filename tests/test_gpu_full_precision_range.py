"""Dense products at full fp32 precision on operands of any range: rows of very different size, values that grow or shrink
along the contraction index, rows that are zero to begin with, outliers, pruned weights, a neighbour that is not finite.
Every output has the precision of its own terms, whatever the other rows of its tile hold.  Against fp64."""
import numpy as np
import pytest

import paper_2408_11746_amd as mst
import synth

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
import test_gpu_exact_products as exact  # noqa: E402
from gpu_util import Rig, DEV, dev  # noqa: E402


@pytest.mark.parametrize("T,I,O", exact.SHAPES + [(256, 256, 256), (255, 31, 257), (257, 33, 255), (300, 513, 32), (64, 511, 512)])
def test_fp32_operands_at_the_edges_of_the_largest_tile(T, I, O):
    exact.test_fp32_operands_of_any_shape(T, I, O, 1256)


def test_infinities_and_one_sided_errors_on_the_largest_tile():
    exact.test_infinite_operands_as_fp32_products_give_them(1256, mst.MST_F32)
    exact.test_infinite_operands_of_the_input_gradient_and_the_dense_gradient(1256, mst.MST_F32)
    exact.test_positive_operands_of_full_mantissas_leave_no_one_sided_error(1256)
    exact.test_values_next_to_the_largest_finite_one(1256)


def _spread(kind, a):
    """what is done to an operand a[rows, k]"""
    rows, k = a.shape
    r, c = np.arange(rows)[:, None], np.arange(k)[None, :]
    return {"rows of any size": lambda: a * np.exp2((r * 37) % 200 - 100.0),           # every row its own
            "zero to begin with": lambda: np.where(c < 70, 0.0, a) * 2.0 ** -60,       # nothing in the first steps
            "zero throughout": lambda: a * 0.0,
            "growing along k": lambda: a * np.exp2(c / 16.0 - 20),                     # by 2^33
            "shrinking along k": lambda: a * np.exp2(-c / 16.0),                       # to 2^-33
            "outliers": lambda: np.where(c % 97 == 5, a * 3e5, a),
            "an outlier in the first unit": lambda: np.where(c == 2, a * 3e5, a)}[kind]().astype(np.float32)


@pytest.mark.parametrize("mode", [1128, 1256])
@pytest.mark.parametrize("kind", ["rows of any size", "zero to begin with", "zero throughout", "growing along k", "shrinking along k",
                                  "outliers", "an outlier in the first unit"])
def test_operands_of_any_range(kind, mode):
    """Error of every output in units of 2^-24 sum |x w|.  An output is the end of at most 6 K / 16 fp32 additions in a row.
    Where one large term makes the sum, every one of them rounds a value as large as sum |x w|, whose last place is at most
    2^-23 of it: uniform over that place, 2^-23 / sqrt(12) = 0.58 units in the root mean square, of either sign.  Six
    times what they leave together is allowed."""
    T, I, O = 270, 515, 290
    print("case", kind, mode, flush=True)
    rng = np.random.default_rng(5)
    X, W, dY = rng.standard_normal((T, I)), 0.02 * rng.standard_normal((O, I)), 1e-3 * rng.standard_normal((T, O))
    G = torch.full((O, I), float("nan"), dtype=torch.float32, device=DEV)
    got = {}
    products = {"Y": (_spread(kind, X), W.astype(np.float32)), "dX": (_spread(kind, dY), W.T.astype(np.float32)),
                "G": (_spread(kind, dY.T), X.T.astype(np.float32))}
    try:
        mst.mst_gemm_force_fp32_mfma(mode)
        for name, (A, B) in products.items():
            Wn = {"Y": B, "dX": B.T, "G": W.astype(np.float32)}[name]
            rig = Rig(np.ascontiguousarray(Wn), np.ones((O, I), np.uint8), T, cap=O * I)
            rig.layer.set_path(mst.MST_PATH_DENSE)
            if name == "Y":
                got[name] = rig.fwd(A)
            elif name == "dX":
                got[name] = rig.bwd_input(A)
            else:
                mst.mst_dense_grad(dev(np.ascontiguousarray(A.T)), dev(np.ascontiguousarray(B.T)), G, T, O, I, mst.MST_F32, None)
                torch.cuda.synchronize()
                got[name] = G.cpu().numpy()
    finally:
        mst.mst_gemm_force_fp32_mfma(0)
    for name, (A, B) in products.items():
        A, B = A.astype(np.float64), B.astype(np.float64)
        size = np.abs(A) @ np.abs(B).T
        err = np.abs(got[name] - A @ B.T)
        bound = 6 * 0.58 * np.sqrt(6 * A.shape[1] / 16) * 2.0 ** -24
        print(name, "largest error %.3g of %.3g allowed" % ((err / np.maximum(size, 1e-300)).max(), bound), flush=True)
        assert (err <= bound * size + 2.0 ** -149).all(), name


# Rows of one operand among rows that differ from them, a[rows, k].  Every one is judged by its own terms.
def _neighbours(kind, a):
    rows, k = a.shape
    r, c = np.arange(rows)[:, None], np.arange(k)[None, :]
    late = np.where((r % 2 == 1) & (c < 32), 0.0, a)                                   # every other row begins with zeros
    return {"zeros first, a row 2^20 larger": lambda: np.where(r == 0, late * 2.0 ** 20, late),
            "zeros first, a row 2^36 larger": lambda: np.where(r == 0, late * 2.0 ** 36, late),
            "zeros first, a row of NaN": lambda: np.where(r == 0, np.nan, late),
            "zeros first, a row of infinities": lambda: np.where(r == 0, np.inf, late),
            "one row in four shrinks by 2^17": lambda: np.where((r % 4 == 3) & (c >= 32), a * 2.0 ** -17, a),
            "one row in four shrinks by 2^30": lambda: np.where((r % 4 == 3) & (c >= 32), a * 2.0 ** -30, a),
            "all rows shrink by 2^24": lambda: np.where(c >= 32, a * 2.0 ** -24, a)}[kind]().astype(np.float32)


@pytest.mark.parametrize("mode", [0, 1032, 1064, 1096, 1128, 1256])
@pytest.mark.parametrize("kind", ["zeros first, a row 2^20 larger", "zeros first, a row 2^36 larger", "zeros first, a row of NaN",
                                  "zeros first, a row of infinities", "one row in four shrinks by 2^17",
                                  "one row in four shrinks by 2^30", "all rows shrink by 2^24"])
def test_rows_keep_their_precision_whatever_their_neighbours_hold(kind, mode):
    """The other operand is pruned to a tenth, and half of its rows have nothing in the first 32 k: their outputs are sums of terms of
    one size and random sign.  The partial sums of such a sum of n terms are sqrt(j) of them, sum |x w| is 0.64 n, and each of at
    most 6 n fp32 additions is off by 2^-24 / sqrt(3) of its partial sum in the root mean square: sqrt(6 n * n / 2 / 3) / (0.64 n) =
    1.6 units of 2^-24 sum |x w| if every product of a term is added by itself.  3.2 is allowed for a row of outputs in the
    root mean square; every output has the bound of the test above."""
    T, I, O = 650, 515, 770
    print("case", kind, mode, flush=True)
    rng = np.random.default_rng(6)
    X, dY = rng.standard_normal((T, I)), rng.standard_normal((T, O))

    def pruned(rows, k):                                                               # [rows, k]
        keep = rng.random((rows, k)) < 0.1
        keep[::2, :32] = False
        keep[::2, 32:64] = True                                                        # (a row has terms at all)
        return np.where(keep, rng.standard_normal((rows, k)), 0.0).astype(np.float32)

    products = {"Y": (_neighbours(kind, X), pruned(O, I)), "dX": (_neighbours(kind, dY), pruned(I, O)),
                "G": (_neighbours(kind, dY.T), pruned(I, T))}
    got = {}
    try:
        mst.mst_gemm_force_fp32_mfma(mode)
        for name, (A, B) in products.items():
            if name == "G":
                G = torch.full((O, I), 7.0, dtype=torch.float32, device=DEV)
                mst.mst_dense_grad(dev(np.ascontiguousarray(A.T)), dev(np.ascontiguousarray(B.T)), G, T, O, I, mst.MST_F32, None)
                torch.cuda.synchronize()
                got[name] = G.cpu().numpy()
                continue
            Wn = np.ascontiguousarray(B if name == "Y" else B.T)
            rig = Rig(Wn, (Wn != 0).astype(np.uint8), T, cap=O * I)
            rig.layer.set_path(mst.MST_PATH_DENSE)
            got[name] = rig.fwd(A) if name == "Y" else rig.bwd_input(A)
    finally:
        mst.mst_gemm_force_fp32_mfma(0)
    for name, (A, B) in products.items():
        A, B = A.astype(np.float64), B.astype(np.float64)
        A, out = (A[1:], got[name][1:]) if not np.isfinite(A[0]).all() else (A, got[name])       # (its own outputs are not finite)
        size = np.abs(A) @ np.abs(B).T
        units = np.abs(out - A @ B.T) / np.maximum(size, 1e-300) * 2.0 ** 24
        even = np.sqrt((units[:, ::2] ** 2).mean(axis=1))                              # per row of A, outputs without the first 32 k
        across = np.sqrt((units[:, ::2] ** 2).mean(axis=0))
        bound = 6 * 0.58 * np.sqrt(6 * A.shape[1] / 16)
        print(name, "units: largest %.3g of %.3g, rows up to %.3g, columns up to %.3g" % (units.max(), bound, even.max(), across.max()), flush=True)
        assert units.max() <= bound and even.max() <= 3.2 and across.max() <= 3.2, name
