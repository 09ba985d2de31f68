"""Dense products with two scaled fp16 parts per fp32 operand: Y, dX and the dense gradient at the edges of the
256 x 256 tile and of its k steps of 32, and values outside the range that the scales of a row cover (the loop over
three bfloat16 parts, entered at any step).  Against fp64."""
import numpy as np
import pytest

import paper_2408_11746_amd as mst
import synth

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
import test_gpu_exact_products as exact  # noqa: E402
from gpu_util import Rig, DEV, dev  # noqa: E402


@pytest.mark.parametrize("T,I,O", exact.SHAPES + [(256, 256, 256), (255, 31, 257), (257, 33, 255), (300, 513, 32), (64, 511, 512)])
def test_fp32_operands_at_the_edges_of_the_256_tile(T, I, O):
    exact.test_fp32_operands_of_any_shape(T, I, O, 1256)


def test_infinities_and_one_sided_errors_on_the_256_tile():
    exact.test_infinite_operands_as_fp32_products_give_them(1256, mst.MST_F32)
    exact.test_infinite_operands_of_the_input_gradient_and_the_dense_gradient(1256, mst.MST_F32)
    exact.test_positive_operands_of_full_mantissas_leave_no_one_sided_error(1256)
    exact.test_values_next_to_the_largest_finite_one(1256)


def _spread(kind, a):
    """what is done to an operand a[rows, k]"""
    rows, k = a.shape
    r, c = np.arange(rows)[:, None], np.arange(k)[None, :]
    return {"rows of any size": lambda: a * np.exp2((r * 37) % 200 - 100.0),           # scales of every row
            "zero to begin with": lambda: np.where(c < 70, 0.0, a) * 2.0 ** -60,       # no scale from the first steps
            "zero throughout": lambda: a * 0.0,
            "growing along k": lambda: a * np.exp2(c / 16.0 - 20),                     # leaves the range upwards
            "shrinking along k": lambda: a * np.exp2(-c / 16.0),                       # ... and downwards
            "outliers": lambda: np.where(c % 97 == 5, a * 3e5, a),
            "an outlier in the first unit": lambda: np.where(c == 2, a * 3e5, a)}[kind]().astype(np.float32)


@pytest.mark.parametrize("mode", [1128, 1256])
@pytest.mark.parametrize("kind", ["rows of any size", "zero to begin with", "zero throughout", "growing along k", "shrinking along k",
                                  "outliers", "an outlier in the first unit"])
def test_values_outside_the_range_of_the_scales(kind, mode):
    """Error of every output in units of 2^-24 sum |x w|.  An output is the end of at most 6 K / 16 fp32 additions in a row.
    Where one large term makes the sum, every one of them rounds a value as large as sum |x w|, whose last place is at most
    2^-23 of it: uniform over that place, 2^-23 / sqrt(12) = 0.58 units in the root mean square, of either sign.  Six
    times what they leave together is allowed.  (A value that the scales did not cover would be off by thousands of units.)"""
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
