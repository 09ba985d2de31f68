"""The dense weight gradient of bfloat16 activations (Algorithm 1's G = dY^T X) on 256 x 256 tiles whose rows go straight to
LDS: partial tiles in both dimensions, one and several steps of 32 tokens, an odd number of them, a last one that is
not full, several k ranges.  Against the fp64 product: products of two bfloat16 numbers are exact, a sum of T of them in fp32 is
off by at most T 2^-23 of the sum of their magnitudes, whatever the order (2^-23: also where the matrix cores truncate)."""
import numpy as np
import pytest

import paper_2408_11746_amd as mst
import synth

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
from gpu_util import DEV, dev  # noqa: E402


@pytest.fixture(autouse=True)
def tile256():
    mst.mst_gemm_force_fp32_mfma(256)                        # (products this small would go to other kernels)
    yield
    mst.mst_gemm_force_fp32_mfma(0)


@pytest.mark.parametrize("T,O,I,ranges", [(1, 8, 8, 1), (31, 256, 256, 1), (32, 264, 248, 1), (33, 256, 520, 1), (64, 512, 256, 1), (97, 776, 136, 1),
                                          (256, 256, 256, 1), (1027, 264, 264, 2), (1536, 256, 512, 3), (3001, 520, 8, 4)])
def test_gradient_against_fp64(T, O, I, ranges):
    print("case", T, O, I, ranges, flush=True)
    X, dY, xb, yb = synth.make_activations(53, 1, T, I, O, "bf16")
    # what follows the last token is not part of the product
    Xd, Yd = torch.full((T + 64, I), float("nan"), device=DEV, dtype=torch.bfloat16), torch.full((T + 64, O), float("nan"), device=DEV, dtype=torch.bfloat16)
    Xd.view(torch.int16)[:T].copy_(dev(xb.view(np.int16)))
    Yd.view(torch.int16)[:T].copy_(dev(yb.view(np.int16)))
    G = torch.full((O + 1, I), 7.0, device=DEV)
    ws = torch.empty(ranges * O * I * 4, device=DEV, dtype=torch.uint8) if ranges > 1 else None
    mst.mst_dense_grad(Yd, Xd, G, T, O, I, mst.MST_BF16, ws)
    G = G.cpu().numpy()
    X, dY = X.astype(np.float64), dY.astype(np.float64)
    assert np.all(np.abs(G[:O] - dY.T @ X) <= T * 2.0 ** -23 * (np.abs(dY).T @ np.abs(X)))
    assert np.all(G[O] == 7.0)


def test_infinite_values_stay_in_their_row_and_column():
    T, O, I = 65, 256, 264
    X, dY, xb, yb = synth.make_activations(54, 1, T, I, O, "bf16")
    xb = xb.copy()
    xb.view(np.uint16)[T - 1, 5] = 0x7F80
    G = torch.zeros((O, I), device=DEV)
    mst.mst_dense_grad(dev(yb.view(np.int16)), dev(xb.view(np.int16)), G, T, O, I, mst.MST_BF16, None)
    G = G.cpu().numpy()
    sign = np.sign(dY[T - 1])
    assert np.all(G[sign != 0, 5] == np.inf * sign[sign != 0])
    assert np.all(np.isfinite(np.delete(G, 5, axis=1)))
