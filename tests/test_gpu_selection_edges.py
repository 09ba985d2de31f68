"""The selections of an update where their passes change over: fewer than four positions, remainders behind the last group of four,
ranges of the flag pass (16384 positions each) that are just full, and thresholds that many equal keys share, so that the
ranges hand each other their counts.  Masks, weights and index sets are bit-exact."""
import numpy as np
import pytest

import synth
from test_gpu_mask_update import _update_and_compare

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("O,I", [(1, 1), (1, 2), (1, 3), (3, 1), (1, 5), (7, 9), (127, 129), (128, 128), (5, 3277), (113, 435), (257, 1023)])
@pytest.mark.parametrize("scores", ["distinct", "few values", "equal", "zero"])
@pytest.mark.parametrize("R", [0.0, 0.4, 1.0])
def test_update(O, I, scores, R):
    W, M = synth.make_layer(31, 4, I, O, 0.3)
    if scores != "distinct":
        W = (np.sign(W) * 0.5).astype(np.float32) * M              # every weight a tie as well
    G = synth.normal(31, 78, (O, I))
    G = {"distinct": G, "few values": np.round(G).astype(np.float32), "equal": np.full_like(G, -2.0), "zero": np.zeros_like(G)}[scores]
    _update_and_compare(W, M, G, 0.3, 0.5, R, seed=77)
