"""pd_score_windows on grids with many windows (the vector-ALU form), around the
line to the wave form: every window against a float64 correlation, and non-finite
features in their own windows only."""
import numpy as np
import pytest

import pd_synth
from test_gpu_score_waves import features, reference, score

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


def entries(hc, wc, m):
    return -(-(hc - 15) // 16) * -(-wc // 128) * m


# narrow and low grids with many models, tiles' last columns and rows, both sides of 512 entries
@pytest.mark.parametrize("hc,wc,m,many", [(16, 2048, 16, False), (2048, 8, 4, False), (2048, 8, 5, True),
                                          (529, 71, 16, True), (528, 135, 8, True), (271, 500, 8, False),
                                          (272, 513, 7, True), (48, 2048, 16, True)])
def test_every_window(hc, wc, m, many):
    assert (entries(hc, wc, m) > 512) == many
    blocks, cells = features(hc, wc, hc * 7 + wc)
    weights, bias = pd_synth.svm_weights(m), np.linspace(-0.3, 0.4, m).astype(np.float32)
    exp = reference(blocks, cells, weights, bias)
    got = score(blocks, cells, weights, bias)
    assert np.all(np.abs(got - exp) <= 1e-4 * np.maximum(np.abs(exp), exp.std()))


def test_non_finite_features_reach_their_own_windows_only():
    hc, wc, m = 530, 200, 16
    assert entries(hc, wc, m) > 512
    blocks, cells = features(hc, wc, 5)
    for c, y, x, v in ((0, 3, 5, np.nan), (35, 220, 198, np.inf), (7, 528, 100, -np.inf)):
        blocks[c, y, x] = v
    weights, bias = pd_synth.svm_weights(m), np.zeros(m, np.float32)
    exp, got = reference(blocks, cells, weights, bias), score(blocks, cells, weights, bias)
    assert np.array_equal(np.isnan(exp), np.isnan(got)) and np.array_equal(np.isfinite(exp), np.isfinite(got))
    fine = np.isfinite(exp)
    assert 0 < fine.sum() < fine.size
    got, exp = got[fine], exp[fine]
    assert np.all(np.abs(got - exp) <= 1e-4 * np.maximum(np.abs(exp), exp.std()))
