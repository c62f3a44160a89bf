"""BF16 scoring of one model at the widths where its staging of channel pairs
changes form: rows shorter than a word's four columns past the tile, tiles of 64
windows with one, two and three columns over, the planes' last channel; against
the exact sum of the BF16 operands, up to FP32 accumulation."""
import numpy as np
import pytest

import pd_synth
from oracle import pd_oracle as O

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
import paper_1611_01642_amd as pd  # noqa: E402

DEV = "cuda:0"


def bf16_round(a):
    return torch.from_numpy(np.ascontiguousarray(a, dtype=np.float32)).to(torch.bfloat16).to(torch.float64).numpy()


@pytest.mark.parametrize("wc", [8, 9, 10, 11, 12, 70, 71, 72, 73, 74, 135, 136, 199])
@pytest.mark.parametrize("hc", [16, 17, 33])
def test_widths(wc, hc):
    rng = np.random.default_rng(100 * hc + wc)
    hog = bf16_round(rng.random((hc - 1, wc - 1, 36)) * 0.4)
    cells = rng.integers(0, 65, (hc, wc, 59)).astype(np.uint8)
    wts = pd_synth.svm_weights(1)
    hi = bf16_round(wts)
    lo = bf16_round(wts.astype(np.float64) - hi)
    lo[:, :O.HOG_DIM] = 0.0  # HOG weights carry their BF16 part only
    # exact sizes: the planes end with their allocation
    planes = torch.from_numpy(np.ascontiguousarray(hog.transpose(2, 0, 1), dtype=np.float32)).to(DEV).to(torch.bfloat16)
    counts = torch.from_numpy(np.ascontiguousarray(cells.transpose(2, 0, 1))).to(DEV)
    packed = pd.pack_models(torch.from_numpy(wts).to(DEV))
    got = pd.score_windows_bf16(planes, counts, packed, torch.zeros(1, device=DEV), 1).cpu().numpy()
    exp = O.window_scores(hog, cells, hi + lo, np.zeros(1))
    absx = O.window_scores(np.abs(hog), cells, np.abs(hi) + np.abs(lo), np.zeros(1))
    assert got.shape == exp.shape
    # FP32 accumulation of ~2 x 11520 exact products
    assert np.all(np.abs(got - exp) <= 2 * 11520 * 2.0 ** -24 * absx + 1e-6)
