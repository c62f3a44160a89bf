"""Cell maps of one image on both sides of the line between waves per cell row
and strips (5400 strip rows): the same bits as those of bands of its rows."""
import numpy as np
import pytest

import pd_synth

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
import paper_1611_01642_amd as pd  # noqa: E402

DEV = "cuda:0"


# strip rows: 8 strips of 62 columns by 675 and 676, 34 by 158 and 159, 17 by 647
@pytest.mark.parametrize("wc,hc", [(496, 675), (496, 676), (2048, 158), (2048, 159), (1024, 647)])
def test_bands(wc, hc):
    w, h = min(8 * wc + 5, 16384), 8 * hc + 3
    part = pd_synth.frame(min(w, 2048), min(h, 2048), wc + hc)
    img = torch.from_numpy(np.tile(part, (-(-h // part.shape[0]), -(-w // part.shape[1])))[:h, :w].copy()).to(DEV)
    hog, lbp, cmap = pd.features_cellmap(img)
    _, lbp_alone = pd.features(img)
    torch.cuda.synchronize()
    assert torch.equal(lbp, lbp_alone)
    for c0 in (0, hc // 3, hc - 30):  # 30 cell rows each, without those that see a cut edge
        last = c0 + 30 == hc
        bhog, blbp, bcmap = pd.features_cellmap(img[8 * c0:h if last else 8 * (c0 + 30)])
        torch.cuda.synchronize()
        lo, hi = (0 if c0 == 0 else 2), (30 if last else 28)
        assert torch.equal(blbp[:, lo:hi], lbp[:, c0 + lo:c0 + hi])
        assert torch.equal(bhog[:, lo:hi - 1], hog[:, c0 + lo:c0 + hi - 1])
        assert torch.equal(bcmap[:, lo:hi], cmap[:, c0 + lo:c0 + hi])
