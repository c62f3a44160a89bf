"""Features with a wave per cell row (the form for few strips) at the edges of
its workgroups, strips and lane groups, against the FP64 oracle: LBP counts
exact, HOG blocks and cell maps within 1e-4, from rows at any alignment."""
import numpy as np
import pytest

import pd_synth
from oracle import pd_oracle as O
from oracle import pruner_oracle as P

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
import paper_1611_01642_amd as pd  # noqa: E402

DEV = "cuda:0"


def device_image(img, shift):
    """The image as a view that starts `shift` bytes past an aligned address, with an odd pitch."""
    h, w = img.shape
    buf = torch.zeros((h, w + 2 * shift + 1), dtype=torch.uint8, device=DEV)
    view = buf[:, shift:shift + w]
    view.copy_(torch.from_numpy(img))
    return view


# cells per row: lane groups of 2 to 64, one and two strips (62 and 63 owned columns); cell rows: one, a workgroup's
# and one more or less, its overlaps; pixels past the last whole cell
@pytest.mark.parametrize("wc,hc,shift", [(1, 1, 0), (2, 2, 1), (3, 9, 0), (4, 33, 3), (9, 17, 0), (17, 8, 2), (33, 5, 0),
                                         (62, 3, 0), (63, 4, 1), (64, 7, 0), (65, 6, 0), (127, 13, 5), (128, 2, 0)])
def test_features_and_cellmap(wc, hc, shift):
    w, h = 8 * wc + (wc * 3) % 8, 8 * hc + (hc * 5) % 8
    img = pd_synth.frame(w, h, 50 + wc + hc)
    dev = device_image(img, shift)
    hog = O.hog_features(img).transpose(2, 0, 1)
    lbp = O.lbp_cell_histograms(img).transpose(2, 0, 1)

    def check(blocks, cells):
        torch.cuda.synchronize()
        if cells is not None:
            assert np.array_equal(cells.cpu().numpy(), lbp)
        if blocks is not None and hog.size:
            got = blocks.float().cpu().numpy()
            tol = 2.0 ** -8 if blocks.dtype == torch.bfloat16 else 0.0
            assert np.all(np.abs(got - hog) <= (1e-4 + tol) * np.abs(hog) + 1e-6)
    check(*pd.features(dev))
    check(*pd.features(dev, bf16=True))
    if hog.size:
        check(pd.hog(dev), None)
    check(None, pd.lbp(dev))
    if wc > 1 and hc > 1:
        blocks, cells, cmap = pd.features_cellmap(dev)
        check(blocks, cells)
        exp = P.cellmap(img).transpose(2, 0, 1)
        got = cmap.cpu().numpy()
        assert np.array_equal(got[9:], exp[9:].astype(np.float32))
        assert np.all(np.abs(got[:9] - exp[:9]) <= 1e-4 * np.abs(exp[:9]) + 2e-6)
