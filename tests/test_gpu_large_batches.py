"""The forms that large batches and images take (bands of FP32 scoring, feature
strips) against the ones small calls take (a wave per sub-tile, a wave per cell
row): a frame's scores, and an image's features, are the same bits in both.  The
sizes are checked against the limits in the sources, so that a limit moved past
them shows here instead of leaving both sides of a comparison to one form."""
import os
import re

import numpy as np
import pytest

import pd_synth

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
import paper_1611_01642_amd as pd  # noqa: E402

DEV = "cuda:0"
W, H, COPIES, IMAGES = 1242, 375, 8, 5
CSRC = os.path.join(os.path.dirname(pd.__file__), "csrc")


def constant(name, files=("pd_internal.h", "score32.hip")):
    text = "".join(open(os.path.join(CSRC, f)).read() for f in files)
    return int(re.search(rf"\b{name}\s*=\s*(\d+)", text).group(1))


def levels(w, h):
    return [(lv.cells_x, lv.cells_y) for lv in pd.plan_pyramid(w, h)[0]]


def strip_rows(w, h):
    return sum(max(1, -(-(cx - 1) // 63)) * cy for cx, cy in levels(w, h))


def entries(w, h):
    return sum(-(-(cy - 15) // 16) * -(-(-(-cx // 64)) // 2) for cx, cy in levels(w, h))


@pytest.fixture(scope="module")
def images():
    return [torch.from_numpy(pd_synth.frame(W, H, 300 + k)).to(DEV) for k in range(IMAGES)]


def windows(frames, m, **kw):
    """Every window of each frame: (level, i, j, model) -> the bits of its score."""
    weights = torch.from_numpy(pd_synth.svm_weights(m)).to(DEV)
    det = pd.Detector(frames, weights, torch.full((m,), 0.25, device=DEV), pd.params(**kw), cap=64)
    det.run(torch.full((len(frames),), -1e30, dtype=torch.float64, device=DEV))
    torch.cuda.synchronize()
    out = []
    for f in range(len(frames)):
        s, k, _ = det.candidates(f)
        k = np.asarray(k)[:, :4]
        order = np.lexsort((k[:, 2], k[:, 1], k[:, 0]))
        out.append((k[order].tobytes(), np.asarray(s, np.float32)[order].tobytes()))
    return out


# window rows per band and a capped grid on the band kernel, strip heights and a capped grid on the strips
@pytest.mark.parametrize("tuning", [{}, dict(tune_score_rows=4), dict(tune_score_rows=16), dict(tune_grid=40),
                                    dict(tune_feat_rows=13, tune_score_rows=16, tune_grid=7)])
@pytest.mark.parametrize("m,kw", [(1, {}), (1, dict(features=pd.FEAT_HOG)), (1, dict(features=pd.FEAT_LBP)), (2, {}),
                                  (2, dict(features=pd.FEAT_HOG)), (3, dict(features=pd.FEAT_LBP)),
                                  (1, dict(precision=pd.PREC_BF16))])
def test_batch_has_each_frame_alone(images, m, kw, tuning):
    n = COPIES * IMAGES
    assert n * entries(W, H) > constant("SW_MAX_ENTRIES") >= m * entries(W, H)
    assert n * strip_rows(W, H) > constant("FR_MAX_ROWS") >= strip_rows(W, H)
    alone = [windows([f], m, **kw)[0] for f in images]
    batch = windows(images * COPIES, m, **kw, **tuning)
    for f, got in enumerate(batch):
        assert got == alone[f % IMAGES], f


@pytest.mark.parametrize("w,h", [(16384, 2801), (2601, 16384)])
def test_large_image_has_its_bands(w, h):
    """Features and cell map of an image past the limit of the form for few strips equal, bit for bit, those of its
    bands of cell rows, which that form takes (without the rows that see a band's cut edge)."""
    tiles = -(-(w // 8 - 1) // 63)
    assert tiles * (h // 8) > constant("FR_MAX_ROWS")
    part = pd_synth.frame(min(w, 2048), min(h, 2048), 77)
    img = torch.from_numpy(np.tile(part, (-(-h // part.shape[0]), -(-w // part.shape[1])))[:h, :w].copy()).to(DEV)
    hog, lbp = pd.features(img)
    only_hog, only_lbp = pd.hog(img), pd.lbp(img)
    hog16, _ = pd.features(img, bf16=True)
    chog, clbp, cmap = pd.features_cellmap(img)
    torch.cuda.synchronize()
    assert torch.equal(hog, only_hog) and torch.equal(lbp, only_lbp) and torch.equal(lbp, clbp)
    assert torch.equal(hog.to(torch.bfloat16), hog16)
    rows = h // 8
    for c0 in (0, rows // 2 - 7, rows - 41):  # 41 cell rows each
        band = img[8 * c0:h if c0 + 41 == rows else 8 * (c0 + 41)]
        bhog, blbp = pd.features(band)
        bchog, _, bcmap = pd.features_cellmap(band)
        torch.cuda.synchronize()
        lo, hi = (0 if c0 == 0 else 1), (41 if c0 + 41 == rows else 40)
        assert torch.equal(blbp[:, lo:hi], lbp[:, c0 + lo:c0 + hi])
        assert torch.equal(bhog[:, lo:hi - 1], hog[:, c0 + lo:c0 + hi - 1])
        assert torch.equal(bchog[:, lo:hi - 1], chog[:, c0 + lo:c0 + hi - 1])
        # a cell's histogram has votes from the rows above and below it too
        lo, hi = (0 if c0 == 0 else 2), (41 if c0 + 41 == rows else 39)
        assert torch.equal(bcmap[:, lo:hi], cmap[:, c0 + lo:c0 + hi])
    assert bool(torch.isfinite(cmap).all()) and bool(torch.isfinite(hog).all())
