"""FP32 scoring with a wave per sub-tile and a few row pairs (the form for few
windows): every window of grids at the edges of its tiles against a float64
correlation, the same bits as the band kernel's, and non-finite features."""
import numpy as np
import pytest

import pd_synth

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
import paper_1611_01642_amd as pd  # noqa: E402

DEV = "cuda:0"


def reference(blocks, cells, weights, bias):
    """[m][ny][nx] float64 of every window that starts on the grid."""
    f = torch.from_numpy
    hog, lbp, w = f(blocks).double(), f(cells).double(), f(weights).double()
    m, ny, nx = len(w), lbp.shape[1] - 15, lbp.shape[2] - 7
    out = f(bias).double().view(m, 1, 1).expand(m, ny, nx).clone()
    for plane, part, rows, cols in ((hog, w[:, :3780], 15, 7), (lbp, w[:, 3780:], 16, 8)):
        part = part.reshape(m, rows, cols, -1)
        for a in range(rows):
            for b in range(cols):
                out += torch.einsum("mc,cyx->myx", part[:, a, b], plane[:, a:a + ny, b:b + nx])
    return out.numpy()


def features(hc, wc, seed):
    rng = np.random.default_rng(seed)
    blocks = rng.random((36, hc - 1, wc - 1), dtype=np.float32) * 0.3
    cells = rng.multinomial(64, np.full(59, 1 / 59), (hc, wc)).transpose(2, 0, 1).astype(np.uint8)
    return blocks, np.ascontiguousarray(cells)


def score(blocks, cells, weights, bias):
    to = lambda a: torch.from_numpy(a).to(DEV)  # noqa: E731
    out = pd.score_windows(to(blocks), to(cells), to(weights), to(bias))
    torch.cuda.synchronize()
    return out.cpu().numpy()


# one window; a tile's, a run's and a sub-tile's last and first columns; one row pair more or less than a band;
# grids past the limits of one and of two row pairs per wave
@pytest.mark.parametrize("hc,wc,m", [(16, 8, 1), (16, 16, 2), (17, 17, 1), (18, 63, 1), (31, 64, 3), (32, 65, 1),
                                     (33, 128, 1), (47, 129, 1), (48, 130, 2), (49, 200, 1), (300, 700, 1), (600, 900, 2)])
def test_every_window(hc, wc, m):
    blocks, cells = features(hc, wc, hc * 1000 + wc)
    weights, bias = pd_synth.svm_weights(m), np.linspace(-0.3, 0.4, m).astype(np.float32)
    exp = reference(blocks, cells, weights, bias)
    got = score(blocks, cells, weights, bias)
    assert np.all(np.abs(got - exp) <= 1e-4 * np.maximum(np.abs(exp), exp.std()))


@pytest.mark.parametrize("features", [pd.FEAT_HOG, pd.FEAT_LBP, pd.FEAT_HOG | pd.FEAT_LBP])
def test_same_bits_as_the_band_kernel(features):
    """110 frames (550 levels) are scored by the band kernel, each alone by the wave kernel; with every window a
    candidate, all scores are the same bits.  40 frames take two or four row pairs per wave."""
    frames = [torch.from_numpy(pd_synth.frame(200, 213, 300 + k % 5)).to(DEV) for k in range(110)]
    weights, bias = torch.from_numpy(pd_synth.svm_weights(1)).to(DEV), torch.full((1,), 0.25, device=DEV)

    def run(part):
        det = pd.Detector(part, weights, bias, pd.params(features=features), cap=64)
        det.run(torch.full((len(part),), -1e30, dtype=torch.float64, device=DEV))
        torch.cuda.synchronize()
        out = []
        for f in range(0, len(part), max(1, len(part) // 5 + 1)):
            s, k, _ = det.candidates(f)
            out.append((f % 5, {tuple(key): v.view(np.int32) for key, v in zip(k.tolist(), s)}))
        return out
    alone = [run([f])[0][1] for f in frames[:5]]
    assert len(alone[0]) > 100
    for part in (frames, frames[:60], frames[:40]):
        for f, got in run(part):
            assert got == alone[f]


def test_non_finite_features_reach_their_own_windows_only():
    blocks, cells = features(40, 50, 5)
    for c, y, x, v in ((0, 3, 5, np.nan), (35, 20, 41, np.inf), (7, 38, 48, -np.inf)):
        blocks[c, y, x] = v
    weights, bias = pd_synth.svm_weights(1), np.zeros(1, np.float32)
    exp, got = reference(blocks, cells, weights, bias), score(blocks, cells, weights, bias)
    assert np.array_equal(np.isnan(exp), np.isnan(got)) and np.array_equal(np.isfinite(exp), np.isfinite(got))
    fine = np.isfinite(exp)
    assert 0 < fine.sum() < fine.size
    assert np.all(np.abs(got - exp)[fine] <= 1e-4 * np.maximum(np.abs(exp[fine]), exp[fine].std()))
