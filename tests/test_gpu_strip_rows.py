"""Feature strips whose rows the library chooses, around the batch sizes where
they begin and where another count of rows is chosen: the same bytes as with
any rows asked for (which give waves per cell row their own form's results)."""
import numpy as np
import pytest

import pd_synth

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
import paper_1611_01642_amd as pd  # noqa: E402

DEV = "cuda:0"

# equal frames in a run, the same size again after another, one window high,
# one block column past a full strip (65 cells), levels one and two strips wide
BATCHES = {
    "rows": [(1242, 375)] * 11,
    "road12": [(1242, 375)] * 12,
    "road16": [(1242, 375)] * 16,
    "mixed": [(520, 400)] * 5 + [(64, 128)] * 3 + [(1920, 1080)] * 3 + [(520, 400)] * 2 + [(200, 131), (513, 240)] * 4,
}


@pytest.mark.parametrize("kw", [dict(), dict(features=1), dict(features=2), dict(precision=pd.PREC_BF16), dict(prune=1)])
@pytest.mark.parametrize("name", sorted(BATCHES))
def test_chosen_rows(name, kw):
    kw = dict(kw)
    frames = [torch.from_numpy(f).to(DEV) for f in pd_synth.frame_batch(BATCHES[name], 321)]
    wts = torch.from_numpy(pd_synth.svm_weights(1)).to(DEV)
    if kw.pop("prune", 0):
        pruner = torch.from_numpy(np.random.default_rng(3).normal(0, 0.05, pd.PRUNER_PARAMS).astype(np.float32)).to(DEV)
        kw.update(precision=pd.PREC_BF16, prune_keep=500, pruner=pruner)
    # a few windows of every frame
    det = pd.Detector(frames, wts, torch.zeros(1, device=DEV), pd.params(**kw), cap=512)
    det.run(torch.full((len(frames),), -1.0e30, dtype=torch.float64, device=DEV))
    torch.cuda.synchronize()
    scores = [np.sort(np.asarray(det.candidates(f)[0]))[::-1] for f in range(len(frames))]
    thr = torch.tensor([float(s[len(s) // 50]) for s in scores], dtype=torch.float64, device=DEV)
    res = []
    for rows in (0, 4, 8, 32):
        det = pd.Detector(frames, wts, torch.zeros(1, device=DEV), pd.params(tune_feat_rows=rows, **kw), cap=512)
        det.run(thr)
        torch.cuda.synchronize()
        boxes, counts = det.results()
        res.append(([b.tobytes() for b in boxes], [c.tobytes() for c in counts]))
    assert sum(int(c["candidates"]) for c in counts) > 0
    assert all(r == res[0] for r in res[1:])


@pytest.mark.parametrize("size", [(1242, 375), (64, 128), (520, 131), (513, 400)])
def test_pruned_alone_and_in_a_batch(size):
    """A pruned frame alone (its cell map by waves per cell row) and in a batch
    long enough for strips: the same boxes."""
    img = torch.from_numpy(pd_synth.frame(*size, 17)).to(DEV)
    rest = [torch.from_numpy(f).to(DEV) for f in pd_synth.frame_batch([(1242, 375)] * 6, 5)]
    wts = torch.from_numpy(pd_synth.svm_weights(1)).to(DEV)
    pruner = torch.from_numpy(np.random.default_rng(3).normal(0, 0.05, pd.PRUNER_PARAMS).astype(np.float32)).to(DEV)
    prm = pd.params(precision=pd.PREC_BF16, prune_keep=300, pruner=pruner)
    out = []
    for frames in ([img], rest + [img]):
        det = pd.Detector(frames, wts, torch.zeros(1, device=DEV), prm, cap=512)
        det.run(torch.full((len(frames),), -1.0e30, dtype=torch.float64, device=DEV))
        torch.cuda.synchronize()
        boxes, counts = det.results()
        b = boxes[-1].copy()
        b["frame"] = 0
        out.append((b.tobytes(), counts[-1].tobytes()))
    assert int(counts[-1]["candidates"]) > 0
    assert out[0] == out[1]
