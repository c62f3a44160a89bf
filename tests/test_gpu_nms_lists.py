"""NMS at the lengths where its sort and its batches of boxes change form, on
the largest frame side's boxes too, and the pruner's top-K over frames with
more windows than its LDS keeps: exact."""
import numpy as np
import pytest

import pd_synth
from oracle import pd_oracle as O

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
import paper_1611_01642_amd as pd  # noqa: E402

DEV = "cuda:0"


# 512: the longest list sorted by counting; 1024 boxes are taken at a time
@pytest.mark.parametrize("n", [2, 128, 129, 256, 257, 511, 512, 513, 1023, 1024, 1025, 2049])
@pytest.mark.parametrize("wh", [[(1242, 375), (1129, 340), (1026, 309)], [(16384, 16384), (14894, 14894)]])
def test_nms_lengths(n, wh):
    rng = np.random.default_rng(n)
    cands, seen = [], set()
    while len(cands) < n:
        k = int(rng.integers(0, len(wh)))
        ny, nx = O.window_grid(*wh[k])
        # corners of the largest grids among them
        i = int(rng.integers(0, ny) if rng.random() < 0.9 else ny - 1)
        j = int(rng.integers(0, nx) if rng.random() < 0.9 else nx - 1)
        if (k, i, j) in seen:
            continue
        seen.add((k, i, j))
        s = float(np.float32(rng.normal() if len(cands) % 5 else 0.75))  # ties
        cands.append({"score": s, "level": k, "i": i, "j": j, "model": 0,
                      "box": O.window_box_q8(*wh[0], *wh[k], i, j)})
    cs = torch.from_numpy(np.array([c["score"] for c in cands], np.float32)).to(DEV)
    ck = torch.from_numpy(np.array([[c["level"], c["i"], c["j"], 0] for c in cands], np.int32)).to(DEV)
    boxes, counts = pd.nms(cs, ck, wh, cap=n)
    got, cnt = pd.decode_boxes(boxes, counts)
    exp = O.nms(cands)
    assert cnt["candidates"] == n and cnt["kept"] == len(exp) and cnt["overflow"] == 0
    assert [(int(b["level"]), int(b["i"]), int(b["j"])) for b in got] == [(c["level"], c["i"], c["j"]) for c in exp]
    assert [tuple(int(b[k]) for k in ("x0", "y0", "x1", "y1")) for b in got] == [c["box"] for c in exp]


# 120,936 windows (read again in each pass) and 3 (all in one)
@pytest.mark.parametrize("w,h,keeps", [(1920, 1080, (1, 1000, 100000)), (80, 136, (1, 2, 3))])
def test_top_k(w, h, keeps):
    """With every window above the threshold, the pruned detector's candidates are the windows whose logit reaches the
    K-th largest: K of them, ties aside."""
    frame = torch.from_numpy(pd_synth.frame(w, h, 9)).to(DEV)
    weights, bias = torch.from_numpy(pd_synth.svm_weights(1)).to(DEV), torch.zeros(1, device=DEV)
    pruner = torch.from_numpy(pd_synth.pruner_init(seed=2)).to(DEV)
    thr = torch.full((1,), -1e30, dtype=torch.float64, device=DEV)
    sizes = [(L.w, L.h) for L in pd.plan_pyramid(w, h, pd.params())[0]]
    views = pd.build_pyramid(frame)[2]
    logits = []
    for (lw, lh), v in zip(sizes, views):
        z = pd.pruner_logits_bf16(v, pruner)
        ny, nx = O.window_grid(lw, lh)
        logits.append(z[7:7 + ny, 3:3 + nx].flatten())
    z = torch.cat(logits).cpu().numpy()
    for keep in keeps:
        det = pd.Detector([frame], weights, bias, pd.params(prune_keep=keep, pruner=pruner), cap=16)
        det.run(thr)
        torch.cuda.synchronize()
        n = int(det.counts.cpu().numpy().view(pd.COUNTS_DTYPE)[0]["candidates"])
        assert n == int((z >= np.sort(z)[::-1][keep - 1]).sum())
