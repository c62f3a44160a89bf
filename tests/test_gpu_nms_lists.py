"""NMS at the lengths where its sort and its batches of boxes change form, on
the largest frame side's boxes too: exact."""
import numpy as np
import pytest

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
