"""NMS of long lists, sorted by buckets or, with many equal scores, by merging,
and of boxes whose overlap is exactly a half or one unit off it (levels twice as
coarse in one direction): exact."""
import numpy as np
import pytest

from oracle import pd_oracle as O

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
import paper_1611_01642_amd as pd  # noqa: E402

DEV = "cuda:0"

# level 1 has boxes exactly twice as wide as level 0's: nested ones overlap by
# exactly a half (kept); the other levels are just above and below that
HALVES = [(2048, 1024), (1024, 1024), (1025, 1024), (1023, 1024), (2048, 512), (2047, 513)]


def check(cands, wh, n):
    cs = torch.from_numpy(np.array([c["score"] for c in cands], np.float32)).to(DEV)
    ck = torch.from_numpy(np.array([[c["level"], c["i"], c["j"], 0] for c in cands], np.int32)).to(DEV)
    boxes, counts = pd.nms(cs, ck, wh, cap=n)
    got, cnt = pd.decode_boxes(boxes, counts)
    exp = O.nms(cands)
    key = [(c["level"], c["i"], c["j"]) for c in exp]
    assert [(int(b["level"]), int(b["i"]), int(b["j"])) for b in got] == key
    assert int(cnt["kept"]) == len(exp)


# ties: none (in the first score word); a fifth of the scores (64 of a bucket are
# still counted); all.  Runs of 64: one more and less than a power of two of
# them, a last run of one, the longest list; 17 groups of 64 after the first
@pytest.mark.parametrize("n", [65, 320, 321, 513, 577, 959, 1024, 1087, 1152, 1153, 2111, 4033, 4095, 4096])
@pytest.mark.parametrize("spread,ties", [(40, 0), (40, 5), (100, 0), (100, 1)])
def test_long_lists(n, spread, ties):
    rng = np.random.default_rng(n + spread)
    wh, cands, seen = HALVES, [], set()
    while len(cands) < n:
        k = int(rng.integers(0, len(wh)))
        ny, nx = O.window_grid(*wh[k])
        i, j = int(rng.integers(0, min(ny, spread))), int(rng.integers(0, min(nx, spread)))
        if (k, i, j) in seen:
            continue
        seen.add((k, i, j))
        s = 0.75 if ties and len(cands) % ties == 0 else float(np.float32(rng.normal()))
        cands.append({"score": s, "level": k, "i": i, "j": j, "model": 0, "box": O.window_box_q8(*wh[0], *wh[k], i, j)})
    check(cands, wh, n)


def test_halves():
    """Pairs of boxes, each far from the others: a box and one that overlaps it
    by a half, or a little more or less, in either order."""
    wh, cands = [(w * 8, h * 8) for w, h in HALVES], []
    q = 0
    for first in (0, 1):
        for k in range(1, len(wh)):
            for dj in (0, 1):
                x, y = (30 * q) % 900, 40 * ((30 * q) // 900)  # level 0 cells
                sx, sy = wh[k][0] / wh[0][0], wh[k][1] / wh[0][1]
                other = (k, int(y * sy), int(x * sx) + dj)
                for lv, i, j, s in ((0, y, x, 2.0 + first), (*other, 2.5)):
                    cands.append({"score": s, "level": lv, "i": i, "j": j, "model": 0,
                                  "box": O.window_box_q8(*wh[0], *wh[lv], i, j)})
                q += 1
    inter = [O.iou_exceeds_half(a["box"], b["box"]) for a, b in zip(cands[::2], cands[1::2])]
    assert 0 < sum(inter) < len(inter)
    check(cands, wh, len(cands))
