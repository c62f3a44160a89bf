"""Detection on frames read in place at any alignment and pitch: exact."""
import numpy as np
import pytest

import pd_synth
from oracle import pd_oracle as O

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
import paper_1611_01642_amd as pd  # noqa: E402

DEV = "cuda:0"


def view_of(img, lead, pitch):
    """`img` on the device inside a larger buffer of 255s: rows `pitch` bytes
    apart, the first `lead` bytes in, the last row ending with the buffer."""
    h, w = img.shape
    buf = torch.full((lead + (h - 1) * pitch + w,), 255, dtype=torch.uint8, device=DEV)
    v = torch.as_strided(buf, (h, w), (pitch, 1), lead)
    v.copy_(torch.from_numpy(np.ascontiguousarray(img)))
    return v


@pytest.mark.parametrize("precision", [pd.PREC_F32, pd.PREC_BF16])
@pytest.mark.parametrize("w,h,lead,pitch", [(64, 128, 1, 64), (128, 203, 3, 131), (131, 137, 6, 133), (132, 136, 5, 132),
                                            (139, 144, 2, 139)])
def test_frames_in_place(w, h, lead, pitch, precision):
    """The last window column's halo, and the words around it, at each distance
    from the row's end; every window is rescored under BF16.  The frame as a
    view of any alignment against a copy with rows of its own 256 bytes."""
    img = pd_synth.frame(w, h, 90 + w)
    wts, bias = torch.from_numpy(pd_synth.svm_weights(2)).to(DEV), torch.zeros(2, device=DEV)
    prm = pd.params(precision=precision, margin=1.0e6)
    thr = torch.full((1,), -1.0e3, dtype=torch.float64, device=DEV)
    res = []
    for v in (view_of(img, lead, pitch), view_of(img, 0, 256)):
        det = pd.Detector([v], wts, bias, prm, cap=1024)
        det.run(thr)
        torch.cuda.synchronize()
        boxes, counts = det.results()
        # (the candidates' order is not defined)
        cs, ck, c64 = det.candidates(0)
        c64 = cs if c64 is None else c64  # FP64 scores under BF16 only
        cand = sorted((tuple(int(x) for x in k), float(s), float(d)) for s, k, d in zip(cs, ck, c64))
        res.append((boxes[0].tobytes(), counts[0].tobytes(), cand))
        n_win = sum(int(np.prod(O.window_grid(*s))) for s in O.level_sizes(w, h))
        assert counts[0]["candidates"] == n_win
        if precision == pd.PREC_BF16:
            # the oracle's FP64 scores of level 0 and the levels above it
            levels = O.frame_scores(img, pd_synth.svm_weights(2), np.zeros(2), clip=float(np.float32(0.2)),
                                    eps=float(np.float32(1e-3)))
            for s64, key in zip(c64, ck):
                ref = float(levels[int(key[0])]["scores"][:, int(key[1]), int(key[2])].max())
                assert abs(float(s64) - ref) <= 1e-9 * max(1.0, abs(ref)), key
    assert res[0] == res[1]
