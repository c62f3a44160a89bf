"""Pyramid resampling where its loads change form (scales 2 and 6, images
narrower than a load) and at the edges of its tiles and rows: exact."""
import ctypes

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


def resample(v, sizes):
    """The levels `sizes` of the view, in one launch; bytes past each row's end too."""
    arr = (pd.Level * len(sizes))()
    off = 0
    for q, (w, h) in zip(arr, sizes):
        q.w, q.h, q.pitch, q.offset = w, h, (w + 15) // 16 * 16, off
        off += (q.pitch * h + 255) // 256 * 256
    out = torch.full((off,), 7, dtype=torch.uint8, device=DEV)
    rc = pd.lib().pd_build_pyramid(ctypes.c_void_p(v.data_ptr()), v.shape[1], v.shape[0], v.stride(0), arr, len(sizes),
                                   ctypes.c_void_p(out.data_ptr()), None)
    assert rc == 0
    torch.cuda.synchronize()
    out = out.cpu().numpy()
    return [out[q.offset:q.offset + q.pitch * q.h].reshape(q.h, q.pitch) for q in arr]


@pytest.mark.parametrize("w,h,lead,pitch", [(1, 1, 0, 1), (7, 9, 1, 7), (8, 70, 3, 11), (9, 33, 0, 16), (257, 131, 5, 259),
                                            (1024, 65, 2, 1027), (1337, 143, 7, 1337)])
def test_levels_of_any_size(w, h, lead, pitch):
    img = pd_synth.frame(max(w, 8), max(h, 8), 77 + w)[:h, :w]
    ws = {1, w, max(1, w - 1), (w + 1) // 2, w // 2 + 1, (w + 2) // 3, (w + 5) // 6, w // 6 + 1, max(1, w // 7), max(1, w * 10 // 11)}
    hs = {1, h, max(1, h - 1), (h + 1) // 2, max(1, h // 3), min(h, 15), min(h, 17), min(h, 64)}
    sizes = [(a, b) for a in sorted(w_ for w_ in ws if w_ <= w) for b in sorted(hs)]
    v = view_of(img, lead, pitch)
    for k in range(0, len(sizes), 32):
        for (lw, lh), got in zip(sizes[k:k + 32], resample(v, sizes[k:k + 32])):
            assert np.array_equal(got[:, :lw], O.resize(img, lw, lh)), (lw, lh)


@pytest.mark.parametrize("w,h", [(1242, 375), (4000, 3000)])
def test_many_tiles(w, h):
    # a few hundred tiles, and more than 8192: 16, 32 and 64 rows per tile
    sizes = [(w, h)] + [(w * 10 // (11 + k), h * 10 // (11 + k)) for k in range(31 if w > 2000 else 2)]
    img = pd_synth.frame(w, h, 5)
    v = view_of(img, 1, w + 3)
    for (lw, lh), got in zip(sizes, resample(v, sizes)):
        assert np.array_equal(got[:, :lw], O.resize(img, lw, lh)), (lw, lh)
