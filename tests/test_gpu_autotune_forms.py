"""pd_autotune times what its candidates change: for a call whose forms take no
notice of a field it returns that field's starting value, every time, and for a
call in strips it starts from the rows the call takes by itself."""
import numpy as np
import pytest

import pd_synth

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
import paper_1611_01642_amd as pd  # noqa: E402

DEV = "cuda:0"


def detector(sizes, prm):
    frames = [torch.from_numpy(f).to(DEV) for f in pd_synth.frame_batch(sizes, 90)]
    wts = torch.from_numpy(pd_synth.svm_weights(1)).to(DEV)
    thr = torch.full((len(sizes),), 3.0, dtype=torch.float64, device=DEV)
    return pd.Detector(frames, wts, torch.zeros(1, device=DEV), prm, cap=1024), thr


def test_fields_without_effect_keep_their_start():
    for k in range(5):
        det, thr = detector([(640, 480)], pd.params())
        tuning, ms = det.autotune(thr, iters=1)
        print(f"\n[autotune] one 640x480 frame, run {k}: {tuning} {ms:.3f} ms", flush=True)
        assert tuning["tune_feat_rows"] == 8 and tuning["tune_score_rows"] == 8
        assert 0.0 < ms < 1000.0
    det, thr = detector([(640, 480)], pd.params(tune_feat_rows=12, tune_score_rows=16))
    tuning, _ = det.autotune(thr, iters=1)
    assert tuning["tune_feat_rows"] == 12 and tuning["tune_score_rows"] == 16


def test_no_slower_than_the_default():
    """16 frames of 1242x375 take strips of an odd number of rows by themselves."""
    sizes = [(1242, 375)] * 16
    det, thr = detector(sizes, pd.params())
    tuning, _ = det.autotune(thr, iters=3)
    det.run(thr)
    torch.cuda.synchronize()
    got = det.results()
    ref, _ = detector(sizes, pd.params())
    ref.run(thr)
    torch.cuda.synchronize()
    exp = ref.results()
    assert got[1].tobytes() == exp[1].tobytes() and sum(int(c["candidates"]) for c in exp[1]) > 0
    assert all(a.tobytes() == b.tobytes() for a, b in zip(got[0], exp[0]))
    times = {}
    for name, d in (("default", ref), ("tuned", det)):
        d.capture(thr)
    for _ in range(5):
        for name, d in (("default", ref), ("tuned", det)):
            e0, e1 = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
            e0.record()
            for _ in range(20):
                d.replay()
            e1.record()
            torch.cuda.synchronize()
            times[name] = min(times.get(name, 1e9), e0.elapsed_time(e1) / 20)
    print(f"\n[autotune] 16 frames: {tuning}, default {times['default']:.4f} ms, tuned {times['tuned']:.4f} ms", flush=True)
    assert times["tuned"] < 1.05 * times["default"]
