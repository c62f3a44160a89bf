"""tune_grid caps the feature and scoring grids of a call of any size: with one
workgroup a small call gives the same bytes and takes many times as long as over
the whole chip (which a call that ignores the cap would not)."""
import numpy as np
import pytest

import pd_synth

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
import paper_1611_01642_amd as pd  # noqa: E402

DEV = "cuda:0"


@pytest.mark.parametrize("kw,stages", [(dict(), ("features", "score")), (dict(features=pd.FEAT_LBP), ("features", "score")),
                                       (dict(precision=pd.PREC_BF16), ("features",)),
                                       (dict(precision=pd.PREC_BF16, prune=1), ("features",))])
def test_one_workgroup(kw, stages):
    kw = dict(kw)
    if kw.pop("prune", 0):
        pruner = torch.from_numpy(np.random.default_rng(3).normal(0, 0.05, pd.PRUNER_PARAMS).astype(np.float32)).to(DEV)
        kw.update(prune_keep=300, pruner=pruner)
    img = torch.from_numpy(pd_synth.frame(640, 480, 41)).to(DEV)
    wts = torch.from_numpy(pd_synth.svm_weights(1)).to(DEV)
    thr = torch.full((1,), 1.5, dtype=torch.float64, device=DEV)
    out, ms = [], []
    for grid in (0, 1):
        det = pd.Detector([img], wts, torch.zeros(1, device=DEV), pd.params(tune_grid=grid, **kw), cap=512)
        pd.profile_enable(True)
        try:
            det.capture_steps(thr, 1)
        finally:
            pd.profile_enable(False)
        least = {}
        for _ in range(3):
            det.replay_step(0)
            torch.cuda.synchronize()
            least = {k: min(v, least.get(k, v)) for k, v in det.step_stage_ms(0).items()}
        boxes, counts = det.results()
        out.append((boxes[0].tobytes(), counts.tobytes()))
        ms.append(least)
        det.release()
    assert int(counts[0]["candidates"]) > 0
    assert out[0] == out[1]
    for stage in stages:
        print(f"\n[grid cap] {kw} {stage}: {ms[0][stage]:.3f} ms, one workgroup {ms[1][stage]:.3f} ms", flush=True)
        assert ms[1][stage] > 4.0 * ms[0][stage]
