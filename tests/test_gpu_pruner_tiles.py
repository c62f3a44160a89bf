"""The pruner's training kernels at the edges of their tiles (64 cells of a
row, 16 cells per matrix tile) and with more tiles than workgroups, against
the FP64 oracle: logits and gradients within 1e-5, the same bits twice."""
import numpy as np
import pytest

import pd_synth
from oracle import pruner_oracle as P

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
import paper_1611_01642_amd as pd  # noqa: E402

DEV = "cuda:0"


# (hc, wc): one cell; 16 and 64 cells and one more or less; a single row; 600 tiles
@pytest.mark.parametrize("sizes", [[(1, 1)], [(2, 15), (3, 16), (1, 17)], [(4, 31), (2, 32), (5, 33), (3, 48)],
                                   [(7, 63), (1, 64), (6, 65)], [(3, 127), (2, 129)], [(300, 70)]])
def test_logits_and_gradient(sizes):
    rng = np.random.default_rng(len(sizes) * 100 + sizes[0][1])
    params = pd_synth.pruner_init(seed=5)
    maps, labels, masks = [], [], []
    for hc, wc in sizes:
        m = rng.random((68, hc, wc))
        m[:9] /= np.sqrt((m[:9] ** 2).sum(axis=0, keepdims=True))
        maps.append(m.astype(np.float32))
        labels.append((rng.random((hc, wc)) < 0.3).astype(np.float32))
        masks.append((rng.random((hc, wc)) < 0.9).astype(np.float32))
    masks[0][0, 0] = 1.0
    to = lambda a: torch.from_numpy(a).to(DEV)  # noqa: E731
    b = pd.PrunerBatch([to(m) for m in maps], [to(x) for x in labels], [to(x) for x in masks])
    w = to(params)
    grad = b.gradient(w, 3.5).clone()
    stats = b.stats.clone()
    assert torch.equal(b.gradient(w, 3.5).view(torch.int32), grad.view(torch.int32))
    torch.cuda.synchronize()
    p64 = params.astype(np.float64)
    fwd = [P.forward(m.transpose(1, 2, 0).astype(np.float64), p64) for m in maps]
    for z, (exp, _) in zip(b.logits, fwd):
        assert np.abs(z.cpu().numpy() - exp).max() <= 1e-5 * max(1.0, np.abs(exp).max())
    loss, dl = P.bce_loss_grad([z for z, _ in fwd], [x.astype(np.float64) for x in labels],
                               [x.astype(np.float64) for x in masks], 3.5)
    exp = sum(P.backward(d, c, p64) for d, (_, c) in zip(dl, fwd))
    got = grad.cpu().numpy()
    assert np.abs(got - exp).max() <= 1e-5 * np.abs(exp).max()
    assert abs(float(stats[0]) - loss) <= 1e-6 * max(1.0, abs(loss)) and float(stats[1]) == sum(x.sum() for x in masks)
