"""The work that programs built on libpd have it do, one dict per case.

`listed()` names the cases, `draw(rng)` makes further ones of the same ranges,
`prepare` builds what a program holds before a call, `run` is one pass through
the package's public entry points, `work` what such a pass cannot do without,
and `exact` its result in 64 bits, in plain torch.

The kinds of calls:
  detect    the whole detector on a batch of resident frames (pd_detect or the
            replay of a captured graph), FP32 or BF16 MFMA + FP64 rescore, all
            features or one family, pruned or not
  features  HOG blocks and LBP cell histograms of one image
  score     every window of one image's features against linear SVMs
  maps      training targets of the window pruner from one frame: pyramid, cell
            maps, plain scores and labels of every level
  train     one training step of the window pruner: gradient and Adam
  video     a clip of host frames through the streaming object
"""
import math

import numpy as np
import torch

import paper_1611_01642_amd as pd
from paper_1611_01642_amd import pruner_train

DEV = "cuda:0"
CH = (68, 32, 32, 16)  # channels of the window pruner
LR, STEP = 2e-3, 200  # the pruner's optimiser: learning rate, steps taken
CAP = 1024  # boxes kept per frame


def listed():
    return [
        # the smallest detector call: one 320x240 frame, three levels at 6/5 (the smoke check's and unit tests' shape)
        _detect("detect_small", "320x240x1", num=6, den=5, levels=3),
        # one camera frame, full pyramid, called eagerly: a driver-assistance loop's latency
        _detect("detect_frame", "1242x375x1"),
        # a recorded sequence, 256 frames per call, as the replay of a captured graph: throughput
        _detect("detect_batch256", "1242x375x256", graph=True),
        # cameras of three resolutions in one call, a new batch each time (eager)
        _detect("detect_mixed64", "640x480x24,1242x375x24,1920x1080x16"),
        # throughput form of the same detector: BF16 scoring, decisions in FP64
        _detect("detect_bf16", "1242x375x64", precision="bf16"),
        # several detectors (object classes, poses) over the same frames
        _detect("detect_bf16_8svm", "1242x375x32", precision="bf16", models=8),
        # the learned window pruner in front of the BF16 detector, half of the windows kept
        _detect("detect_pruned", "1242x375x16", precision="bf16", keep=9200),
        # descriptors of one image for a program that trains its own classifier; 375 rows and a pitch of 1242
        # bytes: ragged cells and rows that are not 8-byte aligned
        {"name": "features_image", "kind": "features", "w": 1242, "h": 375, "bf16": False},
        # scores of all windows of one level, as hard-negative mining reads them
        {"name": "score_image", "kind": "score", "w": 1242, "h": 375, "models": 1},
        # one frame's share of the pruner's training set
        {"name": "pruner_maps", "kind": "maps", "w": 1242, "h": 375, "models": 1},
        # one optimiser step of the pruner on the usual eight frames
        {"name": "pruner_step", "kind": "train", "w": 1242, "h": 375, "frames": 8},
        # eight frames of live video from host memory, three in flight
        {"name": "video_clip", "kind": "video", "w": 1242, "h": 375, "frames": 8, "depth": 3},
    ]


def _detect(name, frames, num=11, den=10, levels=0, precision="f32", models=1, features="both", keep=0, graph=False):
    case = {"kind": "detect", "frames": frames, "num": num, "den": den, "levels": levels, "precision": precision,
            "models": models, "features": features, "keep": keep, "graph": graph}
    return {"name": name, **case} if name else case


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["detect"] * 6 + ["features", "score", "maps", "train", "video"])
    if kind == "detect":
        models = rng.choice([1, 1, 1, 2, 3, 8])
        parts, left = [], 24_000_000 if models < 8 else 12_000_000  # pixels of the batch at most
        for _ in range(rng.choice([1, 1, 2, 3])):
            w, h = _log(rng, 96, 1920), _log(rng, 144, 1080)
            n = min(_log(rng, 1, 64), left // (w * h))
            if n:
                parts.append("%dx%dx%d" % (w, h, n))
                left -= w * h * n
        precision = rng.choice(["f32", "f32", "bf16"])
        features = rng.choice(["both"] * 4 + ["hog", "lbp"])
        num, den, levels = rng.choice([(11, 10, 0), (11, 10, 0), (6, 5, 0), (6, 5, 3), (13, 10, 0)])
        keep = _log(rng, 64, 8192) if features == "both" and precision == "bf16" and rng.random() < 0.3 else 0
        return _detect(None, ",".join(parts), num, den, levels, precision, models, features,
                       keep, rng.random() < 0.4)
    if kind == "features":
        return {"kind": kind, "w": _log(rng, 24, 3840), "h": _log(rng, 24, 2160), "bf16": rng.random() < 0.25}
    if kind == "score":
        return {"kind": kind, "w": _log(rng, 80, 3840), "h": _log(rng, 144, 2160), "models": rng.choice([1, 1, 2, 3])}
    if kind == "maps":
        return {"kind": kind, "w": _log(rng, 96, 1280), "h": _log(rng, 144, 720), "models": rng.choice([1, 1, 2])}
    if kind == "train":
        return {"kind": kind, "w": _log(rng, 96, 1242), "h": _log(rng, 144, 480), "frames": rng.randint(1, 8)}
    return {"kind": kind, "w": _log(rng, 96, 1920), "h": _log(rng, 144, 1080), "frames": rng.randint(1, 8),
            "depth": rng.randint(1, 4)}


# ---------------------------------------------------------------- inputs --
def _sizes(case):
    if case["kind"] != "detect":
        return [(case["w"], case["h"])] * case.get("frames", 1)
    out = []
    for part in case["frames"].split(","):
        w, h, n = (int(v) for v in part.split("x"))
        out += [(w, h)] * n
    return out


def _same_size_frames(n, w, h, seed):
    """uint8 [n][h][w] road-like frames: a smooth background with sensor noise, bright and dark boxes, step edges."""
    g = torch.Generator(device=DEV).manual_seed(seed)
    rng = np.random.default_rng(seed)
    grid = torch.rand((n, 1, -(-h // 16) + 2, -(-w // 16) + 2), device=DEV, generator=g) * 160 + 48
    img = torch.nn.functional.interpolate(grid, scale_factor=16, mode="bilinear", align_corners=False)
    img = img[:, 0, :h, :w].contiguous()
    img += torch.randn((n, h, w), device=DEV, generator=g) * 4
    noise = torch.randn((n, h, w), device=DEV, generator=g) * 4
    ys, xs = torch.arange(h, device=DEV).view(1, h, 1), torch.arange(w, device=DEV).view(1, 1, w)
    for k in range(20):
        def per_frame(v):
            return torch.as_tensor(np.asarray(v, dtype=np.float32), device=DEV).view(n, 1, 1)
        if k % 4:
            bw, bh = rng.integers(8, max(9, w // 4 + 1), n), rng.integers(16, max(17, h // 2 + 1), n)
            x0, y0 = rng.integers(-(bw // 2), w), rng.integers(-(bh // 2), h)
            val = per_frame(np.where(rng.random(n) < 0.5, rng.uniform(200, 255, n), rng.uniform(0, 55, n)))
            inside = ((xs >= per_frame(x0)) & (xs < per_frame(x0 + bw))) & ((ys >= per_frame(y0)) & (ys < per_frame(y0 + bh)))
            img = torch.where(inside, val + noise, img)
        else:
            ang, off = rng.uniform(0, np.pi, n), rng.uniform(30, 80, n) * rng.choice([-1.0, 1.0], n)
            side = (xs - per_frame(rng.uniform(0, w, n))) * per_frame(np.sin(ang)) \
                - (ys - per_frame(rng.uniform(0, h, n))) * per_frame(np.cos(ang)) > 0
            img += per_frame(off) * side
    return img.round().clamp(0, 255).to(torch.uint8)


def _frames(sizes, seed):
    """One uint8 CUDA tensor [h][w] per size."""
    out, at = [], 0
    while at < len(sizes):
        n = 1
        while at + n < len(sizes) and n < 32 and sizes[at + n] == sizes[at]:
            n += 1
        out += list(_same_size_frames(n, *sizes[at], seed * 1000 + at))
        at += n
    return out


def _weights(models, seed):
    """Linear SVMs w ~ N(0, 0.01^2), float32 [models][11332], and their biases."""
    rng = np.random.default_rng([seed, 7])
    w = rng.normal(0.0, 0.01, (models, pd.FEATURE_DIM)).astype(np.float32)
    b = rng.normal(0.0, 0.1, models).astype(np.float32)
    return torch.from_numpy(w).to(DEV), torch.from_numpy(b).to(DEV)


def _pruner(seed):
    """He-normal weights of the window pruner, biases zero."""
    rng = np.random.default_rng([seed, 11])
    parts = []
    for cin, cout in zip(CH[:-1], CH[1:]):
        parts += [rng.normal(0.0, math.sqrt(2.0 / (9 * cin)), cout * cin * 9), np.zeros(cout)]
    parts += [rng.normal(0.0, math.sqrt(1.0 / CH[-1]), CH[-1]), np.zeros(1)]
    return torch.from_numpy(np.concatenate(parts).astype(np.float32)).to(DEV)


def _cut(scores):
    """A threshold that about 1 % of a frame's windows exceed: the middle of the widest gap near that rank."""
    n = len(scores)
    s = np.sort(np.asarray(scores, dtype=np.float64))[::-1]
    if n < 2:
        return float(s[0]) - 1.0 if n else 0.0
    k = min(-(-n // 100), n - 1)
    gaps = s[k - 1:k + 7] - s[k:k + 8][:len(s[k - 1:k + 7])] if n > k + 8 else s[k - 1:k] - s[k:k + 1]
    g = int(np.argmax(gaps))
    return float(0.5 * (s[k - 1 + g] + s[k + g]))


def _params(case, **more):
    feat = {"both": pd.FEAT_HOG | pd.FEAT_LBP, "hog": pd.FEAT_HOG, "lbp": pd.FEAT_LBP}[case["features"]]
    return pd.params(scale=(case["num"], case["den"]), max_levels=case["levels"], features=feat, **more)


def _thresholds(frames, weights, bias, prm):
    """Each frame's threshold, from the plain scores of all its windows."""
    out = []
    for at in range(0, len(frames), 32):
        part = frames[at:at + 32]
        det = pd.Detector(part, weights, bias, prm, cap=16)
        det.run(torch.full((len(part),), -1e30, dtype=torch.float64, device=DEV))
        out += [_cut(det.candidates(f)[0]) for f in range(len(part))]
    return out


def _tensor(values):
    return torch.tensor(values, dtype=torch.float64, device=DEV)


def prepare(case, seed):
    kind = case["kind"]
    if kind == "detect":
        frames = _frames(_sizes(case), seed)
        weights, bias = _weights(case["models"], seed)
        thr = _tensor(_thresholds(frames, weights, bias, _params(case)))
        prec = {"f32": pd.PREC_F32, "bf16": pd.PREC_BF16}[case["precision"]]
        pruner = _pruner(seed) if case["keep"] else None
        det = pd.Detector(frames, weights, bias, _params(case, precision=prec, prune_keep=case["keep"], pruner=pruner), CAP)
        det.boxes.zero_()  # a frame's entries past its kept boxes are never written
        n = len(frames)
        words = det.boxes.view(torch.int32).view(n, CAP, 12)
        outputs = {"boxes": words[..., :9], "score": words.view(torch.float32)[..., 9],
                   "score64": det.boxes.view(torch.float64).view(n, CAP, 6)[..., 5], "counts": det.counts.view(torch.int32).view(n, 4)}
        if case["graph"]:
            det.capture(thr)
        return {"kind": kind, "det": det, "thr": thr, "graph": case["graph"], "pruner": pruner, "outputs": outputs}
    if kind == "features":
        return {"kind": kind, "img": _frames(_sizes(case), seed)[0], "bf16": case["bf16"], "prm": pd.params()}
    if kind == "score":
        blocks, cells = pd.features(_frames(_sizes(case), seed)[0])
        weights, bias = _weights(case["models"], seed)
        return {"kind": kind, "args": (blocks, cells, weights, bias)}
    if kind == "maps":
        img = _frames(_sizes(case), seed)[0]
        weights, bias = _weights(case["models"], seed)
        prm = pd.params()
        return {"kind": kind, "args": (img, weights, bias, _tensor(_thresholds([img], weights, bias, prm)), prm)}
    if kind == "train":
        maps, labels, masks, pos_weight, start = _training_inputs(case, seed)
        return {"kind": kind, "batch": pd.PrunerBatch(maps, labels, masks), "start": start, "now": start.clone(), "pos_weight": pos_weight}
    frames = _frames(_sizes(case), seed)
    weights, bias = _weights(1, seed)
    return {"kind": kind, "frames": [f.cpu().numpy() for f in frames], "thr": _thresholds(frames, weights, bias, pd.params()),
            "depth": case["depth"], "outputs": _clip_results(len(frames)), "video": pd.Video(case["w"], case["h"], weights, bias, cap=CAP, depth=case["depth"])}


def _clip_results(n):
    """Where the program gathers a clip's results: a frame's rows past its kept boxes stay zero."""
    return {"boxes": np.zeros((n, CAP, 9), np.int32), "score": np.zeros((n, CAP), np.float32), "counts": np.zeros((n, 4), np.int32)}


def _training_inputs(case, seed):
    """(cell maps, labels, masks, positive weight, [parameters, Adam's m, v]) of a step in the middle of a training, float32."""
    maps, labels, masks = [], [], []
    g = torch.Generator(device=DEV).manual_seed(seed)
    for img in _frames(_sizes(case), seed):
        for level in _pyramid(img, 11, 10, 0):
            m = _features(level)["map"].float()
            y, x = torch.zeros(m.shape[1:], device=DEV), torch.zeros(m.shape[1:], device=DEV)
            ny, nx = m.shape[1] - 15, m.shape[2] - 7
            x[7:7 + ny, 3:3 + nx] = 1.0
            # positives gather where the gradient is strong, about one window in a hundred
            rank = m[2:5, 7:7 + ny, 3:3 + nx].sum(0) + torch.rand((ny, nx), device=DEV, generator=g)
            y[7:7 + ny, 3:3 + nx] = (rank >= rank.flatten().kthvalue(max(1, ny * nx - ny * nx // 100)).values).float()
            maps.append(m)
            labels.append(y)
            masks.append(x)
    n_pos, n_all = sum(float(y.sum()) for y in labels), sum(float(x.sum()) for x in masks)
    p = _pruner(seed)
    m, v = torch.randn(p.shape, device=DEV, generator=g) * 1e-3, (torch.rand(p.shape, device=DEV, generator=g) + 0.5) * 1e-4
    return maps, labels, masks, (n_all - n_pos) / max(n_pos, 1.0), torch.stack([p, m, v])


# ------------------------------------------------------------------- run --
def run(s):
    kind = s["kind"]
    if kind == "detect":
        if s["graph"]:
            s["det"].replay()
        else:
            s["det"].run(s["thr"])
        return s["outputs"]
    if kind == "features":
        return pd.features(s["img"], s["prm"], bf16=s["bf16"])
    if kind == "score":
        return pd.score_windows(*s["args"])
    if kind == "maps":
        return pruner_train.level_maps(*s["args"])
    if kind == "train":
        b, (p, m, v) = s["batch"], s["now"].copy_(s["start"])  # the same step again in each pass
        b.gradient(p, s["pos_weight"])
        pd.adam_step(p, b.grad, m, v, STEP, lr=LR)
        return {"grad": b.grad, "state": s["now"], "stats": b.stats}
    out, video, pushed = s["outputs"], s["video"], 0
    for k in range(len(s["frames"])):
        while pushed < min(k + s["depth"], len(s["frames"])):
            video.push(s["frames"][pushed], s["thr"][pushed])
            pushed += 1
        b, c, _ = video.pop()
        out["boxes"][k, :len(b)] = b.view(np.int32).reshape(-1, 12)[:, :9]
        out["score"][k, :len(b)] = b["score"]
        out["counts"][k] = c.reshape(1).view(np.int32)
    return out


# ------------------------------------------------------------------ work --
def _levels(w, h, num=11, den=10, limit=0):
    out = []
    while not limit or len(out) < limit:
        k = len(out)
        wk, hk = w * den ** k // num ** k, h * den ** k // num ** k
        if wk < 64 or hk < 128:
            break
        out.append((wk, hk))
    return out


def _windows(w, h):
    return max(0, h // 8 - 15) * max(0, w // 8 - 7)


def _macs(case):
    """Multiply-adds of the pruner's network per cell."""
    return sum(9 * a * b for a, b in zip(CH[:-1], CH[1:])) + CH[-1]


def work(case):
    """Bytes: every input and result once.  Flops: 40 per pixel for the gradients, orientations, votes and LBP codes, two per
    feature, model and window, two per weight and cell of the network (three times that in training)."""
    kind, b, f = case["kind"], 0, 0
    if kind in ("detect", "video", "maps"):
        models = case.get("models", 1)
        for w, h in _sizes(case):
            levels = _levels(w, h, case.get("num", 11), case.get("den", 10), case.get("levels", 0))
            n = sum(_windows(*wh) for wh in levels)
            dim = {"both": 11332, "hog": 3780, "lbp": 7552}[case.get("features", "both")]
            keep = case.get("keep", 0)
            b += w * h + n // 100 * 48
            f += 40 * sum(x * y for x, y in levels) + 2 * dim * models * (min(keep, n) if keep else n)
            if keep:
                f += 2 * _macs(case) * sum((x // 8) * (y // 8) for x, y in levels)
            if kind == "maps":
                b += 70 * 4 * sum((x // 8) * (y // 8) for x, y in levels)
        b += models * 11332 * 4
    elif kind == "features":
        hc, wc = case["h"] // 8, case["w"] // 8
        b = case["w"] * case["h"] + 59 * hc * wc + 36 * (2 if case["bf16"] else 4) * max(0, hc - 1) * max(0, wc - 1)
        f = 40 * case["w"] * case["h"]
    elif kind == "score":
        hc, wc = case["h"] // 8, case["w"] // 8
        n = _windows(case["w"], case["h"])
        b = 59 * hc * wc + 144 * (hc - 1) * (wc - 1) + case["models"] * (4 * n + 4 * 11332)
        f = 2 * 11332 * n * case["models"]
    else:
        cells = case["frames"] * sum((x // 8) * (y // 8) for x, y in _levels(case["w"], case["h"]))
        b, f = cells * 70 * 4 + 7 * 33505 * 4, 6 * _macs(case) * cells
    return {"bytes": int(b), "flops": int(f)}


# ----------------------------------------------------------- in 64 bits --
def _pyramid(img, num, den, limit):
    """The levels of a uint8 image: bilinear samples at 8-bit fractions, rounded half up."""
    def axis(n0, nk):
        x = torch.arange(nk, dtype=torch.int64, device=img.device)
        q = ((2 * x + 1) * n0 - nk) * 128 // nk
        return q >> 8, q & 255, ((q >> 8) + 1).clamp(max=n0 - 1)
    h0, w0 = img.shape
    out = []
    for wk, hk in _levels(w0, h0, num, den, limit):
        (x0, fx, x1), (y0, fy, y1) = axis(w0, wk), axis(h0, hk)
        p = img.to(torch.int64)
        top, bot = (p[y][:, x0] * (256 - fx) + p[y][:, x1] * fx for y in (y0, y1))
        out.append(((top * (256 - fy)[:, None] + bot * fy[:, None] + 32768) >> 16).to(torch.uint8))
    return out


def _uniform_bins():
    table, nxt = [], 0
    for code in range(256):
        turns = bin(code ^ ((code >> 1) | (code & 1) << 7)).count("1")
        table.append(nxt if turns <= 2 else 58)
        nxt += turns <= 2
    return torch.tensor(table, device=DEV)


def _features(img, clip=0.2, eps=1e-3):
    """{"hog": [36][Hb][Wb], "lbp": [59][Hc][Wc], "map": [68][Hc][Wc]} of one level in float64."""
    clip, eps = float(np.float32(clip)), float(np.float32(eps))
    h, w = img.shape
    hc, wc = h // 8, w // 8
    p = img.double()[torch.arange(-1, h + 1, device=DEV).clamp(0, h - 1)][:, torch.arange(-1, w + 1, device=DEV).clamp(0, w - 1)]

    def at(dy, dx):  # the neighbour's value for every pixel of the cell grid
        return p[1 + dy:1 + dy + 8 * hc, 1 + dx:1 + dx + 8 * wc]

    def per_cell(index, value, bins):
        v = torch.zeros((bins, 8 * hc * 8 * wc), dtype=torch.float64, device=DEV)
        return v.scatter_add_(0, index.reshape(1, -1), value.reshape(1, -1))

    dx, dy = at(0, -1) - at(0, 1), at(-1, 0) - at(1, 0)
    mag = torch.sqrt(dx * dx + dy * dy)
    t = torch.rad2deg(torch.atan2(dy, dx)) % 180.0 / 20.0 - 0.5
    low = t.floor()
    b0, up = low.long() % 9, t - low
    votes = per_cell(b0, mag * (1 - up), 9) + per_cell((b0 + 1) % 9, mag * up, 9)
    # every pixel's share for its own cell and the neighbours, bilinear in the distance to their centres: A[bin][cy][dy][cx][dx]
    off = torch.arange(8, dtype=torch.float64, device=DEV) + 0.5
    share = torch.stack([(1 - (off - (8 * d + 4)).abs() / 8).clamp(min=0) for d in (-1, 0, 1)])
    A = votes.view(9, hc, 8, wc, 8) @ share.t()
    A = (A.permute(0, 1, 3, 4, 2) @ share.t()).permute(0, 1, 4, 2, 3)
    hog = []
    for r in (0, 1):
        for c in (0, 1):
            hog.append(sum(A[:, i:i + hc - 1, 1 + r - i, j:j + wc - 1, 1 + c - j] for i in (0, 1) for j in (0, 1)))
    v = torch.cat(hog)
    v = (v / torch.sqrt((v * v).sum(0) + eps * eps)).clamp(max=clip)
    v = v / torch.sqrt((v * v).sum(0) + eps * eps)
    hist = torch.zeros((9, hc + 2, wc + 2), dtype=torch.float64, device=DEV)
    for i in (-1, 0, 1):
        for j in (-1, 0, 1):
            hist[:, 1 + i:1 + i + hc, 1 + j:1 + j + wc] += A[:, :, 1 + i, :, 1 + j]
    hist = hist[:, 1:-1, 1:-1]
    hist = hist / torch.sqrt((hist * hist).sum(0) + eps * eps)
    around = [(-1, -1), (-1, 0), (-1, 1), (0, 1), (1, 1), (1, 0), (1, -1), (0, -1)]
    code = sum((at(*d) >= at(0, 0)).long() << k for k, d in enumerate(around))
    ones = per_cell(_uniform_bins()[code], torch.ones_like(mag), 59)
    lbp = ones.view(59, hc, 8, wc, 8).sum((2, 4))
    return {"hog": v, "lbp": lbp, "map": torch.cat([hist, lbp / 64])}


def _scores(feat, weights, bias, features="both"):
    """[models][ny][nx] in float64."""
    hog, lbp, w = feat["hog"], feat["lbp"], weights.double()
    m, ny, nx = len(w), lbp.shape[1] - 15, lbp.shape[2] - 7
    out = bias.double().view(m, 1, 1).expand(m, ny, nx).clone()
    for plane, rows, cols, part, on in ((hog, 15, 7, w[:, :3780], features != "lbp"), (lbp, 16, 8, w[:, 3780:], features != "hog")):
        part = part.view(m, rows, cols, -1)
        for a in range(rows if on else 0):
            for b in range(cols):
                out += (part[:, a, b] @ plane[:, a:a + ny, b:b + nx].reshape(plane.shape[0], -1)).view(m, ny, nx)
    return out


def _kept(img, weights, bias, num, den, limit, features="both"):
    """(box rows in the order of greedy suppression, their scores, candidates) of one frame."""
    h0, w0 = img.shape
    found, every = [], []
    for k, level in enumerate(_pyramid(img, num, den, limit)):
        s, m = _scores(_features(level), weights, bias, features).max(0)
        every.append(s.flatten().cpu().numpy())
        found.append((k, level.shape, s.cpu().numpy(), m.cpu().numpy()))
    thr = _cut(np.concatenate(every)) if every else 0.0
    rows = []
    for k, (hk, wk), s, m in found:
        for i, j in zip(*(v.tolist() for v in np.nonzero(s > thr))):
            rows.append((-s[i, j], k, i, j, int(m[i, j]), 2048 * j * w0 // wk, 2048 * i * h0 // hk,
                         256 * (8 * j + 64) * w0 // wk, 256 * (8 * i + 128) * h0 // hk))
    rows.sort()
    kept = np.zeros((0, 9))
    for r in rows:
        r = np.array(r)
        inter = (np.minimum(kept[:, 7], r[7]) - np.maximum(kept[:, 5], r[5])).clip(0) \
            * (np.minimum(kept[:, 8], r[8]) - np.maximum(kept[:, 6], r[6])).clip(0)
        both = (kept[:, 7] - kept[:, 5]) * (kept[:, 8] - kept[:, 6]) + (r[7] - r[5]) * (r[8] - r[6]) - inter
        if not (2 * inter > both).any():
            kept = np.vstack([kept, r])
    return kept, len(rows), thr


def exact(case, seed):
    kind = case["kind"]
    if kind in ("detect", "video"):
        sizes = _sizes(case)
        if kind == "detect" and (case["keep"] or sum(w * h for w, h in sizes) > 2_000_000):
            return None
        weights, bias = _weights(case.get("models", 1), seed)
        frames = _frames(sizes, seed)
        num, den, limit = case.get("num", 11), case.get("den", 10), case.get("levels", 0)
        bf16 = case.get("precision") == "bf16"
        got = []
        for f, img in enumerate(frames):
            kept, n, thr = _kept(img, weights, bias, num, den, limit, case.get("features", "both"))
            k = min(len(kept), CAP)
            score = -kept[:k, 0]
            boxes = np.concatenate([np.full((k, 1), f if kind == "detect" else 0), kept[:k, 1:]], 1).astype(np.int32)
            score64 = np.where(np.abs(score - thr) < 0.05, score, np.nan) if bf16 else np.full(k, np.nan)
            got.append((boxes, score, score64, np.array([n, k, 0, 0], np.int32)))

        def whole(i):
            out = np.zeros((len(got), CAP) + got[0][i].shape[1:], got[0][i].dtype)
            for f, g in enumerate(got):
                out[f, :len(g[i])] = g[i]
            return out
        if kind == "video":
            return {"boxes": whole(0), "score": whole(1), "counts": np.stack([g[3] for g in got])}
        return {"boxes": whole(0), "score": whole(1), "score64": whole(2) if bf16 else None,
                "counts": None if bf16 else np.stack([g[3] for g in got])}
    if kind == "features":
        f = _features(_frames(_sizes(case), seed)[0])
        return f["hog"], f["lbp"].to(torch.uint8)
    if kind == "score":
        img = _frames(_sizes(case), seed)[0]
        return _scores(_features(img), *_weights(case["models"], seed))
    if kind == "maps":
        levels = [_features(v) for v in _pyramid(_frames(_sizes(case), seed)[0], 11, 10, 0)]
        scores = [_scores(f, *_weights(case["models"], seed)).max(0).values for f in levels]
        thr = _cut(torch.cat([s.flatten() for s in scores]).cpu().numpy()) if levels else 0.0
        out = []
        for f, s in zip(levels, scores):
            label, mask = torch.zeros_like(f["lbp"][0]), torch.zeros_like(f["lbp"][0])
            label[7:7 + s.shape[0], 3:3 + s.shape[1]] = (s > thr).double()
            mask[7:7 + s.shape[0], 3:3 + s.shape[1]] = 1.0
            out.append((f["map"], label, mask))
        return out
    return _exact_step(case, seed)


def _exact_step(case, seed):
    maps, labels, masks, pos_weight, start = _training_inputs(case, seed)
    p0, m0, v0 = start.double()
    p = p0.clone().requires_grad_()
    layers, at = [], 0
    for cin, cout in zip(CH[:-1], CH[1:]):
        n = cout * cin * 9
        layers.append((p[at:at + n].view(cout, cin, 3, 3), p[at + n:at + n + cout]))
        at += n + cout
    pos_weight = float(np.float32(pos_weight))
    total, loss = sum(float(x.sum()) for x in masks), 0.0
    for x, label, mask in zip(maps, labels, masks):
        x = x.double()
        h, w = x.shape[1:]
        for wgt, b in layers:
            xp = torch.nn.functional.pad(x, (1, 1, 1, 1))
            x = b[:, None] + sum(wgt[:, :, u, v] @ xp[:, u:u + h, v:v + w].reshape(xp.shape[0], -1) for u in range(3) for v in range(3))
            x = torch.relu(x).view(-1, h, w)
        z = (p[at:at + CH[-1]] @ x.reshape(CH[-1], -1)).view(h, w) + p[-1]
        soft = torch.nn.functional.softplus
        part = (mask.double() * (pos_weight * label * soft(-z) + (1 - label) * soft(z))).sum() / total
        part.backward(retain_graph=True)
        loss += float(part.detach())
    g = p.grad
    b1, b2 = float(np.float32(0.9)), float(np.float32(0.999))
    m, v = b1 * m0 + (1 - b1) * g, b2 * v0 + (1 - b2) * g * g
    new = p0 - float(np.float32(LR)) * (m / (1 - b1 ** STEP)) / (torch.sqrt(v / (1 - b2 ** STEP)) + 1e-8)
    return {"grad": g, "state": torch.stack([new, m, v]), "stats": torch.tensor([loss, total], dtype=torch.float64)}
