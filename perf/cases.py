"""Performance cases of the cascade filter: the calls a program that filters
fixed-camera video makes, through the package's public entry points.

Kinds of case ("kind"):
  downsample  nsc_downsample of n frames (the reference image, a detector grid)
  detect      nsc_diff_detect of n frames of a stream in progress
  cascade     CascadeRunner.run: one call of a stream (a live second, a clip, a chunk)
  batch       CascadeRunner.stage per chunk, then finish: staged chunks of a long video
  group       GroupRunner.run: the same second of many cameras, a network each
  cnn         nsc_specialized_cnn on the survivors of a detector
  sweep       nsc_threshold_sweep over the logged scores of an evaluation video

Frame sizes, grids, networks, frame offsets and batch shapes are those of the
workloads in synth/workloads.py and bench.py where one applies; 848x480 is the
common 480p webcam mode, whose rows are no whole number of the column pattern.
A "net" is text: conv widths, "p" after a pooled layer, then the dense width,
as "32p-32p-128".  Inputs are made on the GPU from the seed alone.
"""
import math
import types

import numpy as np
import torch

import paper_1703_02529_amd as nsc
from paper_1703_02529_amd.runner import CascadeRunner, GroupRunner

DEV = "cuda"
METRICS = {"mse": 0, "sad": 1, "nrmse": 2, "psnr": 3}


def listed():
    return [
        # the smallest call: a fixed reference image brought to the detector's grid
        dict(name="reference-image", kind="downsample", h=720, w=1280, dd=50, n=1),
        # one second of one live camera, filtered as it arrives: latency
        _cascade("camera-second", 480, 640, 50, "32p-32p-128", "bf16", n=30, delta=15, occ=0.3),
        # a short clip at the network's own scale, fp32 network (the 100x100 workload)
        dict(_cascade("small-clip", 100, 100, 50, "32p-32p-32", "f32", n=1000, delta=1, occ=0.3),
             loop=False),
        # a chunk of a stored 640x480 video (the 100k-frame workload)
        _cascade("vga-chunk", 480, 640, 50, "32p-32p-128", "bf16", n=4095, delta=15, occ=0.2),
        # 720p against a fixed reference image: half of the frames reach the network
        _cascade("hd-reference", 720, 1280, 50, "64-64p-64-64p-128", "bf16", n=1024, delta=0,
                 occ=0.5),
        # the 1080p stream: chunks staged into a batch, blocked detector 30 frames back
        dict(_cascade("fhd-batch", 1080, 1920, 100, "64-64p-64-64p-128", "bf16", n=2040, delta=30,
                      occ=0.1, blocks=10), kind="batch", chunks=4),
        # one second of two dozen cameras per call, each with its own network
        dict(_cascade("cameras", 480, 640, 50, "32p-32p-128", "bf16", n=30, delta=15, occ=0.2),
             kind="group", cams=24),
        # a 480p webcam stream scored with the sum of absolute differences
        dict(name="webcam-480p", kind="detect", h=480, w=848, dd=50, n=600, delta=15, blocks=1,
             metric="sad", occ=0.2),
        # the 4-layer network on the survivors of a batch of a busy video
        dict(name="net-4conv", kind="cnn", net="64-64p-64-64p-128", dtype="bf16", grid=50, nest=1,
             count=4096),
        # the 3-layer network on a finer detector grid, a ragged number of survivors
        dict(name="net-3conv-nested", kind="cnn", net="64p-64p-64p-64", dtype="bf16", grid=50,
             nest=2, count=1501),
        # the fp32 network on the survivors of a stored clip
        dict(name="net-fp32", kind="cnn", net="32p-32p-32", dtype="f32", grid=50, nest=1,
             count=3000),
        # the optimizer's threshold search over an evaluation video
        dict(name="threshold-search", kind="sweep", n=100_000, cands=64, delta=15),
    ]


def _cascade(name, h, w, dd, net, dtype, n, delta, occ, blocks=1):
    """delta = 0: fixed reference image; blocks > 1: blocked detector."""
    return dict(name=name, kind="cascade", h=h, w=w, dd=dd, net=net, dtype=dtype, n=n, delta=delta,
                occ=occ, blocks=blocks, grid=50, stride=1, loop=True)


NETS = ["32p-32p-128", "32p-32p-32", "64-64p-64-64p-128", "64p-64p-64p-64", "32-64p-128",
        "32p-64-64p-64"]


def draw(rng):
    """One more case of the same kinds: log-uniform call sizes, frame sizes on
    and off the 16-byte rows, every detector form, metric and network type."""
    def size(lo, hi):
        return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))

    def frame(dd):
        # a multiple of 16 pixels (16-byte rows), of 4, or any width; with the
        # detector's denominator small enough for its exact integer sums
        while True:
            form = rng.random()
            if form < 0.3:
                h, w = rng.choice([(480, 640), (720, 1280), (1080, 1920), (480, 848), (576, 768),
                                   (288, 352), (240, 320)])
            elif form < 0.7:
                w = 16 * rng.randint(8, 120)
                h = 2 * int(w * rng.uniform(0.5, 0.8) / 2)
            elif form < 0.9:
                w = 4 * rng.randint(30, 340)
                h = int(w * rng.uniform(0.5, 0.8))
            else:
                w, h = rng.randint(101, 341), rng.randint(101, 300)
            if min(h, w) < dd:
                continue
            den = (h // math.gcd(h, dd)) * (w // math.gcd(w, dd))
            if 255 * den * 4 < 2 ** 31 and (255 * den) ** 2 * dd * dd * 3 < 9e18:
                return h, w

    kind = rng.choice(["downsample", "detect", "detect", "cascade", "cascade", "batch", "group",
                       "cnn", "cnn", "cnn", "sweep"])
    if kind == "sweep":
        return dict(kind=kind, n=size(2_000, 100_000), cands=size(8, 64),
                    delta=rng.choice([0, 1, 15, 30]))
    if kind == "cnn":
        net = rng.choice(NETS)
        dtype = rng.choice(["bf16", "bf16", "f32", "pairs"])
        most = 3000 if net.startswith("32p-32p") else {"bf16": 1500, "pairs": 500, "f32": 60}[dtype]
        return dict(kind=kind, net=net, dtype=dtype, grid=rng.choice([50, 50, rng.randint(24, 64)]),
                    nest=rng.choice([1, 1, 2]), count=size(1, most))
    dd = rng.choice([50, 50, 100])
    h, w = frame(dd)
    most = max(2, int(4e9 / (h * w * 3)))
    if kind == "downsample":
        return dict(kind=kind, h=h, w=w, dd=dd, n=size(1, min(most, 4000)))
    delta = rng.choice([0, 1, 15, 30])
    blocks = rng.choice([1, 1, 10])
    n = size(30, min(most, 4000))
    if kind == "detect":
        metric = rng.choice(["mse", "sad", "nrmse"] if blocks > 1 else list(METRICS))
        return dict(kind=kind, h=h, w=w, dd=dd, n=max(n, delta), delta=delta, blocks=blocks,
                    metric=metric, occ=rng.choice([0.05, 0.2, 0.5]))
    net, dtype = rng.choice(NETS[:4]), rng.choice(["bf16", "bf16", "bf16", "f32"])
    if dtype == "f32" or net.startswith("64"):
        n = min(n, 60 if dtype == "f32" and net.startswith("64") else 600)
    occ = rng.choice([0.05, 0.2, 0.4])
    if delta:
        n = max(delta, n // delta * delta)
    if kind == "group":
        cams = max(2, min(size(2, 24), most // max(n, 1)))
        n = min(n, 60)
        if delta:
            n = max(delta, n // delta * delta)
        return dict(_cascade("", h, w, dd, net, "bf16", n, delta, occ, blocks), kind=kind,
                    cams=cams)
    c = _cascade("", h, w, dd, net, dtype, n, delta, occ, blocks)
    if kind == "batch":
        return dict(c, kind=kind, chunks=rng.choice([2, 3, 5]))
    return dict(c, stride=5 if delta in (0, 15, 30) and n % 5 == 0 and rng.random() < 0.25 else 1,
                loop=rng.random() < 0.8)


# ------------------------------------------------------------------ inputs

def _gen(seed):
    g = torch.Generator(device=DEV)
    g.manual_seed(int(seed))
    return g


def _video(h, w, n, occ, seed):
    """n uint8 RGB frames: a smooth fixed background, sensor noise (sigma 5)
    and, in about `occ` of the frames, one to four moving rectangles."""
    g, rng = _gen(seed), np.random.default_rng(seed)
    coarse = torch.rand((1, 3, h // 40 + 2, w // 40 + 2), device=DEV, generator=g) * 128 + 64
    bg = torch.nn.functional.interpolate(coarse, size=(h, w), mode="bilinear", align_corners=True)
    bg = bg[0].permute(1, 2, 0).contiguous().round().to(torch.int16)
    px = h * w * 3
    bank = (torch.randn(px + 65536, device=DEV, generator=g) * 5).round().to(torch.int16)
    offs = rng.integers(0, 65536, n)
    frames = torch.empty((n, h, w, 3), dtype=torch.uint8, device=DEV)
    on, left, objs = False, int(rng.integers(1, max(2, min(40, n // 2)))), []
    for t in range(n):
        if left == 0:
            on = not on
            length = rng.integers(15, 120)
            left = max(1, int(length if on else length * (1 - occ) / occ))
            objs = []
            for _ in range(int(rng.integers(1, 5)) if on else 0):
                oh, ow = (max(2, int(s * rng.uniform(0.1, 0.25))) for s in (h, w))
                objs.append([int(rng.integers(0, h - oh)), int(rng.integers(0, w - ow)), oh, ow,
                             int(rng.integers(-6, 7)), int(rng.integers(-6, 7)),
                             torch.tensor(rng.integers(0, 256, 3), dtype=torch.int16).to(DEV)])
        left -= 1
        img = bg
        if objs:
            img = bg.clone()
            for o in objs:
                img[o[0]:o[0] + o[2], o[1]:o[1] + o[3]] = o[6]
                for k, s in ((0, h), (1, w)):
                    if not 0 <= o[k] + o[4 + k] <= s - o[2 + k]:
                        o[4 + k] = -o[4 + k]
                    o[k] = min(max(o[k] + o[4 + k], 0), s - o[2 + k])
        noisy = img.view(-1) + bank[int(offs[t]):int(offs[t]) + px]
        frames[t].view(-1).copy_(noisy.clamp_(0, 255))
    return frames, bg


def _net(text):
    *conv, dense = text.split("-")
    return [int(c.rstrip("p")) for c in conv], [c.endswith("p") for c in conv], int(dense)


def _flat(case):
    conv, pool, _ = _net(case["net"])
    s = case["grid"]
    for p in pool:
        s = s // 2 if p else s
    return conv[-1] * s * s, s


def _blob(case, seed):
    """He-normal weights and small biases in nsc_cnn_create's order, an output
    layer that spreads the logits over a few units."""
    conv, _, dense = _net(case["net"])
    rng = np.random.default_rng([seed, 7])
    parts, cin = [], 3
    for c in conv:
        parts += [rng.normal(0, math.sqrt(2 / (9 * cin)), c * cin * 9), rng.normal(0, 0.05, c)]
        cin = c
    flat, _ = _flat(case)
    parts += [rng.standard_normal(dense * flat, dtype=np.float32) * np.float32(math.sqrt(2 / flat)),
              rng.normal(0, 0.05, dense),
              rng.normal(0, 4 / math.sqrt(dense), dense), rng.normal(0, 0.05, 1)]
    return np.concatenate([p.astype(np.float32) for p in parts])


def _threshold(case):
    """Firing thresholds well above the sensor noise of the area averages."""
    if case["blocks"] > 1:
        return 0.0  # the logistic score's own bias is the threshold
    return {"mse": 15.0, "sad": 29_000.0 * (case["dd"] / 50) ** 2, "nrmse": 0.0303,
            "psnr": -36.37}[case.get("metric", "mse")]


def _lr(case, seed):
    """Weights of the blocked detector: about the mean of the block metrics,
    above a bias that the noise does not reach."""
    if case["blocks"] == 1:
        return None, 0.0
    k = case["blocks"] ** 2
    lr = torch.rand(k, device=DEV, generator=_gen(seed + 3)) / k + 0.5 / k
    return lr, {"mse": -4.0, "sad": -200.0, "nrmse": -0.03}[case.get("metric", "mse")]


def _area_sums(frames, dd):
    """Exact area sums [n, dd, dd, 3] (int64) of uint8 frames, in torch."""
    n, h, w, _ = frames.shape

    def weights(n_in):
        g = math.gcd(n_in, dd)
        p, q = n_in // g, dd // g
        o, i = np.arange(dd)[:, None], np.arange(n_in)[None, :]
        lap = np.minimum((o + 1) * p, (i + 1) * q) - np.maximum(o * p, i * q)
        return torch.tensor(np.maximum(lap, 0), dtype=torch.float64, device=DEV)

    wy, wx = weights(h), weights(w)
    out = []
    for part in frames.split(max(1, int(1e8 / (h * w)))):
        rows = torch.matmul(wy, part.reshape(len(part), h, w * 3).double())
        rows = rows.view(len(part), dd, w, 3).permute(0, 1, 3, 2)
        out.append(torch.matmul(rows, wx.t().contiguous()).permute(0, 1, 3, 2).round().long())
    return torch.cat(out)


def _workload(case):
    conv, pool, dense = _net(case["net"])
    g = case["grid"]
    return types.SimpleNamespace(
        video=types.SimpleNamespace(h=case["h"], w=case["w"]), dd_h=case["dd"], dd_w=case["dd"],
        cnn=types.SimpleNamespace(in_h=g, in_w=g, conv=conv, pool=pool, dense=dense,
                                  bf16=case["dtype"] != "f32"),
        ref_mode=nsc.NSC_REF_PREV if case["delta"] else nsc.NSC_REF_FIXED,
        delta=max(1, case["delta"]), grid=(case["blocks"], case["blocks"]),
        delta_diff=_threshold(case), c_low=0.2, c_high=0.8, lr_bias=_lr(case, 0)[1],
        check_stride=case["stride"])


def prepare(case, seed):
    return globals()["_prepare_" + case["kind"]](case, seed)


def _prepare_downsample(case, seed):
    frames, _ = _video(case["h"], case["w"], case["n"], 0.2, seed)
    sums = torch.empty((case["n"], case["dd"], case["dd"], 3), dtype=torch.int32, device=DEV)
    return dict(case=case, frames=frames, sums=sums)


def _prepare_detect(case, seed):
    n, dd, delta = case["n"], case["dd"], case["delta"]
    frames, bg = _video(case["h"], case["w"], n, case["occ"], seed)
    lr, bias = _lr(case, seed)
    ref = _area_sums(bg[None].to(torch.uint8), dd)[0].int() if not delta else None
    cfg = nsc.make_cfg(in_h=case["h"], in_w=case["w"], dd_h=dd, dd_w=dd, cnn_h=dd, cnn_w=dd,
                       ref_mode=nsc.NSC_REF_PREV if delta else nsc.NSC_REF_FIXED,
                       delta=max(1, delta), grid=(case["blocks"],) * 2, lr_w=lr, lr_b=bias,
                       ref_sums=ref, delta_diff=_threshold(case), metric=METRICS[case["metric"]])
    # the stream repeats: the frames before this call are the call's last ones
    prev = _area_sums(frames[n - delta:], dd).int() if delta else None
    return dict(case=case, frames=frames, cfg=cfg, lr=lr, ref=ref, prev=prev, t0=n,
                sums=torch.empty((n, dd, dd, 3), dtype=torch.int32, device=DEV),
                score=torch.empty(n, dtype=torch.float64, device=DEV),
                fire=torch.empty(n, dtype=torch.uint8, device=DEV))


def _prepare_cascade(case, seed):
    n = case["n"]
    frames, bg = _video(case["h"], case["w"], n, case["occ"], seed)
    lr, _ = _lr(case, seed)
    ref = None if case["delta"] else _area_sums(bg[None].to(torch.uint8), case["dd"])[0].int()
    batch = case["kind"] == "batch"
    runner = CascadeRunner(_workload(case), _blob(case, seed), n, lr_w=lr, ref_sums=ref,
                           device=DEV, batch=batch)
    s = dict(case=case, frames=frames, runner=runner, t0=0)
    if batch:
        cut = [n * k // case["chunks"] for k in range(case["chunks"] + 1)]
        s["parts"] = [(a, b - a, frames[a:b]) for a, b in zip(cut, cut[1:])]
    if case["loop"]:  # a stream in progress that repeats these frames
        run(s)
        s["t0"] = n
    return s


_prepare_batch = _prepare_cascade


def _prepare_group(case, seed):
    cams, n = case["cams"], case["n"]
    videos = [_video(case["h"], case["w"], n, case["occ"], seed + 1000 * c) for c in range(cams)]
    frames = torch.cat([v[0] for v in videos])
    refs = [None if case["delta"] else _area_sums(v[1][None].to(torch.uint8), case["dd"])[0].int()
            for v in videos]
    lrs = [_lr(case, seed + 1000 * c)[0] for c in range(cams)]
    runner = GroupRunner([_workload(case)] * cams,
                         [_blob(case, seed + 1000 * c) for c in range(cams)], n, lr_ws=lrs,
                         ref_sums=refs, device=DEV)
    s = dict(case=case, frames=frames, runner=runner, t0=0)
    run(s)
    s["t0"] = n
    return s


def _cnn_den(case):
    return 100  # a denominator of a 500 x 500 crop on the 50 x 50 grid


def _prepare_cnn(case, seed):
    count, hw = case["count"], case["grid"] * case["nest"]
    g = _gen(seed)
    n = count + count // 3 + 1  # survivors are some of the frames
    coarse = torch.rand((n, 3, 6, 6), device=DEV, generator=g) * 160 + 48
    img = torch.nn.functional.interpolate(coarse, size=(hw, hw), mode="bilinear")
    img = img + torch.randn(img.shape, device=DEV, generator=g) * 2
    den = _cnn_den(case)
    sums = (img.permute(0, 2, 3, 1) * den).round().clamp(0, 255 * den).int().contiguous()
    idx = torch.randperm(n, device=DEV, generator=g)[:count].sort().values.int()
    conv, pool, dense = _net(case["net"])
    desc = nsc.make_desc(conv, pool, dense, case["grid"], case["grid"], case["dtype"] != "f32",
                         pairs=case["dtype"] == "pairs")
    cnn = nsc.Cnn(desc, _blob(case, seed))
    ws = torch.empty(nsc.nsc_cnn_workspace_bytes(cnn, count), dtype=torch.uint8, device=DEV)
    return dict(case=case, cnn=cnn, sums=sums, hw=hw, den=den, idx=idx, ws=ws,
                count=torch.tensor([count], dtype=torch.int32, device=DEV),
                logit=torch.empty(count, device=DEV), prob=torch.empty(count, device=DEV))


def _prepare_sweep(case, seed):
    n, k, rng = case["n"], case["cands"], np.random.default_rng([seed, 3])
    truth = np.zeros(n, np.uint8)
    t = int(rng.integers(0, 300))
    while t < n:  # object episodes of 30 to 300 frames, a fifth of the video
        end = t + int(rng.integers(30, 300))
        truth[t:end] = 1
        t = end + int(rng.integers(120, 1200))
    score = np.where(truth == 1, rng.lognormal(3.2, 1.0, n), rng.lognormal(0.5, 0.8, n))
    score[:case["delta"]] = np.inf
    conf = (1 / (1 + np.exp(-rng.normal(np.where(truth == 1, 2.0, -2.0), 2.0)))).astype(np.float32)
    # thresholds from the noise up to the clearest objects
    deltas = np.exp(np.linspace(math.log(0.5), math.log(100.0), k))
    cfg = nsc.SweepCfg(ref_mode=nsc.NSC_REF_PREV if case["delta"] else nsc.NSC_REF_FIXED,
                       delta=max(1, case["delta"]), fp_target=0.01, fn_target=0.01, t_mse=1.7e-7,
                       t_snn=7.3e-8, t_full=0.0125)
    dev = {key: torch.from_numpy(v).to(DEV)
           for key, v in dict(score=score, conf=conf, truth=truth, deltas=deltas).items()}
    rows = torch.zeros(k * nsc.SWEEP_ROW_BYTES, dtype=torch.uint8, device=DEV)
    best = torch.zeros(1, dtype=torch.int32, device=DEV)
    words = nsc.SWEEP_ROW_BYTES // 8
    out = dict(rates=rows.view(torch.float64).view(k, words)[:, :6],
               counts=rows.view(torch.int64).view(k, words)[:, 6:14],
               feasible=rows.view(torch.int32).view(k, 2 * words)[:, 28], best=best)
    return dict(dev, case=case, cfg=cfg, rows=rows, best=best, out=out)


# --------------------------------------------------------------------- run

def run(s):
    case = s["case"]
    kind, n = case["kind"], case.get("n")
    if kind == "downsample":
        nsc.nsc_downsample(s["frames"], n, case["h"], case["w"], case["dd"], case["dd"], s["sums"])
        return s["sums"]
    if kind == "detect":
        nsc.nsc_diff_detect(s["cfg"], s["frames"], n, s["t0"], s["sums"], s["fire"], s["score"],
                            s["prev"])
        return dict(sums=s["sums"], fire=s["fire"], score=s["score"])
    if kind == "cnn":
        nsc.nsc_specialized_cnn(s["cnn"], s["sums"], s["hw"], s["hw"], s["den"], s["idx"],
                                s["count"], case["count"], s["logit"], s["ws"], s["prob"])
        return dict(logit=s["logit"], prob=s["prob"])
    if kind == "sweep":
        nsc.nsc_threshold_sweep(s["cfg"], s["score"], s["conf"], s["truth"], s["deltas"],
                                s["rows"], s["best"])
        return s["out"]
    r = s["runner"]
    if kind == "batch":
        for at, m, part in s["parts"]:
            r.stage(part, m, at)
        r.finish(n, t0=s["t0"])
    else:
        r.run(s["frames"], n, t0=s["t0"])
    return dict(label=r.label, defer=r.defer, score=r.score, fire=r.fire, logit=r.logit)


# -------------------------------------------------------------------- work

def _net_flops(case):
    conv, pool, dense = _net(case["net"])
    s, cin, f = case["grid"], 3, 0
    for c, p in zip(conv, pool):
        f += 2 * 9 * cin * c * s * s
        cin, s = c, s // 2 if p else s
    return f + 2 * _flat(case)[0] * dense


def _weight_bytes(case):
    conv, _, dense = _net(case["net"])
    k = sum(9 * a * b for a, b in zip([3] + conv, conv)) + _flat(case)[0] * dense
    return k * (4 if case["dtype"] == "f32" else 2)


def work(case):
    kind = case["kind"]
    if kind == "sweep":  # the log read once; per candidate a compare and two counts per frame
        return dict(bytes=13 * case["n"] + 128 * case["cands"],
                    flops=4.0 * case["n"] * case["cands"])
    if kind == "cnn":
        c = case["count"]
        return dict(bytes=c * (case["grid"] * case["nest"]) ** 2 * 12 + _weight_bytes(case),
                    flops=float(c) * _net_flops(case))
    n, px = case["n"] * case.get("cams", 1), case["h"] * case["w"] * 3
    raw = n * px
    cells = case["dd"] ** 2 * 3
    if kind == "downsample":
        return dict(bytes=raw + n * cells * 4, flops=2.0 * raw)
    if kind == "detect":  # the sums are an output; the frames before the call are read as sums
        return dict(bytes=raw + n * cells * 4 + case["delta"] * cells * 4,
                    flops=2.0 * raw + 3.0 * n * cells)
    raw //= case["stride"]
    fired = case["occ"] * n / case["stride"]
    return dict(bytes=raw + 15 * n + _weight_bytes(case) * case.get("cams", 1),
                flops=2.0 * raw + fired * _net_flops(case))


def tolerance(case):
    """Integer sums, scores, flags and counts are the same in every correct
    implementation.  Logits: an fp32 network's sums in another order; a bf16
    network's fp16 activations (2^-12 each, some tens of thousands of terms
    that partly cancel); "pairs" activations carry 2^-17.  A decision may fall
    on the other side of c_low or c_high when a logit lies on the threshold."""
    if case["kind"] in ("downsample", "sweep"):
        return "exact"
    if case["kind"] == "detect":
        return dict(rel=1e-12) if case["metric"] == "psnr" else "exact"
    rel = {"f32": 1e-5, "pairs": 1e-4, "bf16": 2e-3}[case["dtype"]]
    return dict(rel=rel, max=20 * rel, differ=0.004)


# ------------------------------------------------------------------- exact

def _bf16(x):
    """fp64 values rounded to bf16 (nearest, ties to even), as fp64."""
    u = x.contiguous().view(torch.int64)
    u = (u + 0x0FFFFFFFFFFF + ((u >> 45) & 1)) & ~0x1FFFFFFFFFFF
    return u.view(torch.float64)


def _logits(case, sums, den, blob):
    """The network in fp64 on area sums [n, g * nest, g * nest, 3]."""
    conv, pool, dense = _net(case["net"])
    g = case["grid"]
    f = sums.shape[1] // g
    narrow = case["dtype"] != "f32"
    w = torch.from_numpy(blob).to(DEV)
    weights, at, cin = [], 0, 3
    flat, _ = _flat(case)
    for rows, cols in [(c, 9 * k) for k, c in zip([3] + conv, conv)] + [(dense, flat)]:
        m = w[at:at + rows * cols].view(rows, cols)
        weights.append(((m.bfloat16() if narrow else m).double(),
                        w[at + rows * cols:at + rows * cols + rows].double()))
        at += rows * (cols + 1)
    out = []
    for s in sums.split(32) if len(sums) else ():
        s = s.view(len(s), g, f, g, f, 3).sum((2, 4))
        x = (2 * s - 255 * den * f * f).double() / float(255 * den * f * f)
        x = (_bf16(x) if narrow else x).permute(0, 3, 1, 2)
        for (m, b), p in zip(weights, pool):
            y = torch.matmul(m, torch.nn.functional.unfold(x, 3, padding=1))
            x = torch.relu(y + b[:, None]).view(len(s), len(b), x.shape[2], x.shape[3])
            x = torch.nn.functional.max_pool2d(x, 2) if p else x
        m, b = weights[-1]
        hidden = torch.relu(torch.matmul(x.reshape(len(s), -1), m.t().contiguous()) + b)
        out.append(hidden @ w[at:at + dense].double() + w[at + dense].double())
    return torch.cat(out) if out else torch.zeros(0, dtype=torch.float64, device=DEV)


def _scores(case, sums, ref, lr, lr_b):
    """Detector scores of sums against ref (both int64 [n, dd, dd, 3])."""
    dd, k = case["dd"], case["blocks"]
    den = float((case["h"] // math.gcd(case["h"], dd)) * (case["w"] // math.gcd(case["w"], dd)))
    cut = [dd * i // k for i in range(k + 1)]
    z = torch.full((len(sums),), lr_b, dtype=torch.float64, device=DEV)
    for by in range(k):
        for bx in range(k):
            a, b = (v[:, cut[by]:cut[by + 1], cut[bx]:cut[bx + 1]].flatten(1) for v in (sums, ref))
            d, metric = a - b, case.get("metric", "mse")
            e = (d * d).sum(1).double()
            if metric == "sad":
                m = d.abs().sum(1).double() / den
            elif metric == "nrmse":
                m = torch.sqrt(e / (b * b).sum(1).double())
            else:
                m = e / (den * den * d.shape[1])
                m = -10.0 * torch.log10(65025.0 / m) if metric == "psnr" else m
            z = m if k == 1 else z + lr[by * k + bx].double() * m
    return z


def _stream(case, frames, bg, seed):
    """Scores and logits of one stream's call, in fp64."""
    delta, st = case["delta"], case["stride"]
    sums = _area_sums(frames[::st], case["dd"])
    d = delta // st
    if delta:
        ref = torch.roll(sums, d, 0)  # the stream repeats
    else:
        ref = _area_sums(bg[None].to(torch.uint8), case["dd"]).expand_as(sums)
    lr, lr_b = _lr(case, seed)
    score = _scores(case, sums, ref, lr, lr_b)
    if delta and not case["loop"]:
        score[:d] = math.inf
    hit = torch.nonzero(score > _threshold(case)).view(-1)
    dd = case["dd"]
    den = (case["h"] // math.gcd(case["h"], dd)) * (case["w"] // math.gcd(case["w"], dd))
    logit = torch.full((case["n"],), math.nan, dtype=torch.float64, device=DEV)
    logit[hit * st] = _logits(case, sums[hit], den, _blob(case, seed))
    full = torch.full((case["n"],), math.nan, dtype=torch.float64, device=DEV)
    full[::st] = score
    return full, logit


def exact(case, seed):
    kind = case["kind"]
    if kind == "sweep":
        return _exact_sweep(case, seed)
    if kind == "cnn":
        s = _prepare_cnn(case, seed)
        z = _logits(case, s["sums"][s["idx"].long()].long(), s["den"], _blob(case, seed))
        return dict(logit=z, prob=torch.sigmoid(z))
    if kind == "downsample":
        return _area_sums(_video(case["h"], case["w"], case["n"], 0.2, seed)[0], case["dd"])
    if kind == "detect":
        frames, bg = _video(case["h"], case["w"], case["n"], case["occ"], seed)
        sums = _area_sums(frames, case["dd"])
        ref = torch.roll(sums, case["delta"], 0) if case["delta"] else \
            _area_sums(bg[None].to(torch.uint8), case["dd"]).expand_as(sums)
        return dict(sums=sums, fire=None, score=_scores(case, sums, ref, *_lr(case, seed)))
    outs = []
    for c in range(case.get("cams", 1)):
        frames, bg = _video(case["h"], case["w"], case["n"], case["occ"], seed + 1000 * c)
        outs.append(_stream(case, frames, bg, seed + 1000 * c))
    return dict(label=None, defer=None, fire=None, score=torch.cat([o[0] for o in outs]),
                logit=torch.cat([o[1] for o in outs]))


def _exact_sweep(case, seed):
    s = _prepare_sweep(case, seed)
    score, conf, truth, deltas = (s[k].cpu().numpy() for k in ("score", "conf", "truth", "deltas"))
    n, cfg = len(score), s["cfg"]
    ref = np.zeros(n, np.uint8)
    if case["delta"]:
        ref[case["delta"]:] = truth[:-case["delta"]]
    pos = int(truth.sum())
    fn_budget = cfg.fn_target * pos if pos else math.inf
    fp_budget = cfg.fp_target * (n - pos) if n > pos else math.inf
    rates = []
    for d in deltas:
        fired = np.isinf(score) | (score > d)
        fn = int((~fired & (truth == 1) & (ref == 0)).sum())
        fp = int((~fired & (truth == 0) & (ref == 1)).sum())
        lo, hi = 0.0, 1.0
        if fn < fn_budget and fp < fp_budget:
            ones, zeros = np.sort(conf[fired & (truth == 1)]), np.sort(conf[fired & (truth == 0)])
            need = fn_budget - fn
            k = len(ones) + 1 if math.isinf(need) else max(1, math.ceil(need))
            lo = float(ones[k - 1]) if k <= len(ones) else 1.0
            need = fp_budget - fp
            k = len(zeros) + 1 if math.isinf(need) else max(1, math.ceil(need))
            hi = max(lo, float(zeros[-k]) if k <= len(zeros) else 0.0)
        c = conf[fired].astype(np.float64)
        f_m = fired.mean()
        f_c = float(((c >= lo) & (c <= hi)).mean()) if len(c) else 0.0
        rates.append([d, lo, hi, f_m, f_c, cfg.t_mse + f_m * cfg.t_snn + f_m * f_c * cfg.t_full])
    return dict(rates=np.array(rates), counts=None, feasible=None, best=None)
