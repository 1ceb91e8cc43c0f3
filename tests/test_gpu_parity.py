"""GPU parity of the HIP path (through the C ABI) against the fp64 oracle.

Every input is seeded and synthetic; every expected value comes from the
oracle on the host.  Integer and index outputs must match bit for bit; logits
within the network's tolerance (1e-3 bf16, 1e-5 fp32, relative to the logit's scale).
"""
import math

import numpy as np
import pytest
import torch

import oracle
import paper_1703_02529_amd as nsc
import synth
from paper_1703_02529_amd.runner import CascadeRunner
from paper_1703_02529_amd.streaming import StreamingCascade
from synth import workloads as W

from helpers import (LOGIT_TOL, LogitErrors, check_properties, check_samples, compare_cascade,
                     lr_weights_for)

pytestmark = pytest.mark.gpu
DEV = "cuda"
rng = np.random.default_rng(20240611)


def _dev(a, dtype=None):
    t = torch.from_numpy(np.ascontiguousarray(a))
    return t.to(DEV) if dtype is None else t.to(DEV, dtype)


def _render(video, t0, n):
    out = torch.empty(max(n, 1) * video.spec.frame_bytes, dtype=torch.uint8, device=DEV)
    video.render_device(out, t0, n)
    return out


# ----------------------------------------------------------------- inputs

@pytest.mark.parametrize("wl", W.ALL, ids=lambda w: w.name.split("-")[0])
def test_device_renderer_matches_host(wl):
    v = synth.Video(wl.video)
    occ = np.flatnonzero(v.occupied)
    t0 = int(occ[0]) if occ.size else 0
    t0 = min(t0, wl.video.n - 3)
    d = _render(v, t0, 3).cpu().numpy().reshape(3, wl.video.h, wl.video.w, 3)
    assert np.array_equal(d, v.frames(t0, t0 + 3))


def test_device_renderer_odd_frame_size():
    # 33 x 17 x 3 = 1683 bytes per frame: frames start off 16-byte boundaries
    spec = synth.VideoSpec(n=600, h=33, w=17, seed=3, obj_min=4, obj_max=12, occupancy=0.6, vmax=3)
    v = synth.Video(spec)
    t0 = int(np.flatnonzero(v.occupied)[0])
    d = _render(v, t0, 7).cpu().numpy().reshape(7, 33, 17, 3)
    assert np.array_equal(d, v.frames(t0, t0 + 7))


# ------------------------------------------------------------- downsample

@pytest.mark.parametrize("H,W,Ho,Wo,pad", [
    (100, 100, 50, 50, 0),      # 4-byte chunks, integer ratio
    (480, 640, 50, 50, 0),      # 16-byte chunks, ratios 9.6 x 12.8
    (480, 640, 50, 50, 48),     # padded frame stride
    (720, 1280, 100, 100, 0),
    (720, 1280, 50, 50, 0),     # 32-byte lane chunks (two 16-byte loads per lane)
    (1080, 1920, 100, 100, 0),  # 16-byte lane chunks, 54 of 64 lanes
    (1080, 1920, 50, 50, 32),   # padded stride, 16-byte chunks
    (33, 17, 5, 4, 0),          # 1-byte chunks, ragged
    (600, 64, 2, 16, 0),        # 300 source rows per output row: unpacked sums
    (64, 64, 64, 64, 0),        # identity
])
def test_downsample_parity(H, W, Ho, Wo, pad):
    n = 7
    fb = H * W * 3
    stride = fb + pad
    host = rng.integers(0, 256, size=(n, stride), dtype=np.uint8)
    dev = _dev(host.reshape(-1))
    out = torch.empty(n * Ho * Wo * 3, dtype=torch.int32, device=DEV)
    nsc.nsc_downsample(dev, n, H, W, Ho, Wo, out, frame_stride=stride)
    got = out.cpu().numpy().reshape(n, Ho, Wo, 3)
    for f in range(n):
        ref = oracle.area_sums(host[f, :fb].reshape(H, W, 3), Ho, Wo)
        assert np.array_equal(got[f], ref), f"frame {f}"


@pytest.mark.parametrize("H,W,Ho,Wo,pad,shift,n", [
    (100, 100, 50, 50, 0, 0, 256),    # whole frames in LDS: 16-byte frames,
    (100, 101, 100, 101, 0, 1, 260),  # ... any alignment, a tail of bytes
    (50, 100, 25, 50, 4, 4, 300),     # ... 4-byte frames
    (100, 100, 50, 50, 0, 0, 3),      # too few for that: general strips, last chunk moved back
    (96, 848, 50, 50, 0, 0, 4),       # three general strips of 16-byte rows
    (96, 848, 50, 100, 12, 4, 4),     # ... of 4-byte rows, padded
    (40, 341, 7, 50, 5, 3, 3),        # ... at any alignment
    (31, 6, 3, 5, 0, 0, 3),           # rows of 18 bytes: two chunks that overlap
    (31, 5, 3, 5, 1, 0, 3),           # rows of 15 bytes: below one chunk
    (700, 340, 2, 17, 0, 0, 3),       # 350 source rows per output row: unpacked general strips
    (20, 1364, 20, 1364, 0, 0, 2),    # identity of a wide 4-byte row
    (12000, 1, 12000, 1, 0, 0, 256),  # a frame that fits LDS, its table of rows does not
])
def test_downsample_general_strips(H, W, Ho, Wo, pad, shift, n):
    """Frames at the end of their allocation, at every alignment, on the forms
    for general widths and small frames."""
    fb = H * W * 3
    stride = fb + pad
    host = rng.integers(0, 256, size=(n - 1) * stride + fb, dtype=np.uint8)
    dev = torch.empty(shift + host.size, dtype=torch.uint8, device=DEV)[shift:]
    dev.copy_(torch.from_numpy(host))
    out = torch.empty(n * Ho * Wo * 3, dtype=torch.int32, device=DEV)
    nsc.nsc_downsample(dev, n, H, W, Ho, Wo, out, frame_stride=stride)
    got = out.cpu().numpy().reshape(n, Ho, Wo, 3)
    for f in sorted({0, 1, n // 2, n - 1}):
        ref = oracle.area_sums(host[f * stride:f * stride + fb].reshape(H, W, 3), Ho, Wo)
        assert np.array_equal(got[f], ref), f"frame {f}"


@pytest.mark.parametrize("H,W,Ho,Wo,pad,shift,below", [
    (96, 848, 50, 50, 0, 0, 199),    # 16-byte rows, bands of 4 rows with 2 left over
    (96, 848, 50, 100, 12, 4, 6),    # 4-byte rows, padded
    (40, 341, 7, 50, 5, 3, 27),      # any alignment
    (31, 6, 3, 5, 0, 0, 1033),       # rows of 18 bytes: two chunks that overlap
    (700, 340, 2, 17, 0, 0, 124),    # periodic 4-byte strips below; unpacked sums
    (20, 1364, 20, 1364, 0, 0, 9),   # identity of a wide 4-byte row
    (100, 100, 50, 50, 0, 0, 9),     # periodic 4-byte strips below, one strip per row
])
def test_downsample_general_strips_from(H, W, Ho, Wo, pad, shift, below):
    """The last call size that leaves the general strips to the forms for few
    output rows, the first that takes them, and twice that."""
    fb = H * W * 3
    stride = fb + pad
    host = rng.integers(0, 256, size=(2 * below + 1) * stride + fb, dtype=np.uint8)
    for n in (below, below + 1, 2 * below + 2):
        end = (n - 1) * stride + fb
        dev = torch.empty(shift + end, dtype=torch.uint8, device=DEV)[shift:]
        dev.copy_(torch.from_numpy(host[:end]))
        out = torch.full((n * Ho * Wo * 3 + 64,), -5, dtype=torch.int32, device=DEV)
        nsc.nsc_downsample(dev, n, H, W, Ho, Wo, out, frame_stride=stride)
        got = out.cpu().numpy()
        assert (got[n * Ho * Wo * 3:] == -5).all()
        got = got[:n * Ho * Wo * 3].reshape(n, Ho, Wo, 3)
        for f in sorted({0, 1, n // 2, n - 1}):
            ref = oracle.area_sums(host[f * stride:f * stride + fb].reshape(H, W, 3), Ho, Wo)
            assert np.array_equal(got[f], ref), f"{n} frames, frame {f}"


def test_downsample_extremes():
    # all-255 frames reach the largest sums; all-0 frames give zeros
    H, W = 720, 1280
    for v in (0, 255):
        dev = torch.full((2 * H * W * 3,), v, dtype=torch.uint8, device=DEV)
        out = torch.empty(2 * 50 * 50 * 3, dtype=torch.int32, device=DEV)
        nsc.nsc_downsample(dev, 2, H, W, 50, 50, out)
        assert (out.cpu().numpy() == v * oracle.area_den(H, W, 50, 50)).all()


# --------------------------------------------------------------- detector

def _diff_case(H, W, Ho, Wo, ref_mode, delta, grid, n, t0, delta_diff):
    frames = rng.integers(0, 256, size=(n + delta, H, W, 3), dtype=np.uint8)
    # make consecutive frames similar so scores straddle the threshold
    for k in range(1, n + delta):
        keep = rng.random((H, W, 1)) < 0.9
        frames[k] = np.where(keep, frames[k - 1], frames[k])
    den = oracle.area_den(H, W, Ho, Wo)
    S = np.stack([oracle.area_sums(f, Ho, Wo) for f in frames])
    lr_w = rng.standard_normal(grid[0] * grid[1]).astype(np.float32)
    ref_img = frames[0]
    kw = dict(in_h=H, in_w=W, dd_h=Ho, dd_w=Wo, cnn_h=Ho, cnn_w=Wo, ref_mode=ref_mode,
              delta=delta, grid=grid, delta_diff=delta_diff, lr_b=-0.5)
    lr_dev = _dev(lr_w)
    ref_dev = _dev(S[0].astype(np.int32).reshape(-1))
    cfg = nsc.make_cfg(lr_w=lr_dev if grid != (1, 1) else None,
                       ref_sums=ref_dev if ref_mode == 1 else None, **kw)
    dframes = _dev(frames[delta:].reshape(-1))
    prev = _dev(S[:delta].astype(np.int32).reshape(-1)) if (ref_mode == 0 and t0 > 0) else None
    sums = torch.empty(n * Ho * Wo * 3, dtype=torch.int32, device=DEV)
    score = torch.empty(n, dtype=torch.float64, device=DEV)
    fire = torch.empty(n, dtype=torch.uint8, device=DEV)
    nsc.nsc_diff_detect(cfg, dframes, n, t0, sums, fire, score_out=score, prev_sums=prev)
    g_s, g_f = score.cpu().numpy(), fire.cpu().numpy()
    assert np.array_equal(sums.cpu().numpy().reshape(n, Ho, Wo, 3), S[delta:])
    for i in range(n):
        t = t0 + i
        cur = S[delta + i]
        ref = S[0] if ref_mode == 1 else S[i]
        if ref_mode == 0 and t < delta:
            exp = math.inf
        elif grid == (1, 1):
            exp = oracle.global_mse(cur, ref, den)[0]
        else:
            exp = oracle.blocked_score(cur, ref, den, grid, lr_w, -0.5)[0]
        assert g_s[i] == exp, (i, g_s[i], exp)
        assert g_f[i] == (1 if (exp > delta_diff or (ref_mode == 0 and t < delta)) else 0)
    return g_f


@pytest.mark.parametrize("case", [
    dict(H=480, W=640, Ho=50, Wo=50, ref_mode=0, delta=15, grid=(1, 1), n=40, t0=100, dd=400.0),
    dict(H=480, W=640, Ho=50, Wo=50, ref_mode=0, delta=3, grid=(1, 1), n=20, t0=0, dd=400.0),
    dict(H=100, W=100, Ho=50, Wo=50, ref_mode=1, delta=1, grid=(1, 1), n=20, t0=5, dd=600.0),
    dict(H=200, W=200, Ho=100, Wo=100, ref_mode=0, delta=1, grid=(10, 10), n=12, t0=9, dd=0.0),
    dict(H=90, W=120, Ho=50, Wo=50, ref_mode=0, delta=2, grid=(3, 4), n=12, t0=0, dd=0.0),
    dict(H=150, W=150, Ho=75, Wo=75, ref_mode=1, delta=1, grid=(1, 1), n=9, t0=0, dd=-math.inf),
])
def test_diff_detect_parity(case):
    c = dict(case)
    dd = c.pop("dd")
    _diff_case(delta_diff=dd, **c)


# ------------------------------------------------------------- compaction

@pytest.mark.parametrize("n", [0, 1, 63, 64, 65, 4095, 4096, 4097, 12345, 100_000, 4_194_305])
@pytest.mark.parametrize("density", [0.0, 0.013, 0.5, 1.0])
def test_compact_parity(n, density):
    fire = (rng.random(n) < density).astype(np.uint8)
    ws = torch.empty(max(nsc.nsc_compact_workspace_bytes(n), 4), dtype=torch.uint8, device=DEV)
    idx = torch.full((max(n, 1),), -7, dtype=torch.int32, device=DEV)
    cnt = torch.full((1,), -1, dtype=torch.int32, device=DEV)
    nsc.nsc_compact(_dev(fire) if n else None, n, idx if n else None, cnt, ws if n else None)
    ref = np.flatnonzero(fire)
    assert int(cnt.item()) == ref.size
    assert np.array_equal(idx.cpu().numpy()[:ref.size], ref)


# -------------------------------------------------------------------- CNN

def _cnn_case(spec, n_frames, n_img, fy=1, seed=5, max_count=None, pairs=False):
    hs, ws_ = spec.in_h * fy, spec.in_w * fy
    den = 9
    S = rng.integers(0, 255 * den + 1, size=(n_frames, hs, ws_, 3)).astype(np.int32)
    idx = np.sort(rng.choice(n_frames, size=n_img, replace=False)).astype(np.int32)
    wts = synth.cnn_weights(spec, seed)
    blob = synth.weight_blob(spec, wts)
    desc = nsc.make_desc(spec.conv, spec.pool, spec.dense, spec.in_h, spec.in_w, spec.bf16, pairs)
    cnn = nsc.Cnn(desc, blob)
    max_count = n_img + 5 if max_count is None else max_count
    ws = torch.empty(nsc.nsc_cnn_workspace_bytes(cnn, max_count), dtype=torch.uint8, device=DEV)
    logit = torch.full((max_count,), math.nan, dtype=torch.float32, device=DEV)
    prob = torch.full((max_count,), math.nan, dtype=torch.float32, device=DEV)
    idx_d = torch.zeros(max_count, dtype=torch.int32, device=DEV)
    idx_d[:n_img] = _dev(idx)
    cnt = torch.tensor([n_img], dtype=torch.int32, device=DEV)
    nsc.nsc_specialized_cnn(cnn, _dev(S.reshape(-1)), hs, ws_, den, idx_d, cnt, max_count, logit,
                            ws, prob_out=prob)
    g = logit.cpu().numpy()
    p = prob.cpu().numpy()
    cnn.close()
    assert np.isnan(g[n_img:]).all(), "entries beyond count must not be written"
    ref = np.zeros(n_img)
    scale = np.zeros(n_img)
    for i, f in enumerate(idx):
        x = S[f].astype(np.int64)
        if fy > 1:
            x = x.reshape(spec.in_h, fy, spec.in_w, fy, 3).sum(axis=(1, 3))
        ref[i], scale[i] = oracle.cnn_logit(spec, blob, x, den * fy * fy, want_scale=True)
    errs = LogitErrors().add(g[:n_img], ref, scale)
    print(f"{spec}: {errs}")
    assert errs.scale <= LOGIT_TOL[spec.bf16], f"max rel err {errs.scale:.3g} ({errs})"
    np.testing.assert_allclose(p[:n_img], 1 / (1 + np.exp(-g[:n_img].astype(np.float64))),
                               rtol=1e-6, atol=1e-7)
    return errs


@pytest.mark.parametrize("wl", [W.TINY, W.VGA], ids=["tiny-fp32", "vga-bf16"])
def test_cnn_parity_small_nets(wl):
    _cnn_case(wl.cnn, n_frames=60, n_img=37)


@pytest.mark.parametrize("wl", [W.HD_REF, W.HD_BLOCKED], ids=["hd4conv", "hd3conv-nested"])
def test_cnn_parity_large_nets(wl):
    fy = wl.dd_h // wl.cnn.in_h
    _cnn_case(wl.cnn, n_frames=30, n_img=17, fy=fy)


def test_cnn_fp32_variants():
    # fp32 inner layers with 4-aligned channels, odd grid, no pooling on the last layer
    spec = synth.CNNSpec(in_h=13, in_w=11, conv=(16, 48), pool=(True, False), dense=16, bf16=False)
    _cnn_case(spec, n_frames=20, n_img=19)
    spec = synth.CNNSpec(in_h=9, in_w=21, conv=(32, 64), pool=(False, True), dense=64, bf16=True)
    _cnn_case(spec, n_frames=20, n_img=3)


def test_cnn_column_segments():
    # layers whose weights plus a full-width band exceed the LDS budget run in
    # column segments (ragged last segment): bf16 64 -> 64 on a 120-wide map,
    # and an fp32 64 -> 64 layer whose weights alone fill most of the LDS
    spec = synth.CNNSpec(in_h=10, in_w=120, conv=(64, 64), pool=(False, True), dense=32, bf16=True)
    _cnn_case(spec, n_frames=12, n_img=5)
    spec = synth.CNNSpec(in_h=12, in_w=40, conv=(16, 64, 64), pool=(False, False, True), dense=16,
                         bf16=False)
    _cnn_case(spec, n_frames=12, n_img=5)


@pytest.mark.parametrize("conv,pool,hw,fy", [
    ((32, 64, 32), (True, False, True), (23, 31), 1),   # fused pair + a layered third layer
    ((64, 16), (True, True), (20, 20), 1),              # 64 then 16 channels
    ((32, 32), (True, True), (50, 50), 2),              # nested 2x2 cells into the first layer
    ((32, 32), (True, False), (13, 9), 1),              # unpooled second layer, tiny odd map
])
def test_cnn_fused_pair_shapes(conv, pool, hw, fy):
    # bf16 nets whose pooled first layer fits in LDS run their first two layers fused
    spec = synth.CNNSpec(in_h=hw[0], in_w=hw[1], conv=conv, pool=pool, dense=32, bf16=True)
    _cnn_case(spec, n_frames=24, n_img=11, fy=fy)


@pytest.mark.parametrize("conv,pool,hw,fy", [
    ((32, 32), (True, True), (50, 50), 2),            # nested cells, pooled, two tile rows per band
    ((32, 16), (False, False), (7, 5), 1),            # maps smaller than a tile row
    ((48, 64), (True, False), (21, 13), 1),           # 48 channels: groups of three; inner fp32 cores
    ((32, 48, 32), (False, True, False), (23, 31), 1),
    ((64, 64), (False, True), (25, 50), 1),           # two channel blocks, two output groups
    ((32, 96, 32), (True, True, False), (18, 22), 1),  # three channel blocks, three output groups
    ((16, 32, 32), (True, True, False), (17, 120), 1),  # wide: several rounds of tiles per band
    ((32, 32), (False, False), (5, 230), 1),          # too wide for the bands: fp32 cores
])
def test_cnn_fp32_split_shapes(conv, pool, hw, fy):
    # fp32 layers as three bf16 parts on the bf16 matrix cores, at the edges of
    # their tiles, bands, channel blocks and output groups
    spec = synth.CNNSpec(in_h=hw[0], in_w=hw[1], conv=conv, pool=pool, dense=32, bf16=False)
    _cnn_case(spec, n_frames=16, n_img=9, fy=fy)
    _cnn_case(spec, n_frames=16, n_img=1, fy=fy, max_count=600)


@pytest.mark.parametrize("conv,pool,hw,bf16", [
    ((16,), (True,), (4, 1200), False),
    ((48, 16), (False, True), (5, 1135), False),
    ((64,), (True,), (6, 1201), False),
    ((16,), (True,), (4, 3500), True),
    ((32,), (False,), (2, 3412), True),
    ((96,), (True,), (5, 3413), True),
])
def test_cnn_first_layer_of_wide_maps(conv, pool, hw, bf16):
    """First layers of which one tile row exceeds the LDS of the kernels for
    usual widths: column segments."""
    spec = synth.CNNSpec(in_h=hw[0], in_w=hw[1], conv=conv, pool=pool, dense=16, bf16=bf16)
    _cnn_case(spec, n_frames=5, n_img=3)
    if bf16:
        _cnn_case(spec, n_frames=5, n_img=2, pairs=True)


@pytest.mark.parametrize("conv,pool,hw,fy", [
    ((64, 64), (True, True), (50, 50), 2),    # pooled 64 channels, nested cells: fp16 into a band
    ((16,), (True,), (7, 5), 1),              # one store lane of four, a last pooled row cut off
    ((32,), (False,), (4, 16), 1),            # one band whose pixels are whole tiles
    ((48,), (True,), (21, 13), 1),            # three blocks, ragged windows
    ((96,), (False,), (9, 18), 1),            # two groups of three blocks
    ((128,), (True,), (18, 3), 1),            # two groups of four, one window per row
    ((16,), (False,), (6, 400), 1),           # rows of several rounds of tiles
])
def test_cnn_first_layer_alone_shapes(conv, pool, hw, fy):
    # a bf16 network's first layer fused with no second one, at the edges of its
    # tiles, bands and output groups; few and many bands per image
    spec = synth.CNNSpec(in_h=hw[0], in_w=hw[1], conv=conv, pool=pool, dense=32, bf16=True)
    _cnn_case(spec, n_frames=16, n_img=9, fy=fy)
    _cnn_case(spec, n_frames=16, n_img=1, fy=fy, max_count=2000)


def _one_layer_logits(w, bias, S, pool=False, out=0, at=(2, 2), cout=16, den=1, bf16=True,
                      pairs=False):
    """Logits of a network of one conv layer whose dense layer passes the value
    of channel `out` at (pooled) pixel `at` through: w [3][3][3] (dy, dx,
    input channel) and bias of that channel; S: area sums [n][h][w][3]."""
    n, h, wd, _ = S.shape
    ho, wo = (h // 2, wd // 2) if pool else (h, wd)
    conv = np.zeros((cout, 3, 3, 3), np.float32)
    conv[out] = np.transpose(np.asarray(w, np.float32), (2, 0, 1))
    cb = np.zeros(cout, np.float32)
    cb[out] = bias
    w1 = np.zeros((16, cout, ho, wo), np.float32)
    w1[3, out, at[0], at[1]] = 1.0
    w2 = np.zeros(16, np.float32)
    w2[3] = 1.0
    blob = np.concatenate([conv.ravel(), cb, w1.ravel(), np.zeros(16, np.float32), w2,
                           np.zeros(1, np.float32)])
    return _net_logits((cout,), (pool,), blob, S, den, bf16, pairs)


def _net_logits(conv, pool, blob, S, den=1, bf16=False, pairs=False):
    n, h, w, _ = S.shape
    cnn = nsc.Cnn(nsc.make_desc(conv, pool, 16, h, w, bf16, pairs), blob)
    ws = torch.empty(nsc.nsc_cnn_workspace_bytes(cnn, n), dtype=torch.uint8, device=DEV)
    logit = torch.full((n,), 77.0, dtype=torch.float32, device=DEV)
    nsc.nsc_specialized_cnn(cnn, _dev(S.astype(np.int32).reshape(-1)), h, w, den,
                            torch.arange(n, dtype=torch.int32, device=DEV),
                            torch.tensor([n], dtype=torch.int32, device=DEV), n, logit, ws)
    got = logit.cpu().numpy()
    cnn.close()
    return got


@pytest.mark.parametrize("pool", [False, True])
@pytest.mark.parametrize("cout", [16, 64, 128])
@pytest.mark.parametrize("pairs", [False, True], ids=["fp16-acts", "bf16-pairs"])
def test_cnn_first_layer_bias_is_added_last(pool, cout, pairs):
    """Two products of 2^20 that cancel across the matrix steps leave the bias
    as it is: its value then only rounds on the way into the dense layer, to 11
    bits (fp16) or 16 (a pair of bf16).  Added to the first product it would
    keep steps of 2^-3."""
    w = np.zeros((3, 3, 3))
    w[0, 0, 0], w[2, 1, 0] = 2.0 ** 20, -2.0 ** 20
    S = np.full((3, 8, 8, 3), 255)
    got = _one_layer_logits(w, 0.1, S, pool=pool, out=cout - 3, cout=cout, pairs=pairs)
    assert np.abs(got / np.float32(0.1) - 1).max() <= (2.0 ** -16 if pairs else 2.0 ** -11), got


@pytest.mark.parametrize("pool", [False, True])
@pytest.mark.parametrize("cout", [16, 32, 48])
def test_cnn_fp32_first_layer_bias(pool, cout):
    """The same in an fp32 network: the bias comes out to the bit."""
    w = np.zeros((3, 3, 3))
    w[0, 0, 0], w[2, 1, 0] = 2.0 ** 20, -2.0 ** 20
    S = np.full((3, 8, 8, 3), 255)
    got = _one_layer_logits(w, 0.1, S, pool=pool, out=cout - 3, cout=cout, bf16=False)
    assert (got == np.float32(0.1)).all(), got


def _operands(r, k, kind):
    if kind == "normal":
        return r.standard_normal(k).astype(np.float32)
    if kind == "positive":
        return r.uniform(0.01, 1, k).astype(np.float32)
    return (1 + r.integers(1, 128, k) / 128 - 2.0 ** -23).astype(np.float32)  # low bits all set


def _check_fp32_sums(got, terms, single):
    """Errors of sums of products (terms [n][k], exact in fp64), relative to
    the sum of their magnitudes: no larger than those of a chain of fp32 fused
    multiply-adds, and of no preferred sign (the mean of n errors of either
    sign stays within four of its standard deviations).  A single product,
    rounded once by the chain, may leave out 2^-24 more of itself."""
    exact, scale = terms.sum(1), np.abs(terms).sum(1)
    chain = np.zeros(len(terms), np.float32)
    for k in range(terms.shape[1]):
        chain = (chain.astype(np.float64) + terms[:, k]).astype(np.float32)
    ok = exact > 1e-3 * scale  # past the ReLU
    e = ((got - exact) / scale)[ok]
    rms = np.sqrt((e ** 2).mean())
    ref = np.sqrt((((chain - exact) / scale)[ok] ** 2).mean())
    print(f"rms {rms:.3e} against {ref:.3e}, mean {e.mean():+.2e}, largest {np.abs(e).max():.2e}")
    assert rms <= (np.hypot(ref, 2.0 ** -25 * np.sqrt(2 / 3)) if single else ref)
    assert abs(e.mean()) <= 4 * rms / np.sqrt(e.size)
    if single:
        assert np.abs(e).max() <= 2.0 ** -23 * (1 + 2.0 ** -7)


DENQ = 8000


def _fine_inputs(r, n, positive):
    S = r.integers(DENQ * 255 // 2 + 1 if positive else 0, DENQ * 255 + 1, size=(n, 6, 6, 3))
    return S, ((2 * S - 255 * DENQ) / (255 * DENQ)).astype(np.float32)


@pytest.mark.parametrize("live", [1, 3, 9, 27])
@pytest.mark.parametrize("kind", ["normal", "positive", "lowbits"])
def test_cnn_fp32_first_layer_sums(kind, live):
    r = np.random.default_rng([live, len(kind)])
    got, terms = [], []
    for _ in range(4):
        S, x = _fine_inputs(r, 4096, kind != "normal")
        w = np.zeros(27, np.float32)
        w[r.choice(27, live, replace=False)] = _operands(r, live, kind)
        got.append(_one_layer_logits(w.reshape(3, 3, 3), 0.0, S, out=5, at=(3, 2), den=DENQ,
                                     bf16=False))
        t = x[:, 2:5, 1:4].reshape(-1, 27).astype(np.float64) * w
        terms.append(t[:, w != 0])
    _check_fp32_sums(np.concatenate(got), np.concatenate(terms), live == 1)


@pytest.mark.parametrize("live", [1, 8, 32, 243])
@pytest.mark.parametrize("kind", ["normal", "positive", "lowbits"])
def test_cnn_fp32_inner_layer_sums(kind, live):
    """The first layer copies each of the 27 neighbouring inputs (positive)
    into a channel of its own, exactly; the second sums `live` products."""
    r = np.random.default_rng([live, len(kind)])
    copy = np.zeros((32, 3, 3, 3), np.float32)
    for c in range(27):
        copy[c, c % 3, c // 9, c // 3 % 3] = 1
    w1 = np.zeros((16, 32, 6, 6), np.float32)
    w1[3, 9, 3, 3] = 1
    out = np.zeros(16, np.float32)
    out[3] = 1
    got, terms = [], []
    for _ in range(4):
        S, x = _fine_inputs(r, 4096, True)
        w = np.zeros((32, 9), np.float32)
        w.reshape(-1)[r.choice(27 * 9, live, replace=False)] = _operands(r, live, kind)
        conv = np.zeros((32, 32, 3, 3), np.float32)
        conv[9] = w.reshape(32, 3, 3)
        blob = np.concatenate([copy.ravel(), np.zeros(32), conv.ravel(), np.zeros(32), w1.ravel(),
                               np.zeros(16), out, np.zeros(1)]).astype(np.float32)
        got.append(_net_logits((32, 32), (False, False), blob, S, den=DENQ))
        xp = np.pad(x, ((0, 0), (1, 1), (1, 1), (0, 0)))
        act = np.stack([xp[:, 2 + c // 9:5 + c // 9, 2 + c // 3 % 3:5 + c // 3 % 3, c % 3]
                        for c in range(27)], 1).astype(np.float64)  # [n][c][3][3] around (3, 3)
        t = act.reshape(len(x), -1) * w[:27].reshape(-1)
        terms.append(t[:, w[:27].reshape(-1) != 0])
    _check_fp32_sums(np.concatenate(got), np.concatenate(terms), live == 1)


@pytest.mark.parametrize("pool", [False, True])
@pytest.mark.parametrize("kind", ["pairs", "f32"])
def test_cnn_first_layer_overflow(kind, pool):
    """Sums that are NaN count as 0 in the ReLU, and an infinite sum stays
    infinite, also where it meets zero parts of an operand."""
    form = dict(bf16=kind == "pairs", pairs=kind == "pairs", pool=pool)
    inf = np.float32(np.inf)
    w = np.zeros((3, 3, 3))
    w[0, 0, 0], w[2, 1, 0] = inf, -inf   # inf - inf, or inf * 0 past the border
    S = np.full((2, 8, 8, 3), 510)
    S[1] = 255                           # the input 0 (den 2)
    got = _one_layer_logits(w, 0.5, S, den=2, **form)
    assert (got == 0).all(), got
    w[0, 0, 0] = np.nan
    got = _one_layer_logits(w, 0.5, S, den=2, **form)
    assert (got == 0).all(), got
    if kind == "f32":
        # one pixel meets the infinite weight with 1, every other one with 0
        w = np.zeros((3, 3, 3))
        w[1, 1, 0] = inf
        S = np.full((3, 8, 8, 3), 255)
        S[0, 4, 4, 0] = 510
        S[1, 4, 4, 0] = 0                # -inf: 0
        got = _one_layer_logits(w, 0.5, S, den=2, out=5, at=(2, 2) if pool else (4, 4), **form)
        assert list(got) == [inf, 0, 0], got
        # finite weights whose sum overflows
        w[1, 1, 0] = w[1, 1, 1] = 3e38
        S[0, 4, 4] = 510
        S[1, 4, 4, 2] = S[2, 4, 4, 0] = 510
        S[1, 4, 4, 0] = 255
        got = _one_layer_logits(w, 0.5, S, den=2, out=5, at=(2, 2) if pool else (4, 4), **form)
        assert list(got) == [inf, 0.5, np.float32(3e38)], got


@pytest.mark.parametrize("w2", [0.5, 0.3], ids=["one-part", "three-parts"])
@pytest.mark.parametrize("pool", [False, True])
def test_cnn_fp32_inner_layer_overflow(pool, w2):
    """An activation that overflows in the first fp32 layer keeps its sums of
    the second one infinite, whatever parts the weight has."""
    S = np.full((2, 8, 8, 3), 255)
    S[0, 4, 4, 0] = 510
    conv0 = np.zeros((32, 3, 3, 3), np.float32)
    conv0[7, 0, 1, 1] = 3e38
    b0 = np.zeros(32, np.float32)
    b0[7] = 3e38
    conv1 = np.zeros((32, 32, 3, 3), np.float32)
    conv1[20, 7, 1, 1] = w2
    o = 4 if pool else 8
    w1 = np.zeros((16, 32, o, o), np.float32)
    w1[3, 20, o // 2, o // 2] = 1.0
    out = np.zeros(16, np.float32)
    out[3] = 1.0
    blob = np.concatenate([conv0.ravel(), b0, conv1.ravel(), np.zeros(32, np.float32), w1.ravel(),
                           np.zeros(16, np.float32), out, np.zeros(1, np.float32)])
    got = _net_logits((32, 32), (False, pool), blob, S, den=2)
    assert got[0] == np.inf
    assert abs(float(got[1]) / (float(np.float32(3e38)) * float(np.float32(w2))) - 1) <= 2.0 ** -23
    # an activation that rounding to bf16 would take to infinity, without the overflow
    blob[32 * 27 + 7] = 3.4e38
    got = _net_logits((32, 32), (False, pool), blob, np.full((2, 8, 8, 3), 255), den=2)
    assert np.abs(got / (float(np.float32(3.4e38)) * float(np.float32(w2))) - 1).max() <= 2.0 ** -23


@pytest.mark.parametrize("conv,pool,hw,fy", [
    ((64, 64), (False, True), (13, 9), 1),                 # fused 64-channel pair, ragged tiles
    ((64, 32, 64), (False, False, True), (23, 31), 1),     # fused pair into 32 channels
    ((64, 64, 64), (False, False, False), (7, 5), 1),      # map smaller than a band
    ((64, 64, 64, 64), (False, True, False, True), (50, 50), 2),  # the 4-layer net, nested cells
    ((32, 64, 64), (True, False, True), (30, 61), 1),      # banded layer after a layered one
    ((64, 64), (False, False), (6, 80), 1),                # pair band over 80 KB: 1 group per CU
    ((32, 64, 64), (True, False, False), (11, 200), 1),    # banded layer 100 wide (160 KB plan)
    ((64, 64), (True, True), (13, 9), 1),                  # pooled 64-channel first layer fused
    ((64, 32, 64), (True, False, True), (23, 31), 1),      # ... into 32 channels, odd map
    ((64, 64, 64), (True, True, True), (50, 50), 2),       # the 3-layer net, nested cells
    ((64, 64), (True, False), (10, 96), 1),                # ... 48-wide second layer
])
@pytest.mark.parametrize("pairs", [False, True], ids=["fp16-acts", "bf16-pairs"])
def test_cnn_banded_shapes(conv, pool, hw, fy, pairs):
    # bf16 layers with 64 input channels run banded, weights streamed in fragment
    # order: on the fp16 matrix cores (fp16 activations between banded layers),
    # or with hi / lo bf16 activation pairs
    spec = synth.CNNSpec(in_h=hw[0], in_w=hw[1], conv=conv, pool=pool, dense=32, bf16=True)
    _cnn_case(spec, n_frames=16, n_img=9, fy=fy, pairs=pairs)


@pytest.mark.parametrize("dense", [16, 32, 64, 128, 256])
@pytest.mark.parametrize("bf16", [True, False], ids=["bf16", "fp32"])
def test_cnn_dense_paths(dense, bf16):
    """The dense layer below 16,384 survivors' capacity (K split over
    workgroups, then a finishing pass) and from it on (row-blocked
    workgroups), at every dense width: a count of 1, 3 or 133 survivors in
    both."""
    spec = synth.CNNSpec(in_h=10, in_w=12, conv=(32, 32), pool=(True, False), dense=dense,
                         bf16=bf16)
    for n_img in (1, 3, 133):
        _cnn_case(spec, n_frames=140, n_img=n_img)
        _cnn_case(spec, n_frames=140, n_img=n_img, max_count=16400)


def test_cnn_zero_count():
    spec = W.VGA.cnn
    desc = nsc.make_desc(spec.conv, spec.pool, spec.dense, 50, 50, True)
    cnn = nsc.Cnn(desc, synth.weight_blob(spec, synth.cnn_weights(spec, 1)))
    ws = torch.empty(nsc.nsc_cnn_workspace_bytes(cnn, 8), dtype=torch.uint8, device=DEV)
    logit = torch.full((8,), 7.0, dtype=torch.float32, device=DEV)
    nsc.nsc_specialized_cnn(cnn, torch.zeros(50 * 50 * 3, dtype=torch.int32, device=DEV), 50, 50,
                            1, torch.zeros(8, dtype=torch.int32, device=DEV),
                            torch.zeros(1, dtype=torch.int32, device=DEV), 8, logit, ws)
    assert (logit.cpu().numpy() == 7.0).all()
    cnn.close()


# ---------------------------------------------------------------- cascade

def _prepare(wl, t0, n, need_ref=False):
    v = synth.Video(wl.video)
    blob = synth.weight_blob(wl.cnn, synth.cnn_weights(wl.cnn, wl.weight_seed))
    lr = lr_weights_for(wl) if wl.grid != (1, 1) else None
    ref_img = v.median_background() if (need_ref or wl.ref_mode == 1) else None
    return v, blob, lr, ref_img


def _gpu_ref_sums(wl, ref_img):
    d = _dev(ref_img.reshape(-1))
    out = torch.empty(wl.dd_h * wl.dd_w * 3, dtype=torch.int32, device=DEV)
    nsc.nsc_downsample(d, 1, wl.video.h, wl.video.w, wl.dd_h, wl.dd_w, out)
    return out


def _run_and_compare(wl, n, chunks=None):
    """Frames [0, n) of the workload's video, optionally fed in chunks."""
    v, blob, lr, ref_img = _prepare(wl, 0, n)
    ref_o = oracle.area_sums(ref_img, wl.dd_h, wl.dd_w) if ref_img is not None else None
    cfg_o, keep = oracle.make_cfg(wl, lr_w=lr, ref_sums=ref_o)
    ref, _ = oracle.cascade(cfg_o, wl.cnn, blob, v.frames(0, n), t0=0)
    lr_d = _dev(lr) if lr is not None else None
    ref_d = _gpu_ref_sums(wl, ref_img) if ref_img is not None else None
    sizes = chunks or [n]
    run = CascadeRunner(wl, blob, max_frames=max(sizes), lr_w=lr_d, ref_sums=ref_d)
    dev_frames = _render(v, 0, n)
    fb = wl.video.frame_bytes
    outs = {k: [] for k in ("score", "fire", "logit", "label", "defer")}
    done = 0
    for s in sizes:
        run.run(dev_frames[done * fb:(done + s) * fb], s, t0=done)
        for k in outs:
            outs[k].append(getattr(run, k)[:s].cpu().numpy().copy())
        done += s
    gpu = {k: np.concatenate(vv) for k, vv in outs.items()}
    run.close()
    return compare_cascade(wl, gpu, ref, t0=0)


def test_cascade_tiny_full_video():
    wl = W.TINY
    rep = _run_and_compare(wl, wl.video.n)
    assert rep["fired"] > 100
    print(rep)
    rep = _run_and_compare(wl, 400, chunks=[100, 1, 99, 200])
    print(rep)


def _first_occupied(wl, lead):
    v = synth.Video(wl.video)
    occ = np.flatnonzero(v.occupied)
    return max(0, int(occ[0]) - lead) if occ.size else 0


def test_cascade_vga_window():
    wl = W.VGA
    rep = _run_and_compare(wl, 30)
    print(rep)
    t0 = _first_occupied(wl, 20)
    rep = _run_and_compare_from_zero_window(wl, t0, 120)
    print(rep)


@pytest.mark.parametrize("frac", [0.0, 0.25, 0.5, 0.9], ids=["start", "q1", "mid", "end"])
def test_cascade_vga_512_windows(frac):
    """Whole windows of 512 consecutive 640x480 frames at four offsets of the
    100k-frame video, every frame compared (the t - 15 label chains included)."""
    wl = W.VGA
    v = synth.Video(wl.video)
    occ = np.flatnonzero(v.occupied)
    t0 = int(occ[np.searchsorted(occ, int(frac * wl.video.n))]) if frac > 0 else 0
    t0 = max(0, min(t0 - 40, wl.video.n - 512))
    rep = _run_and_compare_from_zero_window(wl, t0, 512)
    print(t0, rep)
    assert rep["fired"] > 0


def _run_and_compare_from_zero_window(wl, t0, n):
    """Window [t0, t0+n) of a video whose frames before t0 are dropped: the
    window is treated as its own video (frame indices restart at 0)."""
    spec_v = wl.video
    v = synth.Video(spec_v)
    frames = v.frames(t0, t0 + n)
    blob = synth.weight_blob(wl.cnn, synth.cnn_weights(wl.cnn, wl.weight_seed))
    lr = lr_weights_for(wl) if wl.grid != (1, 1) else None
    ref_img = v.median_background() if wl.ref_mode == 1 else None
    ref_o = oracle.area_sums(ref_img, wl.dd_h, wl.dd_w) if ref_img is not None else None
    cfg_o, keep = oracle.make_cfg(wl, lr_w=lr, ref_sums=ref_o)
    ref, _ = oracle.cascade(cfg_o, wl.cnn, blob, frames, t0=0)
    run = CascadeRunner(wl, blob, max_frames=n, lr_w=_dev(lr) if lr is not None else None,
                        ref_sums=_gpu_ref_sums(wl, ref_img) if ref_img is not None else None)
    dev_frames = _dev(frames.reshape(-1))
    run.run(dev_frames, n, t0=0)
    gpu = {k: getattr(run, k)[:n].cpu().numpy() for k in ("score", "fire", "logit", "label",
                                                          "defer")}
    run.close()
    return compare_cascade(wl, gpu, ref, t0=0)


@pytest.mark.parametrize("wl,lead,n", [(W.HD_REF, 4, 14), (W.HD_BLOCKED, 4, 16),
                                       (W.FHD_STREAM, 2, 40),
                                       (W.FHD_STREAM.with_occupancy(0.01), 2, 40),
                                       (W.FHD_STREAM.with_occupancy(0.5), 2, 40)],
                         ids=["hd-ref", "hd-blocked", "fhd-blocked", "fhd-blocked-occ1",
                              "fhd-blocked-occ50"])
def test_cascade_large_windows(wl, lead, n):
    t0 = _first_occupied(wl, lead)
    rep = _run_and_compare_from_zero_window(wl, t0, n)
    print(rep)


def test_chunked_equals_one_shot_and_oracle():
    wl = W.VGA
    t0 = _first_occupied(wl, 10)
    n = 90
    v = synth.Video(wl.video)
    frames = v.frames(t0, t0 + n)
    blob = synth.weight_blob(wl.cnn, synth.cnn_weights(wl.cnn, wl.weight_seed))
    dev_frames = _dev(frames.reshape(-1))
    fb = wl.video.frame_bytes
    keys = ("score", "fire", "logit", "label", "defer")

    def run_chunks(sizes):
        run = CascadeRunner(wl, blob, max_frames=max(sizes))
        outs = {k: [] for k in keys}
        done = 0
        for s in sizes:
            run.run(dev_frames[done * fb:(done + s) * fb], s, t0=done)
            for k in keys:
                outs[k].append(getattr(run, k)[:s].cpu().numpy().copy())
            done += s
        run.close()
        return {k: np.concatenate(vv) for k, vv in outs.items()}

    one = run_chunks([n])
    for sizes in ([7, 15, 1, 40, 27], [14, 16, 60], [1] * 20 + [70]):
        ch = run_chunks(sizes)
        for k in keys:
            assert np.array_equal(np.nan_to_num(ch[k], nan=-9), np.nan_to_num(one[k], nan=-9)), k
    cfg_o, keep = oracle.make_cfg(wl)
    ref, _ = oracle.cascade(cfg_o, wl.cnn, blob, frames, t0=0)
    print(compare_cascade(wl, one, ref))


def test_threshold_extremes_and_tiny_calls():
    wl = W.TINY.replace(delta=2)
    v = synth.Video(wl.video)
    blob = synth.weight_blob(wl.cnn, synth.cnn_weights(wl.cnn, wl.weight_seed))
    frames = v.frames(300, 340)
    d = _dev(frames.reshape(-1))
    for dd in (-math.inf, math.inf):
        w2 = wl.replace(delta_diff=dd)
        run = CascadeRunner(w2, blob, max_frames=40)
        run.run(d, 40, t0=0)
        fire = run.fire[:40].cpu().numpy()
        run.close()
        if dd < 0:
            assert fire.all()
        else:
            assert list(np.flatnonzero(fire)) == [0, 1]
    # zero frames and a single frame
    run = CascadeRunner(wl, blob, max_frames=4)
    assert run.run(d, 0, t0=0, want_stats=True)["frames"] == 0
    st = run.run(d, 1, t0=0, want_stats=True)
    assert st == dict(frames=1, fired=1, positive=st["positive"], deferred=st["deferred"])
    run.close()


def test_state_required_and_workspace_checks():
    wl = W.TINY
    blob = synth.weight_blob(wl.cnn, synth.cnn_weights(wl.cnn, wl.weight_seed))
    run = CascadeRunner(wl, blob, max_frames=8)
    d = torch.zeros(8 * wl.video.frame_bytes, dtype=torch.uint8, device=DEV)
    small = torch.empty(1024, dtype=torch.uint8, device=DEV)
    with pytest.raises(nsc.NscError) as e:
        nsc.nsc_cascade_run(run.cfg, run.cnn, d, 8, 0, run.state, small, run.label, run.defer)
    assert e.value.status == -4
    with pytest.raises(nsc.NscError) as e:
        nsc.nsc_cascade_run(run.cfg, run.cnn, d, 8, 0, None, run.ws, run.label, run.defer)
    assert e.value.status == -7
    run.close()


# --------------------------------------------------------------- streaming

def test_streamed_chunks_equal_one_shot():
    """Two frame buffers on two streams, ragged last chunk, reference frame
    t - 30 across chunk boundaries: every output equals a one-shot run."""
    wl = W.FHD_STREAM.with_frames(3 * 512 + 77)
    n, fb, chunk = wl.video.n, wl.video.frame_bytes, 512
    v, blob, lr, _ = _prepare(wl, 0, n)
    lr_d = _dev(lr)
    tables = v.device_tables(DEV)
    frames = torch.empty(n * fb, dtype=torch.uint8, device=DEV)
    v.render_device(frames, 0, n, tables)
    one = CascadeRunner(wl, blob, max_frames=n, lr_w=lr_d)
    one.run(frames, n, t0=0)
    keys = ("score", "fire", "logit", "label", "defer")
    ref = {k: getattr(one, k)[:n].cpu().numpy().copy() for k in keys}
    one.close()
    del frames
    out = {k: torch.full((n,), 77, dtype=getattr(one, k).dtype, device=DEV) for k in keys}
    sc = StreamingCascade(wl, blob, chunk, lr_w=lr_d)
    st = sc.run(n, lambda buf, t0, m, s: v.render_device(buf, t0, m, tables, stream=s),
                timing=True, **out)
    sc.close()
    assert st["chunks"] == 4
    g = {k: out[k].cpu().numpy() for k in keys}
    for k in keys:
        assert np.array_equal(np.nan_to_num(g[k], nan=-7), np.nan_to_num(ref[k], nan=-7)), k
    check_properties(wl, g)
    # oracle on frames around the chunk boundaries
    ts = [0, 29, 30, 511, 512, 541, 1024 + 13, n - 1]
    print(check_samples(wl, v, blob, lr, None, g, ts))
    torch.cuda.empty_cache()


# ---------------------------------------------------------- frame skipping

@pytest.mark.parametrize("s,delta,ref_mode", [(3, 3, W.PREV), (4, 8, W.PREV), (5, 1, W.FIXED)])
def test_skipping_tiny_full_video(s, delta, ref_mode):
    wl = W.TINY.replace(check_stride=s, delta=delta, ref_mode=ref_mode)
    rep = _run_and_compare(wl, wl.video.n)
    assert rep["fired"] > 10
    print(rep)
    # chunk boundaries inside skip blocks, a chunk with no checked frame
    rep = _run_and_compare(wl, 400, chunks=[101, 2, 1, 97, 199])
    print(rep)


def test_skipping_vga_window():
    # the benchmark configuration checking every 5th frame (delta 15 = 3 checks back)
    wl = W.VGA.replace(check_stride=5)
    t0 = _first_occupied(wl, 40)
    rep = _run_and_compare_from_zero_window(wl, t0, 160)
    assert rep["fired"] > 0
    print(rep)


def test_skipping_streamed_equals_one_shot():
    wl = W.HD_BLOCKED.with_frames(1300).replace(delta=2, check_stride=2)
    n, fb = wl.video.n, wl.video.frame_bytes
    v, blob, lr, _ = _prepare(wl, 0, n)
    lr_d = _dev(lr)
    tables = v.device_tables(DEV)
    frames = torch.empty(n * fb, dtype=torch.uint8, device=DEV)
    v.render_device(frames, 0, n, tables)
    one = CascadeRunner(wl, blob, max_frames=n, lr_w=lr_d)
    one.run(frames, n, t0=0)
    keys = ("score", "fire", "logit", "label", "defer")
    ref = {k: getattr(one, k)[:n].cpu().numpy().copy() for k in keys}
    one.close()
    del frames
    out = {k: torch.full((n,), 77, dtype=getattr(one, k).dtype, device=DEV) for k in keys}
    sc = StreamingCascade(wl, blob, 301, lr_w=lr_d)   # odd chunks: boundaries inside skip blocks
    sc.run(n, lambda buf, t0, m, st: v.render_device(buf, t0, m, tables, stream=st), **out)
    sc.close()
    g = {k: out[k].cpu().numpy() for k in keys}
    for k in keys:
        assert np.array_equal(np.nan_to_num(g[k], nan=-7), np.nan_to_num(ref[k], nan=-7)), k
    print(check_samples(wl, v, blob, lr, None, g, [0, 1, 2, 301, 302, 603, 1299]))


@pytest.mark.parametrize("H,W", [
    (11, 31),   # 1,023 values: one wave per frame, the last one that does (4-byte loads)
    (17, 20),   # 1,020: one wave, 16-byte loads
    (18, 19),   # 1,026: four waves, 4-byte loads
    (12, 29),   # 1,044: four waves, 16-byte loads, the last wave's batch nearly empty
    (37, 37),   # 4,107: frames at every alignment
])
@pytest.mark.parametrize("metric", [W.MSE, W.SAD, W.NRMSE])
def test_detector_global_forms(H, W, metric):
    """The global score by one wave per frame and by four, on both sides of
    the 1,024 values where the form changes, against the oracle."""
    n, delta = 37, 2
    f = rng.integers(0, 256, size=(n, H, W, 3), dtype=np.uint8)
    f[5:9] = f[3]
    f[20] = f[18] = 0
    cfg = nsc.make_cfg(in_h=H, in_w=W, dd_h=H, dd_w=W, cnn_h=H, cnn_w=W, delta=delta,
                       delta_diff=0.0, metric=metric)
    sums = torch.empty((n, H, W, 3), dtype=torch.int32, device=DEV)
    fire = torch.empty(n, dtype=torch.uint8, device=DEV)
    score = torch.empty(n, dtype=torch.float64, device=DEV)
    nsc.nsc_diff_detect(cfg, _dev(f), n, 0, sums, fire, score_out=score)
    S, g = f.astype(np.int32), score.cpu().numpy()
    assert np.array_equal(sums.cpu().numpy(), S) and np.isinf(g[:delta]).all()
    for i in range(delta, n):
        exp = oracle.global_metric(S[i], S[i - delta], 1, metric)[0]
        assert g[i] == exp, (i, g[i], exp)
    assert np.array_equal(fire.cpu().numpy(), (g > 0).astype(np.uint8))


@pytest.mark.parametrize("H,W,grid", [(18, 21, (18, 21)), (18, 19, (1, 5)), (9, 70, (4, 66))])
def test_detector_blocked_forms_by_call_size(H, W, grid):
    """Blocked scores of small grids in the last call size with four waves per
    frame (2 x 3 H W - 1 frames) and the first with one: the same bits, and the
    oracle's."""
    n, delta = 6 * H * W, 4
    frames = torch.from_numpy(rng.integers(0, 256, size=(n, H, W, 3), dtype=np.uint8)).to(DEV)
    lr = rng.standard_normal(grid[0] * grid[1]).astype(np.float32)
    lr_dev = _dev(lr)
    cfg = nsc.make_cfg(in_h=H, in_w=W, dd_h=H, dd_w=W, cnn_h=H, cnn_w=W, delta=delta, grid=grid,
                       lr_w=lr_dev, lr_b=-0.5, delta_diff=0.0, metric=1)
    got = []
    for m in (n - 1, n):
        sums = torch.empty((m, H, W, 3), dtype=torch.int32, device=DEV)
        fire = torch.empty(m, dtype=torch.uint8, device=DEV)
        score = torch.empty(m, dtype=torch.float64, device=DEV)
        nsc.nsc_diff_detect(cfg, frames, m, 0, sums, fire, score_out=score)
        got.append(score.cpu().numpy())
    assert np.array_equal(got[0], got[1][:-1])
    S = frames.cpu().numpy().astype(np.int32)
    for i in (delta, n // 2, n - 1):
        assert got[1][i] == oracle.blocked_metric(S[i], S[i - delta], 1, grid, lr, -0.5, 1)[0]


@pytest.mark.parametrize("H,W,grid", [
    # blocked frames of more than 1,024 values: one wave per frame in the whole
    # call (from 16,384 frames on), four in the part
    (30, 40, (3, 5)),      # rows of blocks, two slots per lane
    (18, 21, (18, 21)),    # one slot per lane, blocks of one cell, more rows of blocks than waves
    (20, 100, (2, 7)),     # five slots per lane, fewer rows of blocks than waves
    (20, 130, (7, 13)),    # rows of 390 values: the general block walk
    (8, 72, (2, 70)),      # more block columns than lanes
    # one wave per frame in both
    (12, 10, (3, 5)),
    (6, 8, (1, 1)),
    # four in both (the global score's form does not depend on the call)
    (18, 20, (1, 1)),
])
def test_detector_frame_splits(H, W, grid):
    """A call of 16,400 frames gives the scores of the same frames in a call of
    300, bit for bit, and the oracle's at sampled frames."""
    n, delta = 16_400, 3
    frames = torch.from_numpy(rng.integers(0, 256, size=(n, H, W, 3), dtype=np.uint8)).to(DEV)
    lr = rng.standard_normal(grid[0] * grid[1]).astype(np.float32)
    lr_dev = _dev(lr)
    cfg = nsc.make_cfg(in_h=H, in_w=W, dd_h=H, dd_w=W, cnn_h=H, cnn_w=W, delta=delta, grid=grid,
                       lr_w=lr_dev if grid != (1, 1) else None, lr_b=0.25, delta_diff=0.0)
    sums = torch.empty((n, H, W, 3), dtype=torch.int32, device=DEV)
    fire = torch.empty(n, dtype=torch.uint8, device=DEV)
    score = torch.empty(n, dtype=torch.float64, device=DEV)
    nsc.nsc_diff_detect(cfg, frames, n, 0, sums, fire, score_out=score)
    a, b = 16_000, 16_300
    part = torch.empty(b - a, dtype=torch.float64, device=DEV)
    pfire = torch.empty(b - a, dtype=torch.uint8, device=DEV)
    psums = torch.empty((b - a, H, W, 3), dtype=torch.int32, device=DEV)
    nsc.nsc_diff_detect(cfg, frames[a:b], b - a, a, psums, pfire, score_out=part,
                        prev_sums=sums[a - delta:a])
    assert torch.equal(part, score[a:b]) and torch.equal(pfire, fire[a:b])
    S, g = sums.cpu().numpy(), score.cpu().numpy()
    assert np.isinf(g[:delta]).all()
    for i in (3, 77, 9_999, n - 1):
        exp = (oracle.global_mse(S[i], S[i - delta], 1)[0] if grid == (1, 1) else
               oracle.blocked_score(S[i], S[i - delta], 1, grid, lr, 0.25)[0])
        assert g[i] == exp, (i, g[i], exp)
