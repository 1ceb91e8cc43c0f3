"""Label resolution, the carried state and the compaction around a call's
survivors, at the sizes where their one-workgroup forms begin, end and take
another chunk: labels of whole videos against the rule applied to the run's
own fire flags and logits (a fired frame's decision, else the compared
frame's)."""
import types

import numpy as np
import pytest
import torch

import paper_1703_02529_amd as nsc
from paper_1703_02529_amd.runner import CascadeRunner, GroupRunner

pytestmark = pytest.mark.gpu
DEV = "cuda"
HW = 8
BLOB_FLOATS = 27 * 32 + 32 + 16 * 32 * 16 + 16 + 16 + 1


def _workload(delta):
    return types.SimpleNamespace(
        video=types.SimpleNamespace(h=HW, w=HW), dd_h=HW, dd_w=HW,
        cnn=types.SimpleNamespace(in_h=HW, in_w=HW, conv=[32], pool=[True], dense=16, bf16=True),
        ref_mode=nsc.NSC_REF_PREV, delta=delta, grid=(1, 1), delta_diff=4.0, c_low=0.45,
        c_high=0.55, lr_bias=0.0)


def _blob(seed):
    return np.random.default_rng(seed).normal(0, 0.3, BLOB_FLOATS).astype(np.float32)


def _frames(n, seed, rate=0.05):
    """A still 8x8 video whose picture changes for one frame in `rate` of the frames."""
    r = np.random.default_rng(seed)
    f = np.repeat(r.integers(0, 256, (1, HW, HW, 3), dtype=np.uint8), n, 0)
    hot = r.random(n) < rate
    f[hot] = r.integers(0, 256, (int(hot.sum()), HW, HW, 3), dtype=np.uint8)
    return torch.from_numpy(f).to(DEV)


def _expect(fire, logit, delta, n):
    p = 1.0 / (1.0 + np.exp(-logit.astype(np.float64)))
    dec = np.where(p < 0.45, 0, np.where(p > 0.55, 1, 2))
    pad = (-n) % delta
    at = np.where(fire == 1, np.arange(n), -1)
    at = np.concatenate([at, np.full(pad, -1)]).reshape(-1, delta)
    last = np.maximum.accumulate(at, axis=0).reshape(-1)[:n]
    assert (last >= 0).all()  # the first delta frames fire
    return dec[last]


@pytest.mark.parametrize("delta,calls", [
    (1, [1, 1, 4095, 65536, 3]),       # single frames, the last one-workgroup call
    (1, [65537, 2]),                   # the first call in tiles
    (3, [2, 1, 65535, 1, 7]),          # calls shorter than delta, a ragged full call
    (30, [30, 29, 31, 16384, 65536]),
    (256, [100, 300, 255, 1025, 256]),
    (250, [65536, 90_000, 10]),
])
def test_labels_and_state_across_calls(delta, calls):
    n = sum(calls)
    frames = _frames(n, delta)
    run = CascadeRunner(_workload(delta), _blob(delta), max(calls))
    got = {k: [] for k in ("label", "defer", "fire", "logit")}
    t = 0
    for m in calls:
        run.run(frames[t:t + m], m, t0=t)
        for k in got:
            got[k].append(getattr(run, k)[:m].cpu().numpy())
        t += m
    run.close()
    got = {k: np.concatenate(v) for k, v in got.items()}
    assert np.array_equal(np.isnan(got["logit"]), got["fire"] == 0)
    want = _expect(got["fire"], got["logit"], delta, n)
    assert 0 < got["fire"].mean() < 0.9
    assert np.array_equal(got["label"], want & 1)
    assert np.array_equal(got["defer"], want >> 1)


@pytest.mark.parametrize("n", [1, 20, 64, 65_700])
def test_group_labels_equal_each_cameras_cascade(n):
    """Calls shorter than some camera's delta, whole ones, and one of several
    chunks per camera."""
    deltas = (1, 30)
    wls = [_workload(d) for d in deltas]
    blobs = [_blob(d) for d in deltas]
    videos = [_frames(2 * n, 100 + d) for d in deltas]
    group = GroupRunner(wls, blobs, n)
    singles = [CascadeRunner(w, b, n) for w, b in zip(wls, blobs)]
    for call in range(2):
        part = [v[call * n:(call + 1) * n] for v in videos]
        group.run(torch.cat(part), n, t0=call * n)
        for c, (r, f) in enumerate(zip(singles, part)):
            r.run(f, n, t0=call * n)
            for k in ("label", "defer", "fire"):
                assert torch.equal(getattr(group, k)[c * n:(c + 1) * n], getattr(r, k)[:n]), (c, k)
    group.close()
    for r in singles:
        r.close()


@pytest.mark.parametrize("n", [16_384, 16_385, 65_535, 65_536, 65_537])
@pytest.mark.parametrize("shift", [0, 5])
def test_compaction_forms(n, shift):
    """The one-workgroup form's rounds and its last size, flags on and off
    their 16-byte alignment."""
    r = np.random.default_rng(n)
    for density in (0.0, 0.03, 1.0):
        fire = (r.random(n) < density).astype(np.uint8) * 7
        dev = torch.zeros(n + shift, dtype=torch.uint8, device=DEV)[shift:]
        dev.copy_(torch.from_numpy(fire))
        ws = torch.empty(nsc.nsc_compact_workspace_bytes(n), dtype=torch.uint8, device=DEV)
        idx = torch.full((n,), -7, dtype=torch.int32, device=DEV)
        cnt = torch.full((1,), -1, dtype=torch.int32, device=DEV)
        nsc.nsc_compact(dev, n, idx, cnt, ws)
        want = np.flatnonzero(fire)
        assert int(cnt.item()) == want.size
        assert np.array_equal(idx.cpu().numpy()[:want.size], want)
        assert (idx.cpu().numpy()[want.size:] == -7).all()


@pytest.mark.parametrize("cams,n", [(20, 1), (40, 2), (3, 50)])
def test_group_tiles_of_many_cameras(cams, n):
    """Tiles of 16 survivors that hold up to 16 cameras' rows, each row with
    its camera's dense layer and thresholds: logits as in the camera's own
    cascade, up to the order of the dense layer's fp32 sums (256 products of
    fp16 values, a few 2^-24 each of their magnitude)."""
    wls = [_workload(1) for _ in range(cams)]
    blobs = [_blob(c) for c in range(cams)]
    videos = [_frames(n, c) for c in range(cams)]
    group = GroupRunner(wls, blobs, n)
    group.run(torch.cat(videos), n, t0=0)
    for c in range(cams):
        r = CascadeRunner(wls[c], blobs[c], n)
        r.run(videos[c], n, t0=0)
        got, want = group.logit[c * n:(c + 1) * n], r.logit[:n]
        assert torch.equal(torch.isnan(got), torch.isnan(want))
        fired = ~torch.isnan(want)
        assert torch.allclose(got[fired], want[fired], rtol=1e-5, atol=1e-5)
        r.close()
    group.close()


def test_group_with_a_network_that_overflows():
    """One camera's fp32 network has infinite first-layer weights: its frames
    and its neighbours' come out as in their own cascades."""
    wls = [_workload(1) for _ in range(3)]
    for w in wls:
        w.cnn.bf16 = False
    blobs = [_blob(c) for c in range(3)]
    blobs[1][[0, 9, 31]] = np.inf, -np.inf, np.nan
    videos = [_frames(40, c, rate=0.5) for c in range(3)]
    group = GroupRunner(wls, blobs, 40)
    group.run(torch.cat(videos), 40, t0=0)
    for c in range(3):
        r = CascadeRunner(wls[c], blobs[c], 40)
        r.run(videos[c], 40, t0=0)
        got, want = group.logit[c * 40:(c + 1) * 40], r.logit[:40]
        fired = r.fire[:40] == 1
        assert fired.sum() > 5 and not torch.isnan(want[fired]).any()
        assert torch.allclose(got[fired], want[fired], rtol=1e-5, atol=1e-5)
        r.close()
    group.close()
