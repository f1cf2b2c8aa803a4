"""Large batches as two halves on two streams: the rule for taking them, and batches of every kind
of frame whose second half is planned behind the first in the workspace, against each frame alone."""
import numpy as np
import pytest

import workloads as wl

pytestmark = pytest.mark.gpu

# (W, H, L, N, dtype, dirs, flags, block, phase): transforms of every route that halves may hold
# (powers of two, 7-smooth, convolutions), flagged y passes, block windows of both kernels
KINDS = [
    (1024, 1024, 6, 32, np.float32, "xy", True, False, False),
    (1024, 768, 4, 16, np.float16, "xy", False, False, False),
    (512, 512, 11, 11, np.float32, "xy", True, True, True),
    (1000, 700, 7, 15, np.uint8, "xy", True, False, False),
    (1024, 1024, 8, 24, np.float32, "y", True, False, False),
    (640, 480, 15, 15, np.float32, "xy", True, True, True),
    (263, 1021, 5, 14, np.float32, "xy", True, False, False),
    (641, 479, 6, 20, np.float64, "x", False, False, False),
    (500, 300, 5, 5, np.uint8, "xy", True, True, True),
    (1024, 512, 3, 9, np.complex64, "xy", True, False, False),
    (777, 333, 9, 9, np.float32, "y", True, True, False),
]


def spec_of(bm, torch, data, kind, poison):
    W, H, L, N, _, dirs, flags, block, phase = kind
    new = lambda t=torch.float32: torch.full((H, W), poison, dtype=t, device="cuda")
    code = (bm.BM_DIR_X if "x" in dirs else 0) | (bm.BM_DIR_Y if "y" in dirs else 0) | (bm.BM_BLOCK if block else 0)
    return bm.FrameSpec(data, L, N, code, new() if "x" in dirs else None, new() if "y" in dirs else None,
                        new(torch.uint8) if flags else None, phase=new() if phase else None)


def maps(s):
    return [t for t in (s.omega_x, s.omega_y, s.flags, s.phase) if t is not None]


def bits(t):
    import torch
    return t.view(torch.int32) if t.is_floating_point() else t


def inputs(torch, kinds):
    out = []
    for k, (W, H, _, _, dt, *_) in enumerate(kinds):
        if dt is np.complex64:
            a, b = (wl.random_frame(W, H, seed=900 + k + q, snr_db=8.0) for q in (0, 50))
            img = (a - a.mean() + 1j * (b - b.mean())).astype(np.complex64)
        else:
            img = wl.random_frame(W, H, seed=900 + k, dtype=dt, snr_db=6.0 + k)
        out.append(torch.from_numpy(np.ascontiguousarray(img)).cuda())
    return out


def halves(capfd):
    return "on two streams" in capfd.readouterr().err


def handle(bm, monkeypatch, **kw):
    monkeypatch.setenv("BOSMUSIC_LOG", "1")
    d = bm.Demodulator(0, max_width=1024, max_height=1024, **kw)
    monkeypatch.delenv("BOSMUSIC_LOG")
    return d


@pytest.mark.parametrize("frames,dirs,block,split", [(30, "xy", False, False), (31, "xy", False, True),
                                                      (61, "x", False, False), (62, "x", False, True),
                                                      (62, "xy", True, False)])
def test_rule(bm, monkeypatch, capfd, frames, dirs, block, split):
    """64 M pixel directions of line windows; block windows do not count."""
    import torch
    W = H = 1024
    img = torch.from_numpy(wl.random_frame(W, H, seed=5).astype(np.float32)).cuda()
    d = handle(bm, monkeypatch, max_batch_pixels=frames * W * H)
    kind = (W, H, 3, 3 if block else 8, np.float32, dirs, False, block, False)
    specs = [spec_of(bm, torch, img, kind, -7.0) for _ in range(frames)]
    one = spec_of(bm, torch, img, kind, -7.0)
    bm.bosmusic_demodulate(d.h, [one])
    torch.cuda.synchronize()
    assert not halves(capfd)
    bm.bosmusic_demodulate(d.h, specs)
    torch.cuda.synchronize()
    assert halves(capfd) == split
    for t, s in enumerate(specs):
        for a, b in zip(maps(s), maps(one)):
            assert torch.equal(bits(a), bits(b)), t
    d.close()


@pytest.mark.parametrize("reverse", [False, True])
def test_halves_of_every_kind_of_frame(bm, monkeypatch, capfd, reverse):
    """On a side stream with poisoned outputs, two calls in a row without a wait between them, each
    frame the same bits as alone."""
    import torch
    data = inputs(torch, KINDS)
    order = [k for _ in range(12) for k in range(len(KINDS))]
    if reverse:
        order = order[::-1]
    px = sum(KINDS[k][0] * KINDS[k][1] for k in order)
    d = handle(bm, monkeypatch, max_batch_pixels=px)
    alone = [spec_of(bm, torch, data[k], KINDS[k], 3) for k in range(len(KINDS))]
    for s in alone:
        bm.bosmusic_demodulate(d.h, [s])
    specs = [spec_of(bm, torch, data[k], KINDS[k], 77) for k in order]
    torch.cuda.synchronize()
    assert not halves(capfd)
    side = torch.cuda.Stream()
    with torch.cuda.stream(side):
        for rep in range(2):
            for s in specs:
                for t in maps(s):
                    t.fill_(100 + rep)
            bm.bosmusic_demodulate(d.h, specs, stream=side)
        bm.bosmusic_demodulate(d.h, specs, stream=side)
        snap = [[t.clone() for t in maps(s)] for s in specs]
    side.synchronize()
    assert capfd.readouterr().err.count("on two streams") == 3
    for q, k in enumerate(order):
        for c, (a, b) in enumerate(zip(snap[q], maps(alone[k]))):
            assert torch.equal(bits(a), bits(b)), (q, KINDS[k], c)
    d.close()


def test_surrogate_halves(bm, monkeypatch, capfd):
    import torch
    W = H = 1024
    kinds = [(W, H, 8, 32, np.float32, "xy", True, False, False), (W, H, 5, 20, np.float32, "xy", False, False, False),
             (1000, 700, 6, 24, np.uint8, "xy", True, False, False)]
    data = inputs(torch, kinds)
    order = list(range(3)) * 12
    d = handle(bm, monkeypatch, max_batch_pixels=36 * W * H)
    bm.bosmusic_surrogate_load(d.h, bm.init_params(3))
    bm.bosmusic_surrogate_config(d.h, 0.25, 0)
    alone = [spec_of(bm, torch, data[k], kinds[k], 3) for k in range(3)]
    for s in alone:
        bm.bosmusic_demodulate(d.h, [s], bm.BM_SURROGATE)
    specs = [spec_of(bm, torch, data[k], kinds[k], 77) for k in order]
    torch.cuda.synchronize()
    assert not halves(capfd)
    bm.bosmusic_demodulate(d.h, specs, bm.BM_SURROGATE)
    torch.cuda.synchronize()
    assert halves(capfd)
    for q, k in enumerate(order):
        for a, b in zip(maps(specs[q]), maps(alone[k])):
            assert torch.equal(bits(a), bits(b)), (q, k)
    d.close()
