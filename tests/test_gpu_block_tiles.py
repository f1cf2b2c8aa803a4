"""The tiled block-window kernels at the edges of their tiles and dispatch rules: frames of
one window, of one tile, of ragged tiles, one direction or both, few tiles or many, and
windows left to the second kernel.  Oracle or the all-roots option as the reference."""
import numpy as np
import pytest

import oracle
import workloads as wl
from parity_util import compare_omega

pytestmark = pytest.mark.gpu


def run(bm, img, L, dirs="xy", full_roots=False, **kw):
    import torch
    H, W = img.shape
    d = bm.Demodulator(0, max_width=W, max_height=H, full_roots=full_roots)
    out = d.demodulate(torch.from_numpy(np.ascontiguousarray(img)).cuda(), L, L, dirs, block=True, **kw)
    torch.cuda.synchronize()
    d.close()
    return [None if o is None else o.cpu().numpy() for o in out]


@pytest.mark.parametrize("L", [2, 3, 4, 7, 8, 9, 13, 17])
@pytest.mark.parametrize("dw,dh", [(0, 0), (15, 15), (16, 1), (33, 18)])
def test_tile_edges_match_oracle(bm, L, dw, dh):
    """(0, 0): one window; (15, 15): the windows of one tile when centred on it; ragged ones."""
    if L == 2 and dw == 0:
        pytest.skip("a real line of two samples is DC and Nyquist alone: its analytic signal is zero in FP64 and "
                    "rounding residue in FP32, so the oracle has no value to compare with")
    img = wl.random_frame(L + dw, L + dh, seed=L + dw, snr_db=15.0)
    got = run(bm, img, L)
    for a, o, n in zip(got, oracle.demodulate_block(img, L), "xy"):
        compare_omega(a, o, f"L{L} +{dw}x{dh} {n}")


@pytest.mark.parametrize("L", [5, 11, 15])
@pytest.mark.parametrize("dirs", ["x", "y"])
def test_one_direction_is_that_of_both(bm, L, dirs):
    img = wl.random_frame(61, 47, seed=3 * L, snr_db=12.0)
    both, one = run(bm, img, L, flags=True), run(bm, img, L, dirs, flags=True)
    k = "xy".index(dirs)
    compare_omega(one[k], both[k], f"L{L} {dirs}", tol=1e-5)
    assert one[1 - k] is None
    assert np.array_equal(one[2], both[2] & (15 << 4 * k))


@pytest.mark.parametrize("L,W,H", [(3, 400, 352), (7, 400, 352), (9, 96, 70), (9, 1056, 1008), (13, 400, 352),
                                   (15, 1056, 1008)])
def test_pending_windows_agree_with_all_roots(bm, L, W, H):
    """4 dB: windows of every route, with the phase and the flags, under and over 512 and 4096 tiles."""
    img = wl.random_frame(W, H, seed=L, snr_db=4.0)
    a = run(bm, img, L, flags=True, phase=True)
    b = run(bm, img, L, full_roots=True, flags=True, phase=True)
    for u, v, n in zip(a[:2], b[:2], "xy"):
        compare_omega(u, v, f"L{L} {n}")
    assert np.mean(a[2] != b[2]) <= 1e-3 and np.array_equal(a[2] & 0x11, b[2] & 0x11)
    m = np.isfinite(b[3])
    assert np.array_equal(m, np.isfinite(a[3]))
    d = np.abs((a[3][m] - b[3][m] + np.pi) % (2 * np.pi) - np.pi)
    assert np.quantile(d, 0.999) <= 1e-3


@pytest.mark.parametrize("L,frames", [(9, 20), (11, 18)])
def test_blocks_with_many_left_tiles(bm, L, frames):
    """-6 dB: nearly every tile has windows left; each half of the batch holds more than 16 of them
    per block, a single frame four.  The same windows by the same arithmetic, bit for bit."""
    import torch
    W = H = 1024
    img = torch.from_numpy(wl.random_frame(W, H, seed=L, snr_db=-6.0).astype(np.float32)).cuda()
    both = bm.BM_DIR_X | bm.BM_DIR_Y | bm.BM_BLOCK
    dem = bm.Demodulator(0, max_width=W, max_height=H, max_batch_pixels=frames * W * H)
    out = torch.empty((2, frames + 1, H, W), device="cuda")
    fl = torch.empty((frames + 1, H, W), dtype=torch.uint8, device="cuda")
    specs = [bm.FrameSpec(img, L, L, both, out[0, t], out[1, t], flags=fl[t]) for t in range(frames + 1)]
    bm.bosmusic_demodulate(dem.h, specs[:frames])
    bm.bosmusic_demodulate(dem.h, specs[frames:])
    torch.cuda.synchronize()
    dem.close()
    bits = out.view(torch.int32)
    for t in range(frames):
        assert torch.equal(bits[:, t], bits[:, frames]) and torch.equal(fl[t], fl[frames]), t
