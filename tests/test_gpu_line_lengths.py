"""Lines whose length has a prime factor above 13: the convolution route of the analytic
step at the edges of its transform lengths, odd and even, in single frames and batches."""
import numpy as np
import pytest

import oracle
import workloads as wl
from parity_util import compare_omega, oracle_rows

pytestmark = pytest.mark.gpu


# five lines: the 5-smooth transforms of either block size (above 2048 samples the wide one)
@pytest.mark.parametrize("n", [17, 34, 253, 257, 493, 514, 1021, 1023, 1027, 1041, 1850, 2047, 2051, 4087, 4094])
@pytest.mark.parametrize("dt", [np.float32, np.uint8])
def test_convolution_lengths_match_oracle(bm, n, dt):
    import torch
    H = 5                                              # an odd number of lines: the last pairs with zeros
    L, N = (4, 12) if n < 100 else (6, 24)
    img, _, _ = wl.erf_fringe(n, H, 0.13, 20.0, 2.0, H / 2.0, 4.0, 20.0, n, dt)
    d = bm.Demodulator(0, max_width=n, max_height=H)
    wx, _ = d.demodulate(torch.from_numpy(img).cuda(), L, N, "x")
    wx = wx.cpu().numpy()
    d.close()
    compare_omega(wx, oracle_rows(img, range(H), L, N), f"n {n}")


# frames of 2^21 padded samples take the power-of-two transforms: 512, 1024, 2048 and 4096,
# at the longest line of each, the first of the next, and an odd number of lines
@pytest.mark.parametrize("n,H", [(17, 4096), (253, 4099), (257, 2048), (511, 2051), (514, 1024), (1021, 1027),
                                 (1027, 512), (2047, 515)])
def test_convolution_of_many_lines_matches_oracle(bm, n, H):
    import torch
    L, N = (4, 12) if n < 100 else (6, 24)
    img, _, _ = wl.erf_fringe(n, H, 0.13, 20.0, 2.0, H / 2.0, 40.0, 20.0, n, np.float32)
    d = bm.Demodulator(0, max_width=n, max_height=H)
    wx, _ = d.demodulate(torch.from_numpy(img).cuda(), L, N, "x")
    rows = [0, 1, 7, H // 2, H - 2, H - 1]
    wx = wx[rows].cpu().numpy()
    d.close()
    compare_omega(wx, oracle_rows(img, rows, L, N), f"n {n}")


def test_mixed_lengths_in_one_batch_equal_single_calls(bm):
    """Every kernel variant of the analytic step in one group of halves."""
    import torch
    sizes = [(1021, 37), (512, 512), (263, 34), (700, 1850), (96, 60), (2051, 17), (1024, 2047), (1536, 253)]
    specs, single = [], []
    for k, (W, H) in enumerate(sizes):
        img = torch.from_numpy(wl.random_frame(W, H, seed=k, snr_db=15.0)).cuda()
        d = bm.Demodulator(0, max_width=W, max_height=H)
        single += [m.cpu().numpy() for m in d.demodulate(img, 5, 16, "xy")]
        d.close()
        specs.append(bm.FrameSpec(img, 5, 16, 3, torch.empty((H, W), device="cuda"), torch.empty((H, W), device="cuda")))
    d = bm.Demodulator(0, max_width=2051, max_height=2047, max_batch_pixels=sum(W * H for W, H in sizes))
    d.demodulate_many(specs)
    got = [m.cpu().numpy() for s in specs for m in (s.omega_x, s.omega_y)]
    d.close()
    for a, b in zip(got, single):
        assert np.array_equal(a, b, equal_nan=True)
