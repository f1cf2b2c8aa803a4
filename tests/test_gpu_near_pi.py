"""Complex frames whose frequencies lie at the end of the range, next to +-pi, where the half
angle of the closed-form pair's guess is formed from a sine that vanishes."""
import numpy as np
import pytest

from parity_util import compare_omega, oracle_rows

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("L,N", [(2, 8), (4, 16), (6, 32), (7, 24), (8, 24)])
@pytest.mark.parametrize("warm", [False, True])
def test_tones_next_to_pi(bm, L, N, warm):
    """0.2 to 20 mrad on either side of pi, 12 dB.  Three times the 99.9th percentile of the plain
    path's error at these sizes away from pi (5e-6 rad)."""
    import torch
    rng = np.random.default_rng(L)
    H, W = 24, 331
    w = np.pi + np.geomspace(2e-4, 2e-2, H) * np.where(np.arange(H) % 2, 1, -1)
    z = np.exp(1j * (w[:, None] * np.arange(W) + rng.uniform(0, 2 * np.pi, (H, 1))))
    z = (z + 10 ** -0.6 / np.sqrt(2) * (rng.standard_normal((H, W)) + 1j * rng.standard_normal((H, W))))
    z = z.astype(np.complex64)
    g = torch.from_numpy(z).cuda()
    out = torch.empty((H, W), device="cuda")
    prev = torch.from_numpy(np.repeat((w - 2 * np.pi * (w > np.pi))[:, None], W, 1).astype(np.float32)).cuda()
    d = bm.Demodulator(0, max_width=W, max_height=H)
    bm.bosmusic_demodulate(d.h, [bm.FrameSpec(g, L, N, bm.BM_DIR_X, out, None, prev_omega_x=prev if warm else None)])
    torch.cuda.synchronize()
    d.close()
    compare_omega(out.cpu().numpy(), oracle_rows(z, range(H), L, N), f"L{L} N{N} warm {warm}", tol=1.5e-5)
