"""A block frame's maps do not depend on the frames it shares a call with: the tile kernel takes both
directions at once or one after the other by the size of the whole launch, and the results are the
same bits either way."""
import numpy as np
import pytest

import workloads as wl

pytestmark = pytest.mark.gpu


def frame_maps(torch, n, H, W):
    return torch.full((3, n, H, W), -7.0, device="cuda"), torch.full((n, H, W), 255, dtype=torch.uint8, device="cuda")


@pytest.mark.parametrize("L", [3, 6, 8, 9, 13, 15, 17])
@pytest.mark.parametrize("snr", [14.0, 3.0])
def test_block_frame_alone_and_in_a_batch(bm, L, snr):
    """150 x 140: 90 tiles alone (both directions at once) and 720 in the batch (one after the other);
    every other frame with a phase map, so that sizes from 15 x 15 up see launches with and without."""
    import torch
    W, H, n = 150, 140, 8
    both = bm.BM_DIR_X | bm.BM_DIR_Y | bm.BM_BLOCK
    imgs = [torch.from_numpy(wl.random_frame(W, H, seed=10 * L + k, snr_db=snr).astype(np.float32)).cuda()
            for k in range(n)]
    d = bm.Demodulator(0, max_width=W, max_height=H, max_batch_pixels=n * W * H)

    def run(picks, phases):
        m, f = frame_maps(torch, n, H, W)
        specs = [bm.FrameSpec(imgs[k], L, L, both, m[0, k], m[1, k], flags=f[k],
                              phase=m[2, k] if k in phases else None) for k in picks]
        bm.bosmusic_demodulate(d.h, specs)
        torch.cuda.synchronize()
        return m.view(torch.int32), f

    batch, bf = run(range(n), range(0, n, 2))
    bare, _ = run(range(n), ())
    for k in (0, 1, 6):
        one, of = run([k], range(0, n, 2))
        for c, name in enumerate(("omega_x", "omega_y", "phase")):
            a, b = one[c, k], batch[c, k]
            assert torch.equal(a, b), (k, name, int((a != b).sum()))
        assert torch.equal(of[k], bf[k]), k
        assert torch.equal(one[:2, k], bare[:2, k]), (k, "without phase maps")
    d.close()
