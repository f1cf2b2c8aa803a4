"""The training kernel at the edges of its grid: one chunk, one chunk per block, a ragged
second walk, and sample buffers that are only 4-byte aligned."""
import numpy as np
import pytest

import oracle
import workloads as wl
from oracle import surrogate as S
from parity_util import OMEGA_TOL, wrap

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("M", [64, 128, 64 * 255, 64 * 256, 64 * 257])
def test_gradient_sizes_and_alignment(bm, M):
    import torch
    rng = np.random.default_rng(M)
    X = rng.standard_normal((M, 32)).astype(np.float32)
    w = rng.uniform(0.4, 1.5, M)
    T = np.stack([np.cos(w), np.sin(w)], 1).astype(np.float32)
    p = S.init_params(3)
    d = bm.Demodulator(0, max_width=64, max_height=64)
    bm.bosmusic_surrogate_load(d.h, p)

    def grad(offset):
        bx = torch.empty(M * 32 + offset, device="cuda")
        bt = torch.empty(M * 2 + offset, device="cuda")
        x, t = bx[offset:].view(M, 32), bt[offset:].view(M, 2)
        x.copy_(torch.from_numpy(X))
        t.copy_(torch.from_numpy(T))
        g, loss = torch.empty(bm.MLP_PARAMS, device="cuda"), torch.empty(1, device="cuda")
        bm.bosmusic_surrogate_grad(d.h, x, t, g, loss)
        return g.cpu().numpy(), loss.item()

    g, loss = grad(0)
    g1, loss1 = grad(1)
    assert np.array_equal(g, g1) and loss == loss1
    d.close()
    cache = S.forward(p, X, quantize=True)
    ref = S.backward(cache, T)
    assert abs(loss - S.loss(cache["Y"], T)) <= 1e-3 * S.loss(cache["Y"], T)
    off = 0
    for k in ("W1", "b1", "W2", "b2", "W3", "b3"):
        n = int(np.prod(S.SHAPES[k]))
        a, b = g[off:off + n].astype(np.float64), ref[k].reshape(-1)
        off += n
        # bfloat16 operands: 2^-9 per factor, as the tolerance of the larger batch
        assert np.linalg.norm(a - b) <= 1e-2 * np.linalg.norm(b), k


@pytest.mark.parametrize("count", [1, 63, 64, 65, 200])
def test_dataset_sizes(bm, count):
    """Blocks of 64 lines: partial ones give the lines of a longer set, which match the oracle."""
    import torch
    d = bm.Demodulator(0, max_width=64, max_height=64)

    def dataset(first, n):
        X, T, w = (torch.full(s, 7.0, device="cuda") for s in ((n + 1, 32), (n + 1, 2), (n + 1,)))
        bm.bosmusic_surrogate_dataset(d.h, first, X[:n], T[:n], w[:n], seed=5)
        for t in (X, T, w):
            assert bool((t[n:] == 7.0).all())               # nothing is written past the end
        return X[:n].cpu().numpy(), T[:n].cpu().numpy(), w[:n].cpu().numpy()

    got, long = dataset(1000, count), dataset(900, 500)
    d.close()
    for a, b in zip(got, long):
        assert np.array_equal(a, b[100:100 + count])
    lines, _ = wl.philox_training_lines(np.arange(1000, 1000 + count), 5)
    win = oracle.analytic_signal(lines)[:, 48:80]
    omega = oracle.demod_windows(win, 8)
    assert np.max(np.abs(got[0] - S.features(win))) < 2e-4
    assert np.mean(np.abs(wrap(got[2].astype(np.float64) - omega)) > OMEGA_TOL) <= 0.01
    assert np.max(np.abs(got[1] - np.stack([np.cos(got[2]), np.sin(got[2])], 1))) < 1e-6
