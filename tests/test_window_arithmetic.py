"""The kernels' per-window arithmetic (bm_window.h), compiled for the host, against FP64."""
import ctypes
import os
import subprocess

import numpy as np
import pytest

import oracle
import workloads as wl

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)
ROCM = os.environ.get("ROCM_PATH", "/opt/rocm")


@pytest.fixture(scope="module")
def host(tmp_path_factory):
    out = str(tmp_path_factory.mktemp("host") / "window_host.so")
    subprocess.run(["g++", "-O2", "-shared", "-fPIC", "-std=c++17", "-w", "-D__HIP_PLATFORM_AMD__",
                    "-I", os.path.join(ROCM, "include"), "-I", os.path.join(ROOT, "include"),
                    "-I", os.path.join(ROOT, "paper_1910_11872_amd", "csrc"),
                    os.path.join(HERE, "window_host.cpp"), "-o", out], check=True, timeout=300)
    return ctypes.CDLL(out)


def ptr(a):
    return a.ctypes.data_as(ctypes.c_void_p)


def f32(a):
    return np.ascontiguousarray(a, np.float32)


def wrap(a):
    return (a + np.pi) % (2 * np.pi) - np.pi


def unitary(L):
    """Q: u1 = Q v."""
    m, o = L // 2, L - L // 2
    Q = np.zeros((L, L), complex)
    for i in range(m):
        Q[i, i] = Q[L - 1 - i, i] = 1 / np.sqrt(2)
        Q[i, o + i], Q[L - 1 - i, o + i] = 1j / np.sqrt(2), -1j / np.sqrt(2)
    if L & 1:
        Q[m, m] = 1
    return Q


def real_form(S):
    """Trace-normalised T of snapshots S (n, L, K), and the lag-1 sums."""
    Q = unitary(S.shape[1])
    R = S @ S.conj().transpose(0, 2, 1)
    T = (Q.conj().T @ (R + R[:, ::-1, ::-1].conj()) @ Q).real
    return T / np.trace(T, axis1=1, axis2=2)[:, None, None], (S[:, :-1].conj() * S[:, 1:]).sum((1, 2))


def line_snapshots(rng, w, L, N, snr):
    """Snapshots of noisy tones of N samples at frequencies w."""
    n = len(w)
    x = np.exp(1j * (w[:, None] * np.arange(N) + rng.uniform(0, 2 * np.pi, (n, 1))))
    x = x + 10 ** (-snr / 20) / np.sqrt(2) * (rng.standard_normal((n, N)) + 1j * rng.standard_normal((n, N)))
    return np.stack([x[:, i:i + N - L + 1] for i in range(L)], 1)


def signal_vectors(rng, w, L, N, snr):
    """FP32 signal vectors (real form) of noisy tones."""
    T, _ = real_form(line_snapshots(rng, w, L, N, snr))
    return f32(np.linalg.eigh(T)[1][:, :, -1])


def root_omega(v, L):
    """omega of each vector's pair nearest the circle, all roots in FP64."""
    out = np.empty(len(v))
    for t, u in enumerate(v.astype(float) @ unitary(L).T):
        u = u / np.linalg.norm(u)
        c = np.array([np.sum(u[:L - k] * u[k:].conj()) for k in range(L)])
        z = np.roots(np.concatenate([-c[:0:-1].conj(), [L - c[0].real], -c[1:]])[::-1])
        i = np.argmin(np.abs(np.abs(z) - 1))
        d = np.abs(z - 1 / z[i].conj())
        d[i] = np.inf
        out[t] = np.angle(z[i] + z[np.argmin(d)])
    return out


@pytest.mark.parametrize("L,N,snr", [(2, 8, 14), (4, 16, 10), (6, 32, 8), (7, 24, 8), (8, 24, 8)])
@pytest.mark.parametrize("lo,hi", [(0.0, 0.006), (0.006, 0.05)])
def test_closed_form_near_pi(host, L, N, snr, lo, hi):
    """Frequencies within lo .. hi of +-pi, the guess a few 1e-3 off the peak in directions that carry
    the hardware's sine and cosine error.  Tolerance: atan2f and the correction (one unit each), their
    sum and the wrap by 2 pi (half a unit each and 1.7e-7) at 2.4e-7 per unit: 9e-7."""
    rng = np.random.default_rng(int(100 * L + 1000 * hi))
    n = 1500
    w = wrap(np.pi - rng.uniform(lo, hi, n) * rng.choice([-1, 1], n))
    v = signal_vectors(rng, w, L, N, snr)
    cw, sw = f32(np.cos(w) + rng.uniform(-5e-7, 5e-7, n)), f32(np.sin(w) + rng.uniform(-5e-7, 5e-7, n))
    omega, ok = np.empty(n, np.float32), np.empty(n, np.uint8)
    assert host.host_tone(L, ptr(v), ptr(cw), ptr(sw), n, ptr(omega), ptr(ok)) == 0
    ok = ok.astype(bool)
    assert ok.mean() > 0.9
    d = np.abs(wrap(omega.astype(float) - root_omega(v, L)))[ok]
    assert d.max() <= 9e-7, (d.max(), np.mean(d > 9e-7))


def plain_power(T, c1, tol=1e-5):
    """The power iteration on T itself (no shift), FP64, from the lag-1 direction: each window's vector
    of the first step (from the second on, of eight) whose angle the residual bound proves below tol."""
    n, L = T.shape[:2]
    s = np.arange(L) - (L - 1) / 2
    a = np.exp(1j * np.angle(c1)[:, None] * s) / np.sqrt(L)
    v = (a @ unitary(L).conj()).real
    t2 = (T ** 2).sum((1, 2))
    done, out = np.zeros(n, bool), np.full((n, L), np.nan)
    for it in range(8):
        y = np.einsum("nij,nj->ni", T, v)
        rho = np.einsum("ni,ni->n", v, y)
        r = np.linalg.norm(y - rho[:, None] * v, axis=1)
        l2 = np.sqrt(np.maximum(t2 - rho ** 2, 0))
        sb = r / np.maximum(rho - l2, 1e-30)
        ok = ~done & (rho > l2) & (sb <= 0.5) & (l2 / rho * sb * np.sqrt(4 / 3) <= tol) & (it >= 1)
        v = y / np.linalg.norm(y, axis=1)[:, None]
        out[ok] = v[ok]
        done |= ok
    return out, done


def angles(v, top):
    s = np.sign(np.einsum("ni,ni->n", v, top))
    return np.linalg.norm(v - top * s[:, None], axis=1)


@pytest.mark.parametrize("L,N,snr", [(4, 32, 8), (6, 32, 8), (8, 48, 8), (6, 6, 11), (8, 8, 11), (9, 9, 10), (11, 11, 10),
                                     (13, 13, 10), (15, 15, 9), (17, 17, 9), (11, 11, 16)])
def test_shifted_power_iteration_is_as_accurate_as_the_plain_one(host, L, N, snr):
    """The shift tightens the bound as well as the convergence: the vectors it accepts are no further
    from the top eigenvector than those of the plain iteration accepted at 1e-5 (or within what FP32
    leaves of any vector, 1.5e-7).  N = L: block windows."""
    rng = np.random.default_rng(17 * L + N)
    n = 3000
    w = rng.uniform(0.3, 1.6, n)
    if N > L:
        S = line_snapshots(rng, w, L, N, snr)
    else:
        y, x = np.mgrid[:L, :L]
        S = np.exp(1j * (rng.uniform(0.02, 0.3, (n, 1, 1)) * y + w[:, None, None] * x))
        S = S + 10 ** (-snr / 20) / np.sqrt(2) * (rng.standard_normal(S.shape) + 1j * rng.standard_normal(S.shape))
        S = S.transpose(0, 2, 1)
    T, c1 = real_form(S)
    T = f32(T)
    top = np.linalg.eigh(T.astype(float))[1][:, :, -1]
    v, steps, ok = np.empty((n, L), np.float32), np.empty(n, np.int32), np.empty(n, np.uint8)
    cr, ci = f32(c1.real), f32(c1.imag)
    assert host.host_power(L, ptr(T), ptr(cr), ptr(ci), n, int(N == L), ptr(v), ptr(steps), ptr(ok)) == 0
    ok = ok.astype(bool)
    ref, done = plain_power(T.astype(float), c1)
    assert ok.mean() >= done.mean() - 0.01
    rms = np.sqrt(np.mean(angles(v, top)[ok] ** 2))
    assert rms <= max(np.sqrt(np.mean(angles(ref, top)[done] ** 2)), 1.5e-7), (rms, steps[ok].mean())


@pytest.mark.parametrize("L,N,snr", [(4, 16, 10), (6, 32, 8), (7, 15, 12), (8, 24, 8)])
@pytest.mark.parametrize("shift", [0.0, 0.1, -2.0])
def test_warm_start_keeps_the_closed_form(host, L, N, snr, shift):
    """A window that the closed form serves takes it whatever the previous frame's frequency was: the
    same omega in the same one step each as without a warm start."""
    rng = np.random.default_rng(L * N)
    n = 2000
    w = rng.uniform(0.3, 1.6, n)
    v = signal_vectors(rng, w, L, N, snr)
    out = []
    for prev in (np.full(n, np.nan), w + shift):
        prev, omega, steps = f32(prev), np.empty(n, np.float32), np.empty((n, 2), np.int32)
        assert host.host_window(L, ptr(v), ptr(prev), n, ptr(omega), ptr(steps)) == 0
        out.append((omega, steps))
    closed = (out[0][1] == 1).all(1)
    assert closed.mean() > 0.99
    assert np.array_equal(out[0][1][closed], out[1][1][closed])
    assert np.array_equal(out[0][0][closed], out[1][0][closed])


@pytest.mark.parametrize("L", [9, 11, 13, 15])
@pytest.mark.parametrize("snr", [10, 16])
def test_closed_form_serves_curved_windows(host, L, snr):
    """Windows over which the frequency bends (the diffusion front of a 64-line frame): the root lies
    up to 1e-3 rad from the spectrum's peak, and the closed form of the tile kernel still serves what
    is within its bound of one tone.  Tolerance: atan2f and the sum (two units of 1.2e-7 below 2 rad) and 1e-8."""
    img, _, _ = wl.erf_fringe(120, 64, 0.11, 35.0, 6.0, 32.0, 9.0, float(snr), 5, np.float32)
    G = oracle.to_complex_field(img, 1)
    S = np.lib.stride_tricks.sliding_window_view(G, (L, L)).reshape(-1, L, L)      # rows as samples: omega_y
    T, _ = real_form(S)
    v = f32(np.linalg.eigh(T)[1][:, :, -1])
    n = len(v)
    u = v.astype(float) @ unitary(L).T
    g = (u[:, 1:] * u[:, :-1].conj()).sum(1)
    cw, sw = f32(g.real / np.abs(g)), f32(g.imag / np.abs(g))
    omega, ok = np.empty(n, np.float32), np.empty(n, np.uint8)
    assert host.host_tone(L, ptr(v), ptr(cw), ptr(sw), n, ptr(omega), ptr(ok)) == 0
    closed = ok.astype(bool)
    omega = np.where(closed, omega, np.angle(g).astype(np.float32))
    s = np.arange(L) - (L - 1) / 2
    a = np.exp(1j * omega.astype(float)[:, None] * s) / np.sqrt(L)
    s2 = 1 - np.abs(np.einsum("ni,ni->n", u.conj(), a)) ** 2
    assert closed[s2 <= 0.06].all(), (np.mean(~closed[s2 <= 0.06]), np.mean(s2 <= 0.06))
    pick = closed & (rng_pick(n, 1500) | (s2 > 0.02))
    d = np.abs(wrap(omega.astype(float)[pick] - root_omega(v[pick], L)))
    assert d.max() <= 2.5e-7


def rng_pick(n, k):
    out = np.zeros(n, bool)
    out[np.random.default_rng(0).permutation(n)[:k]] = True
    return out
