"""The single-tone shortcut of the pair certificate (tone_omega in bm_window.h): its
constants against the bound they come from, its claim on polynomials built at the
bound, and the kernels near it against finding every root."""
import os
import re

import numpy as np
import pytest

import workloads as wl
from parity_util import OMEGA_TOL, compare_omega

HEADER = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_1910_11872_amd", "csrc",
                      "bm_window.h")
SIZES = (3, 4, 5, 6, 7, 8, 9, 11, 13, 15, 17)


def constants(L):
    """(s^2 bound, kappa) of the header."""
    text = open(HEADER).read()
    lo, hi = map(float, re.search(r"tone_s2\(int L\) \{ return L == 3 \? ([\d.]+)f : ([\d.]+)f", text).groups())
    body = re.search(r"tone_kappa\(int L\) \{(.*?)\}", text, re.S).group(1)
    kappa = None
    for op, at, value in re.findall(r"L (<=|==) (\d+) \? ([\d.]+)f", body):
        if (L <= int(at)) if op == "<=" else (L == int(at)):
            kappa = float(value)
            break
    if kappa is None:
        kappa = float(re.findall(r": ([\d.]+)f;", body)[-1])
    return (lo if L == 3 else hi), kappa


def real_steering(z, L):
    """Real form of the unit steering vector at complex frequencies z, (len(z), L)."""
    m, s = L // 2, np.arange(L) - (L - 1) / 2
    parts = [np.sqrt(2) * np.cos(z[:, None] * s[:m]), np.sqrt(2) * np.sin(z[:, None] * s[:m])]
    if L & 1:
        parts.insert(1, np.ones((len(z), 1)))
    return np.concatenate(parts, 1) / np.sqrt(L)


@pytest.mark.parametrize("L", SIZES)
def test_bound_holds_on_the_whole_circle(L):
    s2, kappa = constants(L)
    z = np.linspace(-np.pi, np.pi, 8193) - 1j * np.log(kappa)
    A = real_steering(z, L)
    a0 = real_steering(np.zeros(1), L)[0].real
    D = A @ a0
    rest = A - D[:, None] * a0
    rr, ii, ri = (rest.real ** 2).sum(1), (rest.imag ** 2).sum(1), (rest.real * rest.imag).sum(1)
    H = np.sqrt(0.5 * (rr + ii + np.sqrt((rr - ii) ** 2 + 4 * ri ** 2)))
    off = 2 * np.sqrt(s2 * (1 - s2)) * np.abs(D) * H + s2 * (H ** 2 + np.abs(D) ** 2)
    assert np.all(off < 0.98 * np.abs(1 - D ** 2)), np.max(off / np.abs(1 - D ** 2))


@pytest.mark.parametrize("L", SIZES)
def test_one_pair_in_the_annulus_at_the_bound(L):
    """Signal vectors at the bound: the annulus holds one root pair, all others lie outside it."""
    s2, kappa = constants(L)
    rng = np.random.default_rng(L)
    m = L // 2
    for w in rng.uniform(-np.pi, np.pi, 40):
        a = real_steering(np.array([w]), L)[0].real
        d = rng.standard_normal(L)
        d -= (d @ a) * a
        v = np.sqrt(1 - s2) * a + np.sqrt(s2) * d / np.linalg.norm(d)
        vm, vo = v[:m], v[L - m:]
        u = np.concatenate([vm + 1j * vo, v[m:m + 1] * np.sqrt(2) if L & 1 else [], (vm - 1j * vo)[::-1]]) / np.sqrt(2)
        c = np.array([np.sum(u[:L - k] * u[k:].conj()) for k in range(L)])
        poly = np.concatenate([-c[:0:-1].conj(), [L - c[0].real], -c[1:]])
        r = np.abs(np.roots(poly[::-1]))
        assert np.sum((r >= kappa) & (r <= 1 / kappa)) == 2


@pytest.mark.gpu
@pytest.mark.parametrize("L,N,snr", [(3, 6, 2.0), (4, 9, 1.0), (5, 11, 3.0), (7, 14, 2.0), (8, 16, 0.0), (8, 20, 6.0)])
def test_windows_about_the_bound_agree_with_all_roots(bm, L, N, snr):
    """Short windows at low SNR, where some pass the shortcut and some do not."""
    import torch
    img = torch.from_numpy(np.ascontiguousarray(wl.random_frame(523, 31, seed=7 * L + N, snr_db=snr))).cuda()
    maps = []
    for full in (False, True):
        d = bm.Demodulator(0, max_width=1024, max_height=64, full_roots=full)
        maps.append([m.cpu().numpy() for m in d.demodulate(img, L, N, "xy")])
        d.close()
    for a, b, name in zip(*maps, "xy"):
        compare_omega(a, b, f"L{L} N{N} {name}", tol=OMEGA_TOL)
