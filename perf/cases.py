"""Performance cases of the library: what a program asks of it, through its public entry points.

A case names a kind of call and its sizes:

  frame      one recorded frame, demodulated by ``Demodulator.demodulate`` (or, with the temporal
             warm start, by ``bosmusic_demodulate``): the smallest calls, where launches and
             latency count, up to one camera frame
  stack      a series of equal frames in one ``bosmusic_demodulate`` call
  uneven     frames of mixed sizes and covariance sizes in one call of a handle with BM_OPT_GRAPH
  surrogate  a series of frames in BM_SURROGATE mode with a trained network
  block      frames with the paper's own L x L block window (and its phase)
  integrate  a series of frequency maps integrated by one ``bosmusic_integrate_many`` call
  train      minibatch Adam steps of the surrogate network (forward, backward and update)
  dataset    generation of labelled training windows

Sizes are those of the repository's workloads (``workloads/``): the 256 x 256 single frame, the
100 x 1024 x 1024 series, the uneven batch, the 4096 x 4096 series, the surrogate, and the
1850 x 700 8-bit camera series of the experiment.  Frames are synthetic fringes
0.5 + 0.4 cos(carrier + erf diffusion phase) + noise, made on the GPU from the seed.
"""
import math

import torch

import paper_1910_11872_amd as bm

A_DC, B_AC = 0.5, 0.4
DTYPES = {"u8": (torch.uint8, 1), "f16": (torch.float16, 2), "f32": (torch.float32, 4), "f64": (torch.float64, 8),
          "c32": (torch.complex64, 8)}
UNEVEN_SIZES = ((512, 512), (768, 512), (768, 768), (1024, 768), (1024, 1024), (1536, 1024), (1536, 1536),
                (2048, 1536))
UNEVEN_L = (4, 6, 8)
MAX_PIXELS = 16 * 4096 * 4096       # of the largest listed series
EXACT_WINDOWS = 10_000_000          # windows that the 64-bit evaluation below does in a few seconds


def listed():
    return [
        # the smallest real call: one small FP64 frame, one direction; launches and host work count
        {"name": "frame_256_f64_x", "kind": "frame", "width": 256, "height": 256, "dtype": "f64", "L": 4, "N": 16,
         "dirs": "x", "flags": False, "warm": False, "snr": 20.0, "f0": 0.125, "angle": 0.0},
        # one frame of the 8-bit camera as it arrives, with the per-pixel flags a live display masks by
        {"name": "frame_1850x700_u8", "kind": "frame", "width": 1850, "height": 700, "dtype": "u8", "L": 7, "N": 15,
         "dirs": "xy", "flags": True, "warm": False, "snr": 12.0, "f0": 0.11, "angle": 35.0},
        # complex frames (the analytic signal given directly) of an odd size, each warm-started
        # from the maps of the frame before, with the longest window
        {"name": "frame_1531x1023_c32_warm", "kind": "frame", "width": 1531, "height": 1023, "dtype": "c32", "L": 8,
         "N": 64, "dirs": "xy", "flags": False, "warm": True, "snr": 15.0, "f0": 0.125, "angle": 40.0},
        # the time-lapsed FP32 series, processed after the recording
        {"name": "stack_100x1024_f32", "kind": "stack", "width": 1024, "height": 1024, "frames": 100, "dtype": "f32",
         "L": 6, "N": 32, "dirs": "xy", "snr": 10.0, "f0": 0.1, "angle": 30.0},
        # frames of many regions of interest with their own sizes and windows, the same batch again
        # and again (a captured graph is replayed)
        {"name": "uneven_64_graph", "kind": "uneven", "frames": 64, "first": 0, "dtype": "f32"},
        # the large FP16 series: the headline workload
        {"name": "series_16x4096_f16", "kind": "stack", "width": 4096, "height": 4096, "frames": 16, "dtype": "f16",
         "L": 8, "N": 32, "dirs": "xy", "snr": 10.0, "f0": 0.125, "angle": 45.0},
        # the same frames through the learned surrogate
        {"name": "surrogate_4x4096_f16", "kind": "surrogate", "width": 4096, "height": 4096, "frames": 4,
         "dtype": "f16", "L": 8, "N": 32, "dirs": "xy", "snr": 10.0, "f0": 0.125, "angle": 45.0},
        # the paper's simulation window, 11 x 11, on a series
        {"name": "block11_20x1024_f32", "kind": "block", "width": 1024, "height": 1024, "frames": 20, "dtype": "f32",
         "L": 11, "dirs": "xy", "phase": False, "snr": 10.0, "f0": 0.1, "angle": 30.0},
        # the paper's experimental window, 15 x 15, with the block phase, on one camera frame
        {"name": "block15_1850x700_u8", "kind": "block", "width": 1850, "height": 700, "frames": 1, "dtype": "u8",
         "L": 15, "dirs": "xy", "phase": True, "snr": 12.0, "f0": 0.11, "angle": 35.0},
        # frequency maps of the large series to phase, FP64
        {"name": "integrate_16x4096", "kind": "integrate", "width": 4096, "height": 4096, "frames": 16, "N": 32,
         "carrier": True, "both": True},
        # one stretch of the network's training at its production batch, losses and weights read back
        {"name": "train_16384x32", "kind": "train", "batch": 16384, "steps": 32, "rows": 262144, "lr": 2e-4},
        # labelled training windows, one generation chunk
        {"name": "dataset_262144", "kind": "dataset", "rows": 262144, "first": 0},
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def _size(rng, lo=64, hi=2048):
    """A side length over the whole range: powers of two and their multiples, even and odd ones."""
    n = _log(rng, lo, hi)
    how = rng.randrange(3)
    return n if how == 0 else n | 1 if how == 1 else max(lo, n // 64 * 64)


def _fringe(rng, dtypes):
    return {"dtype": rng.choice(dtypes), "snr": round(rng.uniform(10.0, 20.0), 2),
            "f0": round(rng.uniform(1.0 / 12.0, 1.0 / 6.0), 5), "angle": round(rng.uniform(30.0, 60.0), 2)}


def draw(rng):
    kind = rng.choice(("frame", "frame", "stack", "stack", "uneven", "surrogate", "block", "block", "integrate",
                       "train", "dataset"))
    if kind == "frame":
        L = rng.randint(2, 8)
        warm = rng.random() < 0.25
        return {"kind": kind, "width": _size(rng), "height": _size(rng), **_fringe(rng, tuple(DTYPES)), "L": L,
                "N": rng.randint(2 * L, 64), "dirs": "xy" if warm else rng.choice(("x", "y", "xy", "xy")),
                "flags": not warm and rng.random() < 0.3, "warm": warm}
    if kind in ("stack", "surrogate"):
        w, h = _size(rng, 128, 4096), _size(rng, 128, 4096)
        L = rng.randint(4, 8)
        most = max(2, min(100, MAX_PIXELS // 4 // (w * h)))
        return {"kind": kind, "width": w, "height": h, "frames": min(most, _log(rng, 2, 100)),
                **_fringe(rng, ("u8", "f16", "f32")), "L": L, "N": rng.randint(max(16, 2 * L), 48), "dirs": "xy"}
    if kind == "uneven":
        return {"kind": kind, "frames": rng.randint(3, 64), "first": rng.randrange(1000),
                "dtype": rng.choice(("f16", "f32"))}
    if kind == "block":
        L = rng.choice((3, 4, 5, 6, 7, 8, 9, 11, 13, 15, 17))
        w, h = _size(rng, 64, 1024), _size(rng, 64, 1024)
        most = max(1, min(20, 4_000_000 // (w * h)))
        return {"kind": kind, "width": w, "height": h, "frames": min(most, _log(rng, 1, 20)),
                **_fringe(rng, ("u8", "f16", "f32")), "L": L, "dirs": "xy", "phase": rng.random() < 0.5}
    if kind == "integrate":
        w, h = _size(rng, 64, 8192), _size(rng, 64, 4096)
        most = max(1, min(100, MAX_PIXELS // (w * h)))
        return {"kind": kind, "width": w, "height": h, "frames": min(most, _log(rng, 1, 100)),
                "N": rng.randint(4, 48), "carrier": rng.random() < 0.5, "both": rng.random() < 0.8}
    if kind == "train":
        batch = 64 * _log(rng, 1, 512)
        return {"kind": kind, "batch": batch, "steps": _log(rng, 4, 64), "rows": batch * rng.randint(1, 8), "lr": 2e-4}
    return {"kind": kind, "rows": _log(rng, 256, 262144), "first": rng.randrange(1 << 24)}


# ----------------------------------------------------------------------------
# Inputs
# ----------------------------------------------------------------------------
def _generator(seed, k=0):
    return torch.Generator(device="cuda").manual_seed((int(seed) * 1000003 + k) % (1 << 62))


def _carrier(case):
    th = math.radians(case["angle"])
    return 2.0 * math.pi * case["f0"] * math.cos(th), 2.0 * math.pi * case["f0"] * math.sin(th)


def _frame(W, H, wx, wy, w_t, snr, dtype, gen):
    """One fringe frame: carrier (wx, wy), diffusion phase 6 erf((y - H/2) / w_t), noise at `snr` dB."""
    y = torch.arange(H, dtype=torch.float64, device="cuda")[:, None]
    x = torch.arange(W, dtype=torch.float64, device="cuda")[None, :]
    phase = wx * x + (wy * y + 6.0 * torch.erf((y - H / 2.0) / w_t))
    if dtype == "c32":
        s = math.sqrt(10.0 ** (-snr / 10.0) / 2.0)
        noise = torch.randn((H, W, 2), dtype=torch.float32, device="cuda", generator=gen) * s
        return (torch.polar(torch.ones_like(phase), phase) + torch.view_as_complex(noise)).to(torch.complex64)
    s = math.sqrt(B_AC * B_AC / 2.0 * 10.0 ** (-snr / 10.0))
    img = A_DC + B_AC * torch.cos(phase)
    img += torch.randn((H, W), dtype=torch.float32, device="cuda", generator=gen) * s
    if dtype == "u8":
        return torch.round(img * 255.0).clamp_(0, 255).to(torch.uint8)
    return img.to(DTYPES[dtype][0])


def _stack(case, seed):
    """The frames of a series: the diffusion front widens from frame to frame."""
    W, H, n = case["width"], case["height"], case.get("frames", 1)
    wx, wy = _carrier(case)
    out = torch.empty((n, H, W), dtype=DTYPES[case["dtype"]][0], device="cuda")
    for t in range(n):
        w_t = H / 64.0 * 16.0 ** (t / max(1, n - 1)) + 8.0
        out[t] = _frame(W, H, wx, wy, w_t, case["snr"], case["dtype"], _generator(seed, t))
    return out


def _uneven_shape(case, k):
    i = case["first"] + k
    return (*UNEVEN_SIZES[i % len(UNEVEN_SIZES)], UNEVEN_L[i % len(UNEVEN_L)])


def _uneven(case, seed):
    frames = []
    for k in range(case["frames"]):
        W, H, L = _uneven_shape(case, k)
        gen = _generator(seed, k)
        u = torch.rand(4, dtype=torch.float64, device="cuda", generator=gen).tolist()
        f0, ang = 1 / 12 + u[0] / 12, math.radians(30.0 + 30.0 * u[1])
        wx, wy = 2 * math.pi * f0 * math.cos(ang), 2 * math.pi * f0 * math.sin(ang)
        frames.append((_frame(W, H, wx, wy, 16.0 + 112.0 * u[2], 8.0 + 12.0 * u[3], case["dtype"], gen), L))
    return frames


def _maps(case, seed):
    """Frequency maps as the demodulation gives them: the carrier, a smooth part and noise, NaN borders."""
    W, H, n, N = case["width"], case["height"], case["frames"], case["N"]
    out = []
    for k, d in enumerate("xy" if case["both"] else "x"):
        gen = _generator(seed, k)
        m = torch.randn((n, H, W), dtype=torch.float32, device="cuda", generator=gen).mul_(0.01).add_(0.5 + 0.1 * k)
        m += 0.2 * torch.sin(torch.arange(H, device="cuda", dtype=torch.float32) / 97.0)[None, :, None]
        lo = N // 2
        if d == "x":
            m[:, :, :lo] = math.nan
            m[:, :, max(0, W - N + lo + 1):] = math.nan
        else:
            m[:, :lo] = math.nan
            m[:, max(0, H - N + lo + 1):] = math.nan
        out.append(m)
    return out


def _windows(rows, seed):
    """Features [Re(16), Im(16)] of noisy tones and their targets (cos w, sin w), as the training set has them."""
    gen = _generator(seed)
    u = torch.rand((rows, 2), dtype=torch.float64, device="cuda", generator=gen)
    w = 2 * math.pi / 16 + u[:, :1] * (2 * math.pi / 4 - 2 * math.pi / 16)
    s = torch.sqrt(0.5 * 10.0 ** (-3.0 * u[:, 1:]))
    n = torch.randn((rows, 16, 2), dtype=torch.float64, device="cuda", generator=gen)
    m = torch.arange(-8, 8, dtype=torch.float64, device="cuda")
    z = torch.polar(torch.ones((), dtype=torch.float64, device="cuda"), w * m) + s * torch.view_as_complex(n)
    z = z * torch.conj(z[:, 8:9]) / z[:, 8:9].abs() / z.abs().square().mean(1, keepdim=True).sqrt()
    X = torch.cat((z.real, z.imag), 1).float().contiguous()
    return X, torch.cat((torch.cos(w), torch.sin(w)), 1).float().contiguous()


def _weights(seed):
    """Starting weights of the 32-64-64-2 network: W ~ N(0, 1/fan_in), b ~ N(0, 0.01), flat FP32 on the host."""
    gen = torch.Generator().manual_seed(int(seed))
    parts = []
    for fan_in, n in ((32, 32 * 64), (0, 64), (64, 64 * 64), (0, 64), (64, 64 * 2), (0, 2)):
        z = torch.randn(n, dtype=torch.float64, generator=gen)
        parts.append((z / math.sqrt(fan_in) if fan_in else 0.1 * z).float())
    return torch.cat(parts).numpy()


# ----------------------------------------------------------------------------
# The measured calls
# ----------------------------------------------------------------------------
def _dirs(case):
    return (bm.BM_DIR_X if "x" in case["dirs"] else 0) | (bm.BM_DIR_Y if "y" in case["dirs"] else 0)


def prepare(case, seed):
    kind = case["kind"]
    s = {"case": case}
    if kind == "frame":
        s["dem"] = bm.Demodulator(0, max_width=case["width"], max_height=case["height"])
        s["frame"] = _stack(case, seed)[0]
        if case["warm"]:
            # the maps of the frame before: the same scene, other noise
            before = _stack(case, seed + 7919)[0]
            px, py = s["dem"].demodulate(before, case["L"], case["N"], case["dirs"])
            wx, wy = torch.empty_like(px), torch.empty_like(py)
            s["specs"] = [bm.FrameSpec(s["frame"], case["L"], case["N"], _dirs(case), wx, wy, prev_omega_x=px,
                                       prev_omega_y=py)]
            s["out"] = [wx, wy]
    elif kind in ("stack", "surrogate", "block"):
        W, H, n = case["width"], case["height"], case["frames"]
        s["dem"] = bm.Demodulator(0, max_width=W, max_height=H, max_batch_pixels=n * W * H)
        if kind == "surrogate":
            X, T = _windows(65536, 20)
            bm.bosmusic_surrogate_load(s["dem"].h, _weights(21))
            bm.bosmusic_surrogate_train(s["dem"].h, X, T, 4096, 400, 2e-3, want_losses=False)
        data = _stack(case, seed)
        maps = torch.empty((3 if case.get("phase") else 2, n, H, W), dtype=torch.float32, device="cuda")
        L, dirs = case["L"], _dirs(case) | (bm.BM_BLOCK if kind == "block" else 0)
        s["specs"] = [bm.FrameSpec(data[t], L, case.get("N", L), dirs, maps[0, t], maps[1, t],
                                   phase=maps[2, t] if case.get("phase") else None) for t in range(n)]
        s["out"] = list(maps)
    elif kind == "uneven":
        frames = _uneven(case, seed)
        px = sum(f.numel() for f, _ in frames)
        s["dem"] = bm.Demodulator(0, max_width=max(f.shape[1] for f, _ in frames),
                                  max_height=max(f.shape[0] for f, _ in frames), graph=True, max_batch_pixels=px)
        flat = torch.empty((2, px), dtype=torch.float32, device="cuda")   # the maps of all frames, one after another
        s["specs"], at = [], 0
        for f, L in frames:
            m = flat[:, at:at + f.numel()]
            s["specs"].append(bm.FrameSpec(f, L, 2 * L + 8, bm.BM_DIR_X | bm.BM_DIR_Y, m[0].view(f.shape),
                                           m[1].view(f.shape)))
            at += f.numel()
        s["out"] = list(flat)
    elif kind == "integrate":
        W, H, n, N = case["width"], case["height"], case["frames"], case["N"]
        s["dem"] = bm.Demodulator(0, max_width=W, max_height=H)
        maps = _maps(case, seed)
        phi = torch.empty((n, H, W), dtype=torch.float64, device="cuda")
        cx, cy = (0.5, 0.6) if case["carrier"] else (0.0, 0.0)
        s["jobs"] = [(maps[0][t], maps[1][t] if case["both"] else None, N, N, cx, cy, phi[t]) for t in range(n)]
        s["out"] = phi
    elif kind == "train":
        s["dem"] = bm.Demodulator(0, max_width=64, max_height=64)
        s["X"], s["T"] = _windows(case["rows"], seed)
        bm.bosmusic_surrogate_load(s["dem"].h, _weights(seed))
    else:
        s["dem"] = bm.Demodulator(0, max_width=64, max_height=64)
        n = case["rows"]
        s["X"], s["T"], s["w"] = (torch.empty(shape, device="cuda") for shape in ((n, 32), (n, 2), (n,)))
        s["seed"] = int(seed)
    return s


def run(state):
    case, dem = state["case"], state["dem"]
    kind = case["kind"]
    if kind == "frame" and not case["warm"]:
        return list(dem.demodulate(state["frame"], case["L"], case["N"], case["dirs"], flags=case["flags"]))
    if kind in ("frame", "stack", "uneven", "block"):
        bm.bosmusic_demodulate(dem.h, state["specs"])
        return state["out"]
    if kind == "surrogate":
        bm.bosmusic_demodulate(dem.h, state["specs"], bm.BM_SURROGATE)
        return state["out"]
    if kind == "integrate":
        bm.bosmusic_integrate_many(dem.h, state["jobs"])
        return state["out"]
    if kind == "train":
        losses = bm.bosmusic_surrogate_train(dem.h, state["X"], state["T"], case["batch"], case["steps"], case["lr"])
        return [losses, bm.bosmusic_surrogate_save(dem.h)]
    bm.bosmusic_surrogate_dataset(dem.h, case["first"], state["X"], state["T"], state["w"], seed=state["seed"])
    return [state["X"], state["T"], state["w"]]


# ----------------------------------------------------------------------------
# The work of one pass: each input read once, each output written once, and the
# arithmetic of the method with its sums shared (lag sums slid from window to
# window, one eigenvector by three products with the L x L matrix, the
# polynomial's L lags of the eigenvector, two evaluations of it at a root).
# ----------------------------------------------------------------------------
def _window_flops(L):
    return 16 * L + 6 * L * L + 4 * L * L + 64 * L


def _frame_work(W, H, esize, L, ndir, extra):
    px = W * H
    fft = 5.0 * (W * H) * (math.log2(W) + math.log2(H)) / 2
    return px * (esize + 4 * ndir + extra), ndir * (px * _window_flops(L) + fft)


def work(case):
    kind = case["kind"]
    if kind == "frame":
        extra = (1 if case["flags"] else 0) + (4 * len(case["dirs"]) if case["warm"] else 0)
        b, f = _frame_work(case["width"], case["height"], DTYPES[case["dtype"]][1], case["L"], len(case["dirs"]), extra)
    elif kind in ("stack", "surrogate", "block"):
        b, f = _frame_work(case["width"], case["height"], DTYPES[case["dtype"]][1], case["L"], len(case["dirs"]),
                           4 if case.get("phase") else 0)
        b, f = b * case["frames"], f * case["frames"]
    elif kind == "uneven":
        b = f = 0
        for k in range(case["frames"]):
            W, H, L = _uneven_shape(case, k)
            x, y = _frame_work(W, H, DTYPES[case["dtype"]][1], L, 2, 0)
            b, f = b + x, f + y
    elif kind == "integrate":
        px = case["width"] * case["height"] * case["frames"]
        # of omega_y only the anchor column is needed
        b = px * (4 + 8) + (4 * case["height"] * case["frames"] if case["both"] else 0)
        f = 3 * px
    elif kind == "train":
        b = case["steps"] * case["batch"] * 34 * 4
        f = case["steps"] * case["batch"] * 3 * 2 * (32 * 64 + 64 * 64 + 64 * 2)
    else:
        b = case["rows"] * (32 + 2 + 1) * 4
        f = case["rows"] * (_window_flops(8) + 128 * 60 + 33 * 100)
    return {"bytes": float(b), "flops": float(f)}


# ----------------------------------------------------------------------------
# The same results in 64 bits, in plain torch
# ----------------------------------------------------------------------------
def _analytic(lines):
    """Analytic signal of real lines (last axis): the one-sided DFT mask without DC and Nyquist."""
    n = lines.shape[-1]
    h = torch.zeros(n, dtype=torch.float64, device=lines.device)
    h[1:(n + 1) // 2] = 2.0
    return torch.fft.ifft(torch.fft.fft(lines.double(), dim=-1) * h, dim=-1)


def _omega_of(R):
    """Root-MUSIC frequency of each Hermitian L x L covariance of R (n, L, L)."""
    L = R.shape[-1]
    n = 2 * L - 2
    R = R + torch.flip(R.conj(), (1, 2))
    M = R / torch.diagonal(R, dim1=1, dim2=2).real.sum(1)[:, None, None]
    for _ in range(11):                                     # M^(2^11): the projector on the top eigenvector
        M = torch.matmul(M, M)
        M = M / torch.diagonal(M, dim1=1, dim2=2).real.sum(1)[:, None, None]
    k = torch.diagonal(M, dim1=1, dim2=2).real.argmax(1)
    u = torch.gather(M, 2, k[:, None, None].expand(-1, L, 1))[:, :, 0]
    u = u / u.abs().square().sum(1, keepdim=True).sqrt()
    c = torch.stack([(u[:, :L - k] * u[:, k:].conj()).sum(1) for k in range(L)], 1)
    a = torch.empty((R.shape[0], n + 1), dtype=torch.complex128, device=R.device)
    a[:, L - 1:] = -c
    a[:, L - 1] += L
    a[:, :L - 1] = torch.flip(a[:, L:].conj(), (1,))
    # all roots by Aberth's iteration, from two circles of L - 1 points turned to the lag-1 frequency
    w0 = -torch.angle(c[:, 1:2])
    th = 2 * math.pi * torch.arange(L - 1, dtype=torch.float64, device=R.device) / (L - 1)
    rad = torch.where(th == 0, 0.93, 0.55).double()
    z = torch.cat((torch.polar(rad.expand(len(R), -1), w0 + th + 0.01),
                   torch.polar((1 / rad).expand(len(R), -1), w0 + th - 0.01)), 1)
    eye = torch.eye(n, dtype=torch.bool, device=R.device)
    for _ in range(60):
        out = z.abs() > 1                                   # evaluated at 1/z: no overflow
        e = torch.where(out, 1 / z, z)
        p, q, d, g = a[:, n:n + 1].expand_as(z), a[:, :1].expand_as(z), torch.zeros_like(z), torch.zeros_like(z)
        for j in range(1, n + 1):
            d, g = d * e + p, g * e + q
            p, q = p * e + a[:, n - j:n - j + 1], q * e + a[:, j:j + 1]
        step = torch.where(out, z * q / (n * q - e * g), p / d)
        diff = z[:, :, None] - z[:, None, :]
        inv = torch.where(eye, 0, 1 / torch.where(eye, 1, diff))
        step = step / (1 - step * inv.sum(2))
        step = torch.where(torch.isfinite(torch.view_as_real(step)).all(-1), step, 0)
        z = z - step
        if float((step.abs() / z.abs().clamp(min=1e-3)).max()) < 1e-13:
            break
    i = (z.abs() - 1).abs().argmin(1, keepdim=True)
    zs = torch.gather(z, 1, i)
    away = (z - 1 / zs.conj()).abs().scatter(1, i, math.inf)
    zm = torch.gather(z, 1, away.argmin(1, keepdim=True))
    return torch.angle((zs + zm)[:, 0])


def _chunked(R_of, count, L):
    chunk = max(4096, (1 << 26) // (2 * L) ** 2)
    return torch.cat([_omega_of(R_of(i, min(count, i + chunk))) for i in range(0, count, chunk)])


def _sums(g, L, K):
    """Lag sums S_d[m] = sum_{k<K} g[m+k] conj(g[m+k+d]) along the last axis, d < L, zero beyond the end."""
    n = g.shape[-1]
    out = []
    for d in range(L):
        p = torch.zeros(g.shape[:-1] + (n + K,), dtype=torch.complex128, device=g.device)
        p[..., 1:n - d + 1] = g[..., :n - d] * g[..., d:].conj()
        c = p.cumsum(-1)
        out.append(c[..., K:K + n] - c[..., :n])
    return torch.stack(out)


def _line_omega(g, L, N):
    """omega of every window of the lines g (rows, length), NaN where the window does not fit."""
    rows, n = g.shape
    out = torch.full((rows, n), math.nan, dtype=torch.float64, device=g.device)
    cols = n - N + 1
    if cols <= 0:
        return out
    S = _sums(g, L, N - L + 1)
    i = torch.arange(L, device=g.device)
    lag, row = (i[None, :] - i[:, None]).abs(), torch.minimum(i[:, None], i[None, :])
    low = i[:, None] > i[None, :]

    def cov(a, b):
        m = torch.arange(a, b, device=g.device)
        r, x = (m // cols)[:, None, None], (m % cols)[:, None, None]
        v = S[lag, r, x + row]
        return torch.where(low, v.conj(), v)

    out[:, N // 2:N // 2 + cols] = _chunked(cov, rows * cols, L).view(rows, cols)
    return out


def _block_omega(g, L, phase):
    """omega_x, omega_y (and the block phase) of the L x L blocks of the complex field g."""
    H, W = g.shape
    h, cw, ch = L // 2, W - L + 1, H - L + 1
    maps = [torch.full((H, W), math.nan, dtype=torch.float64, device=g.device) for _ in range(3 if phase else 2)]
    if cw <= 0 or ch <= 0:
        return maps
    blocks = g.unfold(0, L, 1).unfold(1, L, 1).reshape(-1, L, L) if ch * cw < 1 << 18 else None

    def block(a, b):
        if blocks is not None:
            return blocks[a:b]
        m = torch.arange(a, b, device=g.device)
        i = torch.arange(L, device=g.device)
        return g[(m // cw)[:, None, None] + i[:, None], (m % cw)[:, None, None] + i[None, :]]

    def cov(direction):
        def f(a, b):
            B = block(a, b)
            s = B if direction == "y" else B.transpose(1, 2).contiguous()     # snapshots are the columns
            return torch.matmul(s, s.conj().transpose(1, 2).contiguous())
        return f

    wx, wy = _chunked(cov("x"), ch * cw, L), _chunked(cov("y"), ch * cw, L)
    got = [wx, wy]
    if phase:
        i = torch.arange(L, dtype=torch.float64, device=g.device) - h
        parts = []
        for a in range(0, ch * cw, 1 << 16):
            b = min(ch * cw, a + (1 << 16))
            ex = torch.polar(torch.ones((), dtype=torch.float64, device=g.device), -wx[a:b, None] * i)
            ey = torch.polar(torch.ones((), dtype=torch.float64, device=g.device), -wy[a:b, None] * i)
            parts.append(torch.angle((block(a, b) * ex[:, None, :] * ey[:, :, None]).sum((1, 2))))
        got.append(torch.cat(parts))
    for m, v in zip(maps, got):
        m[h:h + ch, h:h + cw] = v.view(ch, cw)
    return maps


def _xy_omega(img, L, N, dirs):
    """(omega_x or None, omega_y or None) of one frame, real or complex."""
    out = []
    for d, a in (("x", img), ("y", img.T)):
        if d not in dirs:
            out.append(None)
            continue
        g = a.to(torch.complex128) if a.is_complex() else _analytic(a)
        w = _line_omega(g, L, N)
        out.append(w if d == "x" else w.T.contiguous())
    return out


def _adam(case, seed):
    """The training steps in FP64: mean squared error, exact GELU, Adam (0.9, 0.999, 1e-8)."""
    X, T = (t.double() for t in _windows(case["rows"], seed))
    p = torch.from_numpy(_weights(seed)).to("cuda", torch.float64)
    m, v, losses = torch.zeros_like(p), torch.zeros_like(p), []
    b, batches = case["batch"], case["rows"] // case["batch"]
    gelu = torch.nn.functional.gelu
    for t in range(case["steps"]):
        q = p.clone().requires_grad_(True)
        W1, b1, W2, b2, W3, b3 = (w.view(s) for w, s in zip(q.split((2048, 64, 4096, 64, 128, 2)),
                                                            ((32, 64), (64,), (64, 64), (64,), (64, 2), (2,))))
        rows = slice(t % batches * b, (t % batches + 1) * b)
        y = gelu(gelu(X[rows] @ W1 + b1) @ W2 + b2) @ W3 + b3
        loss = (y - T[rows]).square().sum(1).mean()
        g, = torch.autograd.grad(loss, q)
        losses.append(loss.detach())
        m, v = 0.9 * m + 0.1 * g, 0.999 * v + 0.001 * g * g
        p = p - case["lr"] * (m / (1 - 0.9 ** (t + 1))) / ((v / (1 - 0.999 ** (t + 1))).sqrt() + 1e-8)
    return [torch.stack(losses), p]


def _philox(c, seed):
    """Philox4x32-10 of the counters c (..., 4): int64 words of 32 bits, products taken modulo 2^64."""
    low = 0xFFFFFFFF
    c0, c1, c2, c3 = c.unbind(-1)
    k0, k1 = seed & low, seed >> 32 & low
    for _ in range(10):
        p0, p1 = 0xD2511F53 * c0, 0xCD9E8D57 * c2
        c0, c1, c2, c3 = (p1 >> 32 & low) ^ c1 ^ k0, p1 & low, (p0 >> 32 & low) ^ c3 ^ k1, p0 & low
        k0, k1 = k0 + 0x9E3779B9 & low, k1 + 0xBB67AE85 & low
    return (torch.stack((c0, c1, c2, c3), -1).double() + 0.5) / 4294967296.0


def _dataset(case, seed):
    n = case["rows"]
    c = torch.zeros((n, 33, 4), dtype=torch.int64, device="cuda")
    c[:, :, 0] = torch.arange(case["first"], case["first"] + n, device="cuda")[:, None]
    c[:, :, 1] = torch.arange(33, device="cuda")
    u = _philox(c, int(seed))
    w = 2 * math.pi / 16 + u[:, 0, :1] * (2 * math.pi / 4 - 2 * math.pi / 16)
    th = 2 * math.pi * u[:, 0, 1:2]
    sig = torch.sqrt(0.08 * 10.0 ** (-3.0 * u[:, 0, 2:3]))
    q = u[:, 1:]
    z = [torch.sqrt(-2 * torch.log(q[..., i])) * f(2 * math.pi * q[..., i + 1]) for i in (0, 2)
         for f in (torch.cos, torch.sin)]
    t = torch.arange(128, dtype=torch.float64, device="cuda")
    g = _analytic(A_DC + B_AC * torch.cos(w * t + th) + sig * torch.stack(z, -1).view(n, 128))[:, 48:80].contiguous()
    omega = _line_omega(g, 8, 32)[:, 16]
    x = g[:, 8:24] * torch.conj(g[:, 16:17]) / g[:, 16:17].abs() / g.abs().square().mean(1, keepdim=True).sqrt()
    return [torch.cat((x.real, x.imag), 1), torch.stack((torch.cos(omega), torch.sin(omega)), 1), omega]


def _integral(case, seed):
    N, W, H = case["N"], case["width"], case["height"]
    maps = _maps(case, seed)
    cx, cy = (0.5, 0.6) if case["carrier"] else (0.0, 0.0)
    phi = torch.full(maps[0].shape, math.nan, dtype=torch.float64, device="cuda")
    x0, x1 = N // 2, W - N + N // 2 + 1
    y0, y1 = (x0, H - N + N // 2 + 1) if case["both"] else (0, H)
    if x1 <= x0 or y1 <= y0:
        return phi

    def trapezoid(v):
        out = torch.zeros_like(v)
        out[..., 1:] = (0.5 * (v[..., 1:] + v[..., :-1])).cumsum(-1)
        return out

    for t in range(case["frames"]):
        part = trapezoid(maps[0][t, y0:y1, x0:x1].double() - cx)
        if case["both"]:
            part += trapezoid(maps[1][t, y0:y1, x0].double() - cy)[:, None]
        phi[t, y0:y1, x0:x1] = part
    return phi


def exact(case, seed):
    kind = case["kind"]
    if kind == "train":
        return _adam(case, seed)
    if kind == "dataset":
        return _dataset(case, seed)
    if kind == "integrate":
        return _integral(case, seed)
    if kind == "uneven":
        shapes = [_uneven_shape(case, k) for k in range(case["frames"])]
        if 2 * sum(W * H for W, H, _ in shapes) > EXACT_WINDOWS:
            return None
        maps = [_xy_omega(f, L, 2 * L + 8, "xy") for f, L in _uneven(case, seed)]
        return [torch.cat([m[k].reshape(-1) for m in maps]) for k in (0, 1)]
    windows = len(case["dirs"]) * case["width"] * case["height"] * case.get("frames", 1)
    if windows * max(1.0, (case["L"] / 8.0) ** 2) > EXACT_WINDOWS:
        return None
    data = _stack(case, seed)
    if kind == "frame":
        out = _xy_omega(data[0], case["L"], case["N"], case["dirs"])
        return out + [None] if case["flags"] else out
    if kind == "block":
        maps = [_block_omega(_analytic(f), case["L"], case["phase"]) for f in data]
    else:
        maps = [_xy_omega(f, case["L"], case["N"], case["dirs"]) for f in data]
    return [torch.stack(m) for m in zip(*maps)]
