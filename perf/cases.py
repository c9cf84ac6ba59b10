"""Timed cases: the calls that a program using this library spends its time in.

Each case prepares what a program has in hand (a stream with a full window,
the next frames on the GPU, output buffers) and a pass makes the calls of one
step through the package's public entry points:

  push    one new snapshot into a dense window, then the DMD modes or the POD
          modes; with "read" the eigenvalues and singular values are read on
          the host as well, as a controller or monitor does every frame
  bg      one new frame, then its background subtraction
  block   k new snapshots at once, then the modes of all k windows, on two
          streams as a pipelined ingest does
  sparse  one sparse complex (Fourier-coefficient) snapshot, then the modes
  fourier the same from a spatial frame, transformed on the device
  gram    the stateless Gram of a whole window (a first fill, a resync)
  tick    one frame for each of many unlike streams, with their modes

Snapshots are a few oscillating patterns with amplitudes over one decade, a
constant background in odd ranks and in every video case, and pixel noise of
1e-3: as many patterns as modes are asked for.  Frames repeat with a period
longer than the window, so that a stream can be advanced for ever without a
jump in its data.
"""

import math

import numpy as np
import torch

import paper_1612_07875_amd as dmd

NOISE = 1e-3


def listed():
    return [
        # a small FP64 sensor array followed frame by frame: latency is all that counts
        dict(name="modal_f64", kind="push", n=4096, m=32, r=10, dtype="f64", out="modes", read=True),
        # the smallest stream of the serving mix, eigenvalues read every frame
        dict(name="small_f32", kind="push", n=65536, m=16, r=8, dtype="f32", out="modes", read=True),
        # full-HD video, one frame at a time
        dict(name="hd_frame", kind="push", n=1920 * 1080, m=64, r=20, dtype="f32", out="modes", read=False),
        # a long window over a simulation's field: the small solves at their largest
        dict(name="waves_m256", kind="push", n=1 << 20, m=256, r=32, dtype="f32", out="modes", read=False),
        # streaming SVD of 2560 x 1440 video with 90 columns: singular values read, POD modes kept
        dict(name="svd_1440p", kind="push", n=2560 * 1440, m=90, r=16, dtype="f32", out="pod", read=True),
        # background subtraction of full-HD video with 120 columns
        dict(name="hd_background", kind="bg", n=1920 * 1080, m=120, r=15, dtype="f32"),
        # full-HD video in blocks of 32 frames, every window solved and projected
        dict(name="hd_block32", kind="block", n=1920 * 1080, m=64, r=20, k=32, precision="default"),
        # the same with split-BF16 projections
        dict(name="hd_block32_bf16x3", kind="block", n=1920 * 1080, m=64, r=20, k=32, precision="bf16x3"),
        # 512 x 512 Fourier coefficients at 1 %, 5 % of the support new in every frame
        dict(name="sparse_512", kind="sparse", side=512, nnz=2621, m=128, r=24),
        # first fill of the longest window from FP64 data
        dict(name="gram_f64_257", kind="gram", n=1 << 20, k=257, dtype="f64", precision="default"),
        # first fill of the full-HD window
        dict(name="gram_f32_65", kind="gram", n=1920 * 1080, k=65, dtype="f32", precision="default"),
        # a serving tick: 24 unlike streams, one frame and the modes of each
        dict(name="tick_24", kind="tick", streams=24, n_lo=65536, n_hi=2097152),
    ]


def _log_int(rng, lo, hi):
    return max(lo, min(hi, int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))))


def draw(rng):
    kind = rng.choice(["push", "push", "push", "push", "bg", "block", "block", "sparse", "fourier", "gram", "gram", "tick"])
    if kind in ("push", "bg"):
        m = _log_int(rng, 12, 256)
        r = rng.randint(2, max(2, min(32, m // 3)))
        n = _log_int(rng, 2000, 3686400)
        dtype = rng.choice(["f32", "f32", "f32", "f64"])
        if dtype == "f64" or m > 128:
            n = min(n, 1 << 21)
        c = dict(kind=kind, n=n, m=m, r=r, dtype=dtype)
        if kind == "push":
            c.update(out=rng.choice(["modes", "modes", "pod"]), read=rng.random() < 0.5)
        return c
    if kind == "block":
        m = _log_int(rng, 16, 128)
        return dict(kind=kind, n=_log_int(rng, 65536, 1920 * 1080), m=m, r=rng.randint(4, min(24, m // 3)),
                    k=rng.randint(4, 32), precision=rng.choice(["default", "default", "bf16x3"]))
    if kind in ("sparse", "fourier"):
        side = _log_int(rng, 128, 512)
        m = _log_int(rng, 16, 128)
        return dict(kind=kind, side=side, nnz=max(64, int(side * side * rng.uniform(0.005, 0.012))), m=m,
                    r=rng.randint(4, min(24, m // 3)))
    if kind == "gram":
        k = _log_int(rng, 9, 257)
        dtype = rng.choice(["f32", "f64"])
        return dict(kind=kind, n=_log_int(rng, 4096, 1 << 20), k=k, dtype=dtype,
                    precision=rng.choice(["default", "fp64"]))
    lo = _log_int(rng, 20000, 131072)
    return dict(kind="tick", streams=rng.randint(3, 24), n_lo=lo, n_hi=_log_int(rng, 200000, 2097152))


# ---------------------------------------------------------------- data
def _gen(seed):
    g = torch.Generator(device="cuda")
    g.manual_seed((int(seed) * 1000003 + 12345) % (1 << 62))
    return g


def _period(m, k=1):
    """Frames before the data repeat: more than the m + k columns in use, a multiple of 2 k."""
    p = max(m + k + 1, int(1.25 * (m + 1)) + 1)
    return -(-p // (2 * k)) * 2 * k


def _frames(n, m, r, dtype, seed, video=False, period=None):
    """(P, n) snapshots of rank r plus noise with period P."""
    P = period or _period(m)
    rng = np.random.default_rng([7, int(seed)])
    t = np.arange(P)
    cols = []
    if r % 2 or video:
        cols.append(np.ones(P))
    if video and r % 2 == 0:
        cols.append(0.2 * (-1.0) ** t)  # a flicker at half the frame rate
    waves = (r - len(cols)) // 2
    step = max(1, (P // 2 - 1) // (waves + 1)) if waves else 1
    for j in range(waves):
        w = 2 * np.pi * (step * (j + 1)) / P
        a, ph = 10.0 ** (-j / max(1, waves)), rng.uniform(0, 2 * np.pi)
        cols += [a * np.cos(w * t + ph), a * np.sin(w * t + ph)]
    C = torch.tensor(np.stack(cols, axis=1), device="cuda")
    dt = torch.float64 if dtype == "f64" else torch.float32
    g = _gen(seed)
    out = torch.empty((P, n), dtype=dt, device="cuda")
    chunk = max(1, (1 << 27) // max(P, 1))
    for a in range(0, n, chunk):
        b = min(n, a + chunk)
        S = torch.randn((C.shape[1], b - a), generator=g, device="cuda", dtype=torch.float32).to(dt)
        if r % 2 or video:
            S[0] = torch.rand(b - a, generator=g, device="cuda", dtype=torch.float32).to(dt)
        out[:, a:b] = C.to(dt) @ S
        out[:, a:b] += NOISE * torch.randn((P, b - a), generator=g, device="cuda", dtype=torch.float32).to(dt)
    return out


def _lowest(side, count):
    k = np.arange(side)
    k = np.where(k < (side + 1) // 2, k, k - side)
    k2 = (k[:, None] ** 2 + k[None, :] ** 2).reshape(-1)
    return np.lexsort((np.arange(side * side), k2))[:count], k


def _sparse_frames(side, nnz, m, seed):
    """P sparse frames: nnz of the 2 nnz lowest wavenumbers, 5 % of them new in each frame, advected."""
    rng = np.random.default_rng([11, int(seed)])
    P = _period(m)
    pool, k = _lowest(side, 2 * nnz)
    ky, kx = k[pool // side], k[pool % side]
    amp = (rng.standard_normal(2 * nnz) + 1j * rng.standard_normal(2 * nnz)) * np.maximum(np.hypot(ky, kx), 1.0) ** (-5.0 / 3.0)
    cycles = np.round((3.0 * kx + 1.7 * ky) * P / side)  # turns per period
    inside = np.zeros(2 * nnz, dtype=bool)
    inside[:nnz] = True
    swap = max(1, nnz // 20)
    frames = []
    for t in range(P):
        if t:
            drop = rng.choice(np.flatnonzero(inside), swap, replace=False)
            add = rng.choice(np.flatnonzero(~inside), swap, replace=False)
            inside[drop], inside[add] = False, True
        sel = np.flatnonzero(inside)
        sel = sel[np.argsort(pool[sel])]
        val = amp[sel] * np.exp(2j * np.pi * cycles[sel] * t / P)
        frames.append((torch.tensor(pool[sel].astype(np.int32), device="cuda"),
                       torch.tensor(val.astype(np.complex64), device="cuda")))
    return frames


def _field_frames(side, m, seed):
    """P spatial frames (side x side) of a smooth random field carried along, plus noise."""
    P = _period(m)
    g = _gen(seed)
    k = torch.fft.fftfreq(side, 1.0 / side, device="cuda", dtype=torch.float64)
    k2 = k[:, None] ** 2 + k[None, :] ** 2
    spec = torch.fft.fft2(torch.randn((side, side), generator=g, device="cuda", dtype=torch.float64))
    spec = spec * torch.clamp(k2, min=1.0) ** (-5.0 / 6.0)
    turns = torch.round((1.7 * k[:, None] + 3.0 * k[None, :]) * P / side)
    out = torch.empty((P, side, side), dtype=torch.float32, device="cuda")
    for t in range(P):
        f = torch.fft.ifft2(spec * torch.exp(-2j * math.pi * t / P * turns)).real
        out[t] = f.float() + NOISE * torch.randn((side, side), generator=g, device="cuda")
    return out


def _tick_streams(case, seed):
    rng = np.random.default_rng([13, case["streams"], case["n_lo"], case["n_hi"]])
    shapes = []
    for i in range(case["streams"]):
        n = int(round(math.exp(rng.uniform(math.log(case["n_lo"]), math.log(case["n_hi"])))))
        m = (16, 32, 64, 128)[i % 4]
        shapes.append((n, m, min(m // 2 - m // 8, 32), int(seed) * 64 + i))
    return shapes


# ---------------------------------------------------------------- cases
_STREAMS = []


def _two_streams():
    """A program's ingest stream and projection stream."""
    if not _STREAMS:
        _STREAMS.extend([torch.cuda.Stream(), torch.cuda.Stream()])
    return _STREAMS


def _fill(s, X, m):
    for t in range(m + 1):
        s.push(X[t])


def prepare(case, seed):
    kind = case["kind"]
    st = dict(case=case, t=0)
    if kind in ("push", "bg"):
        n, m, r = case["n"], case["m"], case["r"]
        st["x"] = _frames(n, m, r, case["dtype"], seed, video=kind == "bg" or case.get("out") == "pod")
        s = st["s"] = dmd.Stream(n, m, r, dtype=case["dtype"])
        _fill(s, st["x"], m)
        st["t"] = m + 1
        if kind == "bg":
            st["out"] = [torch.zeros(n, dtype=s.pod_dtype, device="cuda") for _ in range(2)]
        else:
            st["out"] = torch.zeros((r, n), dtype=s.mode_dtype if case["out"] == "modes" else s.pod_dtype, device="cuda").T
    elif kind == "block":
        n, m, r, k = case["n"], case["m"], case["r"], case["k"]
        st["x"] = _frames(n, m, r, "f32", seed, video=True, period=_period(m, k))
        s = st["s"] = dmd.Stream(n, m, r, max_block=k, precision=case["precision"])
        P = st["x"].shape[0]
        while st["t"] < m + 1:
            s.push_block(st["x"][st["t"]:st["t"] + k])
            st["t"] = (st["t"] + k) % P
        s.sync()
        st["out"] = torch.zeros((k, r, n), dtype=s.mode_dtype, device="cuda")
    elif kind in ("sparse", "fourier"):
        side, m, r, nnz = case["side"], case["m"], case["r"], case["nnz"]
        s = st["s"] = dmd.Stream(side * side, m, r, dtype="c64_csr", max_nnz=nnz)
        if kind == "sparse":
            st["x"] = _sparse_frames(side, nnz, m, seed)
            for t in range(m + 1):
                s.push_csr(*st["x"][t])
        else:
            s.fourier_setup(side, side, nnz)
            st["x"] = _field_frames(side, m, seed)
            for t in range(m + 1):
                s.push_fourier(st["x"][t])
        st["t"] = m + 1
        st["out"] = torch.zeros((r, side * side), dtype=s.mode_dtype, device="cuda").T
    elif kind == "gram":
        n, k = case["n"], case["k"]
        per = 16 // (8 if case["dtype"] == "f64" else 4)
        ld = -(-n // per) * per  # columns 16 bytes aligned, as the call asks for
        x = _frames(n, k, min(32, max(2, k // 3)), case["dtype"], seed)[:k]
        if ld != n:
            x = torch.nn.functional.pad(x, (0, ld - n))[:, :n]
        st["x"] = x
        st["out"] = torch.empty((k, k), dtype=torch.float64, device="cuda")
    else:
        b = st["b"] = dmd.Batch(max_streams=case["streams"])
        st["x"], st["s"], st["out"] = [], [], []
        for n, m, r, sd in _tick_streams(case, seed):
            x = _frames(n, m, r, "f32", sd)
            s = dmd.Stream(n, m, r)
            _fill(s, x, m)
            b.attach(s)
            st["x"].append(x)
            st["s"].append(s)
            st["out"].append(torch.zeros((r, n), dtype=torch.complex64, device="cuda").T)
        st["at"] = [s.m + 1 for s in st["s"]]
    return st


def run(st):
    case, t = st["case"], st["t"]
    kind = case["kind"]
    s = st.get("s")
    if kind == "push":
        s.push(st["x"][t])
        st["t"] = (t + 1) % st["x"].shape[0]
        out = s.modes(st["out"]) if case["out"] == "modes" else s.pod(st["out"])
        if not case["read"]:
            return out
        lam, sigma, _ = s.eigs()
        return [out, lam, sigma]
    if kind == "bg":
        s.push(st["x"][t])
        st["t"] = (t + 1) % st["x"].shape[0]
        s.background(*st["out"])
        return st["out"]
    if kind == "block":
        ingest, project = _two_streams()
        s.push_block(st["x"][t:t + case["k"]], stream=ingest)
        st["t"] = (t + case["k"]) % st["x"].shape[0]
        return s.block_modes(st["out"], stream=project)
    if kind == "sparse":
        s.push_csr(*st["x"][t])
        st["t"] = (t + 1) % len(st["x"])
        return s.modes(st["out"])
    if kind == "fourier":
        s.push_fourier(st["x"][t])
        st["t"] = (t + 1) % st["x"].shape[0]
        return s.modes(st["out"])
    if kind == "gram":
        return dmd.window_gram(st["x"], precision=case["precision"], out=st["out"])
    frames = [x[a] for x, a in zip(st["x"], st["at"])]
    st["at"] = [(a + 1) % x.shape[0] for x, a in zip(st["x"], st["at"])]
    st["b"].tick(st["s"], frames, modes=st["out"])
    return st["out"]


# ---------------------------------------------------------------- least work
def _small(m, r, cplx=False):
    """Operations of the small solves: tridiagonalization, r eigenvectors, A~, its Schur form and vectors."""
    return (4 if cplx else 1) * (4.0 / 3 * m ** 3 + 4.0 * m * m * r + 4.0 * m * r * r) + 25.0 * r ** 3 + 8.0 * m * r * r


def work(case):
    kind = case["kind"]
    if kind in ("push", "bg"):
        n, m, r = case["n"], case["m"], case["r"]
        e = 8 if case["dtype"] == "f64" else 4
        if kind == "bg":
            out, cols = 2 * n * e, 2
        elif case["out"] == "modes":
            out, cols = n * r * 2 * e, 2 * r
        else:
            out, cols = n * r * e, r
        return dict(bytes=(m + 3) * n * e + out, flops=2.0 * n * (m + 1) + 2.0 * n * m * cols + _small(m, r))
    if kind == "block":
        n, m, r, k = case["n"], case["m"], case["r"], case["k"]
        return dict(bytes=(m + 2 * k) * n * 4 + k * n * r * 8,
                    flops=2.0 * n * k * (m + 1) + 2.0 * n * m * 2 * r * k + k * _small(m, r))
    if kind in ("sparse", "fourier"):
        n, m, r, z = case["side"] ** 2, case["m"], case["r"], case["nnz"]
        first = 0.0 if kind == "sparse" else 4.0 * n
        fft = 0.0 if kind == "sparse" else 5.0 * n * math.log2(n)
        return dict(bytes=(m + 2) * z * 12 + n * r * 8 + first,
                    flops=8.0 * (m + 1) * z + 8.0 * m * z * r + _small(m, r, True) + fft)
    if kind == "gram":
        e = 8 if case["dtype"] == "f64" else 4
        return dict(bytes=case["k"] * case["n"] * e + case["k"] ** 2 * 8, flops=1.0 * case["n"] * case["k"] * (case["k"] + 1))
    total = dict(bytes=0.0, flops=0.0)
    for n, m, r, _ in _tick_streams(case, 0):
        w = work(dict(kind="push", n=n, m=m, r=r, dtype="f32", out="modes"))
        total = dict(bytes=total["bytes"] + w["bytes"], flops=total["flops"] + w["flops"])
    return total


# ---------------------------------------------------------------- 64 bits
def _solve(G, m, r):
    """sigma, V, lambda, W (leading r) of the Gram of m + 1 columns, in the library's conventions."""
    cplx = np.iscomplexobj(G)
    d, V = np.linalg.eigh(G[:m, :m])
    order = np.argsort(-np.abs(d), kind="stable")[:r]
    sigma, V = np.sqrt(np.abs(d[order])), V[:, order]
    big = V[np.argmax(np.abs(V), axis=0), np.arange(r)]
    V = V * (np.conj(big) / np.abs(big))
    A = (V.conj().T @ G[:m, 1:m + 1] @ V) / np.outer(sigma, sigma)
    lam, W = np.linalg.eig(A if cplx else A.real)
    lam, W = lam.astype(np.complex128), W.astype(np.complex128)
    order = np.lexsort((np.angle(lam), -np.abs(lam)))
    lam, W = lam[order], W[:, order]
    W = W / np.linalg.norm(W, axis=0)
    big = W[np.argmax(np.abs(W), axis=0), np.arange(r)]
    return sigma, V, lam, W * (np.conj(big) / np.abs(big))


def _modes64(X, m, coef):
    """(coef columns, n) combinations of the m rows of X."""
    C = torch.tensor(np.ascontiguousarray(coef.T), device="cuda")
    if X.is_complex() or not C.is_complex():
        return C @ X
    return torch.complex(C.real.contiguous() @ X, C.imag.contiguous() @ X)


def _window64(x, P, first, m):
    rows = [(first + i) % P for i in range(m + 1)]
    return x[rows].double()


def _gram64(X):
    return (X.conj() @ X.T).cpu().numpy() if X.is_complex() else (X @ X.T).cpu().numpy()


def exact(case, seed):
    kind = case["kind"]
    if kind in ("push", "bg"):
        m, r = case["m"], case["r"]
        x = _frames(case["n"], m, r, case["dtype"], seed, video=kind == "bg" or case.get("out") == "pod")
        X = _window64(x, x.shape[0], 1, m)
        sigma, V, lam, W = _solve(_gram64(X), m, r)
        if kind == "push":
            if case["out"] == "modes":
                out = _modes64(X[1:], m, (V / sigma) @ W).T
            else:
                out = _modes64(X[:m], m, V / sigma).T
            return [out, lam, sigma] if case["read"] else out
        b = np.linalg.solve(W * lam, sigma * V[0])
        i = int(np.argmin(np.abs(np.log(lam))))
        c = ((V / sigma) @ W[:, i]) * b[i] * lam[i] ** m
        bg = _modes64(X[1:], m, c[:, None])[0].abs()
        return [X[m] - bg, bg]
    if kind == "block":
        n, m, r, k = case["n"], case["m"], case["r"], case["k"]
        x = _frames(n, m, r, "f32", seed, video=True, period=_period(m, k))
        P = x.shape[0]
        end = -(-(m + 1) // k) * k + k  # frames pushed after one pass
        X = x[[(end - m - k + i) % P for i in range(m + k)]].double()  # the columns of all k windows
        del x
        G = _gram64(X)
        out = torch.empty((k, r, n), dtype=torch.complex128, device="cuda")
        for w in range(k):
            sigma, V, lam, W = _solve(G[w:w + m + 1, w:w + m + 1], m, r)
            out[w] = _modes64(X[w + 1:w + m + 1], m, (V / sigma) @ W)
        return out
    if kind in ("sparse", "fourier"):
        side, m, r, nnz = case["side"], case["m"], case["r"], case["nnz"]
        n = side * side
        X = torch.zeros((m + 1, n), dtype=torch.complex128, device="cuda")
        if kind == "sparse":
            for i, (idx, val) in enumerate(_sparse_frames(side, nnz, m, seed)[1:m + 2]):
                X[i, idx.long()] = val.to(torch.complex128)
        else:
            keep = torch.tensor(_lowest(side, nnz)[0], device="cuda")
            for i, f in enumerate(_field_frames(side, m, seed)[1:m + 2]):
                X[i, keep] = (torch.fft.fft2(f.double()) / side).reshape(-1)[keep]
        sigma, V, lam, W = _solve(_gram64(X), m, r)
        return _modes64(X[1:], m, (V / sigma) @ W).T
    if kind == "gram":
        x = _frames(case["n"], case["k"], min(32, max(2, case["k"] // 3)), case["dtype"], seed)[:case["k"]].double()
        return x @ x.T
    out = []
    for n, m, r, sd in _tick_streams(case, seed):
        x = _frames(n, m, r, "f32", sd)
        X = _window64(x, x.shape[0], 1, m)
        sigma, V, lam, W = _solve(_gram64(X), m, r)
        out.append(_modes64(X[1:], m, (V / sigma) @ W).T)
    return out
