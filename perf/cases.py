"""The work that users of this library have it do, as cases that can be timed.

Every case is one call (or one short sequence of calls) of the public entry
points on ultrasound-shaped windows: a speckle background of rank two that
drifts slowly, fixed bubbles, bubbles that move along straight tracks and
white noise.  Sizes come from the benchmark, the tests and the paper's windows.

FP32 solves run a fixed number of iterations (tol = 0, or the default
tolerance with a cap that is reached first), so that two runs that round
differently still do the same number; the FP64 latency case stops by its
tolerance.
"""
from __future__ import annotations

import math

import numpy as np
import torch

import paper_2506_10257_amd as rp
from paper_2506_10257_amd import postproc

PSF = 1.5          # px, blur of the speckle and size of the bubbles
AMPLITUDE = 3.0    # bubble amplitude over the mean of the tissue
DRIFT = 0.05       # size of the slow drift of the tissue


def listed() -> list:
    """The cases of every comparison."""
    return [
        # the smallest call in use (a 64 x 64 preview): host path and launches count
        {"name": "solve_64x64x10_f32", "kind": "solve", "H": 64, "W": 64, "n": 10,
         "dtype": "f32", "mode": 0, "tol": 0.0, "maxit": 25},
        # latency of one FP64 window, stopped by its tolerance
        {"name": "solve_128x128x20_f64", "kind": "solve", "H": 128, "W": 128, "n": 20,
         "dtype": "f64", "mode": 0, "tol": 1e-7, "maxit": 500},
        # sliding windows of the paper's in vivo size, each started from the
        # previous window's S and Y (odd number of pixels)
        {"name": "warm_338x260x20_f32", "kind": "warm", "H": 338, "W": 260, "n": 20,
         "dtype": "f32", "step": 5, "tol": 0.0, "maxit": 60},
        # the benchmark's window with the default tolerance and cap
        {"name": "solve_512x512x20_f32", "kind": "solve", "H": 512, "W": 512, "n": 20,
         "dtype": "f32", "mode": 0, "tol": 1e-7, "maxit": 500},
        # the same window in FP64
        {"name": "solve_512x512x20_f64", "kind": "solve", "H": 512, "W": 512, "n": 20,
         "dtype": "f64", "mode": 0, "tol": 0.0, "maxit": 150},
        # large images, split-BF16 contractions at FP32 accuracy
        {"name": "solve_1024x1024x40_bf16x6", "kind": "solve", "H": 1024, "W": 1024, "n": 40,
         "dtype": "f32", "mode": 2, "tol": 0.0, "maxit": 40},
        # offline processing: every (image size x frames) cell of the batch workload
        {"name": "batch_16_windows_f32", "kind": "many", "count": 16, "dtype": "f32",
         "pick": 0, "tol": 0.0, "maxit": 50},
        # continuous batching of requests of mixed sizes, 100-frame ones among them
        {"name": "serve_12_requests_f32", "kind": "serve", "count": 12, "dtype": "f32",
         "pick": 0, "quantum": 16, "tol": 0.0, "maxit": 48},
        # long windows: the serve workload's longest and the paper's in vivo window
        {"name": "solve_512x512x100_f32", "kind": "solve", "H": 512, "W": 512, "n": 100,
         "dtype": "f32", "mode": 0, "tol": 0.0, "maxit": 40},
        {"name": "solve_512x512x132_f32", "kind": "solve", "H": 512, "W": 512, "n": 132,
         "dtype": "f32", "mode": 0, "tol": 0.0, "maxit": 40},
        # a long window in FP64, ragged rows and an odd number of frames
        {"name": "solve_251x383x97_f64", "kind": "solve", "H": 251, "W": 383, "n": 97,
         "dtype": "f64", "mode": 0, "tol": 0.0, "maxit": 20},
        # the steps around the solve, on a full in vivo sequence
        {"name": "process_1024x1024x132_f32", "kind": "process", "H": 1024, "W": 1024, "n": 132,
         "W_avg": 20, "dtype": "f32"},
    ]


MOST = 512 * 512 * 132  # entries of the largest single window drawn


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng) -> dict:
    """One more case of the listed cases' ranges."""
    kind = rng.choice(["solve", "solve", "solve", "long", "long", "warm", "many", "serve", "process"])
    if kind == "solve":  # up to 64 frames
        n = rng.choice([rng.randint(2, 24), rng.randint(8, 32), rng.randint(33, 64)])
        dtype = rng.choice(["f32", "f32", "f64"])
        side = _log_int(rng, 48, 640)
        H, W = side, max(32, int(side * rng.uniform(0.6, 1.4)))
        mode = 2 if dtype == "f32" and n > 8 and rng.random() < 0.2 else 0
        return {"kind": "solve", "H": H, "W": W, "n": n, "dtype": dtype, "mode": mode, "tol": 0.0,
                "maxit": _log_int(rng, 20, 150)}
    if kind == "long":  # 65 frames and more
        dtype = rng.choice(["f32", "f32", "f64"])
        n = rng.randint(65, 144 if dtype == "f32" else 128)
        side = _log_int(rng, 64, 480)
        H, W = side, max(32, int(side * rng.uniform(0.6, 1.4)))
        while H * W * n > MOST:
            W -= 8
        return {"kind": "solve", "H": H, "W": W, "n": n, "dtype": dtype, "mode": 0, "tol": 0.0,
                "maxit": _log_int(rng, 8, 30)}
    if kind == "warm":
        n = rng.randint(8, 40)
        side = _log_int(rng, 96, 320)
        return {"kind": "warm", "H": side, "W": max(32, int(side * rng.uniform(0.6, 1.4))), "n": n,
                "dtype": rng.choice(["f32", "f32", "f64"]), "step": rng.randint(1, max(1, n // 3)),
                "tol": 0.0, "maxit": _log_int(rng, 20, 60)}
    if kind == "many":
        return {"kind": "many", "count": rng.randint(2, 16), "dtype": rng.choice(["f32", "f32", "f64"]),
                "pick": rng.randint(1, 10**6), "tol": 0.0, "maxit": _log_int(rng, 16, 50)}
    if kind == "serve":
        return {"kind": "serve", "count": rng.randint(2, 12), "dtype": "f32",
                "pick": rng.randint(1, 10**6), "quantum": rng.choice([7, 16]), "tol": 0.0,
                "maxit": _log_int(rng, 12, 48)}
    n = rng.randint(24, 132)
    side = _log_int(rng, 100, 1000)
    return {"kind": "process", "H": side, "W": max(64, int(side * rng.uniform(0.6, 1.0))), "n": n,
            "W_avg": rng.randint(1, 24), "dtype": rng.choice(["f32", "f64"])}


def _shapes(case) -> list:
    """(H, W, n) of the windows of a batch or of a serving run."""
    if case["kind"] == "many":
        if case["pick"] == 0:
            return [(h, w, n) for h, w in ((256, 256), (384, 512), (512, 512), (512, 768))
                    for n in (10, 20, 40, 60)][: case["count"]]
        r = np.random.default_rng(case["pick"])
        return [(int(r.integers(64, 513)), int(r.integers(64, 641)), int(r.integers(4, 61)))
                for _ in range(case["count"])]
    if case["pick"] == 0:
        sides = (256, 512, 1024, 384, 640, 288, 448, 768, 320, 576, 352, 416)
        frames = (20, 100, 10, 40, 20, 100, 10, 20, 100, 10, 40, 20)
        return [(s, s, n) for s, n in zip(sides, frames)][: case["count"]]
    r = np.random.default_rng(case["pick"])
    return [(32 * int(r.integers(4, 21)),) * 2 + (int(r.choice([10, 20, 40, 100])),)
            for _ in range(case["count"])]


def _speckle(gen, H, W, dev):
    fy = torch.fft.fftfreq(H, device=dev, dtype=torch.float64)
    fx = torch.fft.fftfreq(W, device=dev, dtype=torch.float64)
    g = torch.exp(-2.0 * (math.pi * PSF) ** 2 * (fy[:, None] ** 2 + fx[None, :] ** 2))
    z = torch.randn((2, H, W), generator=gen, device=dev, dtype=torch.float64)
    z = torch.fft.ifft2(torch.fft.fft2(z) * g).real
    env = torch.hypot(z[0], z[1])
    return env / env.mean()


def _spots(y, x, H, W, dev):
    """Sum of Gaussian spots at the centres (y, x)."""
    gy = torch.exp(-((torch.arange(H, device=dev, dtype=torch.float64)[:, None] - y) ** 2) / (2 * PSF**2))
    gx = torch.exp(-((torch.arange(W, device=dev, dtype=torch.float64)[:, None] - x) ** 2) / (2 * PSF**2))
    return AMPLITUDE * (gy @ gx.t().contiguous())


def _frames(H, W, n, seed, snr_db=20.0, parts=False, moving=2.0):
    """(n, H, W) float64 sequence; with `parts` also its noise-free bound part."""
    dev = torch.device("cuda")
    gen = torch.Generator(device=dev)
    gen.manual_seed(int(seed) & 0x7FFFFFFF)
    r = np.random.default_rng(int(seed) & 0x7FFFFFFF)
    nb, nf = max(1, H * W // 1300), max(1, int(moving * H * W / 1300))
    put = lambda a: torch.as_tensor(a, device=dev, dtype=torch.float64)  # noqa: E731
    by, bx = put(r.uniform(0, H, nb)), put(r.uniform(0, W, nb))
    fy, fx, ang, v = (r.uniform(0, H, nf), r.uniform(0, W, nf), r.uniform(0, 2 * math.pi, nf),
                      r.uniform(2.0, 6.0, nf))
    p1, p2 = r.uniform(0, 2 * math.pi, 2)
    t1, t2 = _speckle(gen, H, W, dev), _speckle(gen, H, W, dev)
    bound = _spots(by, bx, H, W, dev)
    out = torch.empty((n, H, W), device=dev, dtype=torch.float64)
    for t in range(n):
        a = 1.0 + DRIFT * math.sin(2 * math.pi * t / (4 * n) + p1)
        b = DRIFT * math.cos(2 * math.pi * t / (4 * n) + p2)
        y, x = put((fy + t * v * np.sin(ang)) % H), put((fx + t * v * np.cos(ang)) % W)
        out[t] = a * t1 + b * t2 + bound + _spots(y, x, H, W, dev)
    rms = torch.sqrt(torch.mean(out * out))
    for t in range(n):
        out[t] += rms * 10.0 ** (-snr_db / 20.0) * torch.randn((H, W), generator=gen, device=dev,
                                                               dtype=torch.float64)
    return (out, t1 + bound) if parts else out


def _type(case):
    return torch.float32 if case["dtype"] == "f32" else torch.float64


def _alm(X, tol, maxit, S0=None, Y0=None):
    """The iteration in plain 64-bit torch, on the (n, pixels) matrix X:
    (L, S, Y, iterations)."""
    n, m = X.shape
    mu = m * n / (4.0 * float(X.abs().sum()))
    lam = 1.0 / math.sqrt(max(m, n))
    S = torch.zeros_like(X) if S0 is None else S0
    Y = torch.zeros_like(X) if Y0 is None else Y0
    norm = float(torch.linalg.vector_norm(X))
    k = 0
    while True:
        k += 1
        A = X - S + Y / mu
        d, V = torch.linalg.eigh((A @ A.t()).cpu())
        s = d.clamp_min(0).sqrt()
        w = torch.where(s > 1.0 / mu, (s - 1.0 / mu) / s.clamp_min(1e-300), torch.zeros_like(s))
        L = ((V * w) @ V.t()).to(X.device) @ A
        T = X - L + Y / mu
        S = T - T.clamp(-lam / mu, lam / mu)
        Z = X - L - S
        Y = Y + mu * Z
        if k >= maxit or (tol > 0 and float(torch.linalg.vector_norm(Z)) < tol * norm):
            return L, S, Y, k


def _warm_inputs(case, seed):
    """A window of a sequence, and the S and Y that 40 iterations on the
    window before it left, shifted by the step."""
    H, W, n, s = case["H"], case["W"], case["n"], case["step"]
    seq = _frames(H, W, n + s, seed)
    _, S, Y, _ = _alm(seq[:n].reshape(n, H * W), 0.0, 40)
    X = seq[s:].to(_type(case)).contiguous()
    shifted = []
    for a in (S, Y):
        b = torch.zeros_like(a)
        b[: n - s] = a[s:]
        shifted.append(b.reshape(n, H, W).to(_type(case)).contiguous())
    return X, shifted[0], shifted[1]


def _process_inputs(case, seed):
    H, W, n = case["H"], case["W"], case["n"]
    seq, bound = _frames(H, W, n, seed, parts=True, moving=0.4)
    bad = np.random.default_rng(seed & 0x7FFFFFFF).choice(n, size=3, replace=False)
    gen = torch.Generator(device=seq.device)
    gen.manual_seed((seed + 1) & 0x7FFFFFFF)
    for t in bad:  # frames that jumped (motion): unrelated to their neighbours
        seq[int(t)] = 2.0 * _speckle(gen, H, W, seq.device)
    M = seq.to(_type(case)).contiguous()
    G = bound.to(_type(case)).expand(n, H, W).contiguous()
    mask = (G >= 2.5).to(torch.uint8).contiguous()
    return M, G, mask


def _seeds(case, seed):
    return [seed * 131 + 17 * i for i in range(case["count"])]


def prepare(case, seed) -> dict:
    """What a program has in hand before the call: windows in device memory
    (with the previous window's S and Y for a warm start), a server."""
    kind, st = case["kind"], {"case": case}
    if kind == "solve":
        st["M"] = _frames(case["H"], case["W"], case["n"], seed).to(_type(case)).contiguous()
    elif kind == "warm":
        st["M"], st["S0"], st["Y0"] = _warm_inputs(case, seed)
    elif kind in ("many", "serve"):
        st["Ms"] = [_frames(*s, q).to(_type(case)).contiguous()
                    for s, q in zip(_shapes(case), _seeds(case, seed))]
        if kind == "serve":
            st["server"] = rp.Server(dtype=rp.RPCA_F32, hbm_budget=64 << 30, max_active=64,
                                     quantum=case["quantum"])
    else:
        st["M"], st["G"], st["mask"] = _process_inputs(case, seed)
    return st


def run(st):
    """One pass through the public entry points."""
    case = st["case"]
    kind = case["kind"]
    if kind == "solve":
        r = rp.solve(st["M"], tol=case["tol"], maxit=case["maxit"], gram_mode=case["mode"])
        return {"L": r.L, "S": r.S, "iterations": r.iterations, "status": r.status}
    if kind == "warm":
        r = rp.solve(st["M"], tol=case["tol"], maxit=case["maxit"], S0=st["S0"], Y0=st["Y0"],
                     return_Y=True)
        return {"L": r.L, "S": r.S, "Y": r.Y, "iterations": r.iterations, "status": r.status}
    if kind == "many":
        rs = rp.solve_many(st["Ms"], tol=case["tol"], maxit=case["maxit"])
        return {"L": [r.L for r in rs], "S": [r.S for r in rs],
                "iterations": np.array([r.iterations for r in rs])}
    if kind == "serve":
        sv = st["server"]
        for i, M in enumerate(st["Ms"]):
            sv.submit(M, i, tol=case["tol"], maxit=case["maxit"])
        got = {}
        while len(got) < len(st["Ms"]):
            for c in sv.step():
                got[c.tag] = c
        done = [got[i] for i in range(len(st["Ms"]))]
        return {"L": [c.L for c in done], "S": [c.S for c in done],
                "iterations": np.array([c.iterations for c in done])}
    M, G = st["M"], st["G"]
    rho = postproc.frame_correlation(M)
    keep = postproc.frame_keep(rho)
    kept = postproc.frame_select(M, keep)
    avg = postproc.moving_average(kept, case["W_avg"])
    level = postproc.masked_mean(G, st["mask"])
    dice, counts = postproc.dice(M, 2.5, G, 2.5)
    return {"rho": rho, "keep": keep.astype(np.int64), "average": avg, "level": level, "dice": dice,
            "counts": np.array(counts), "rmse": postproc.rmse(M, G)}


def exact(case, seed):
    """run()'s outputs in 64 bits, from plain torch."""
    kind = case["kind"]

    def solved(M, S0=None, Y0=None):
        X = M.to(torch.float64).reshape(M.shape[0], -1)
        flat = lambda a: None if a is None else a.to(torch.float64).reshape(X.shape)  # noqa: E731
        L, S, Y, k = _alm(X, case["tol"], case["maxit"], flat(S0), flat(Y0))
        return L.reshape(M.shape), S.reshape(M.shape), Y.reshape(M.shape), k

    if kind == "solve":
        L, S, _, k = solved(_frames(case["H"], case["W"], case["n"], seed).to(_type(case)))
        return {"L": L, "S": S, "iterations": None, "status": None}
    if kind == "warm":
        L, S, Y, k = solved(*_warm_inputs(case, seed))
        return {"L": L, "S": S, "Y": Y, "iterations": None, "status": None}
    if kind in ("many", "serve"):
        rs = [solved(_frames(*s, q).to(_type(case)))[:2] for s, q in zip(_shapes(case), _seeds(case, seed))]
        return {"L": [r[0] for r in rs], "S": [r[1] for r in rs], "iterations": None}
    M, G, mask = _process_inputs(case, seed)
    n = M.shape[0]
    X = M.to(torch.float64).reshape(n, -1)
    C = X - X.mean(1, keepdim=True)
    v = (C * C).sum(1)
    rho = ((C[:-1] * C[1:]).sum(1) / (v[:-1] * v[1:]).sqrt()).cpu().numpy()
    best = np.maximum(np.concatenate([[-2.0], rho]), np.concatenate([rho, [-2.0]]))
    K = X[torch.as_tensor(best >= 0.8, device=X.device)]
    w = case["W_avg"]
    avg = torch.stack([K[t:t + w].mean(0) for t in range(K.shape[0] - w + 1)]).t()
    Gd = G.to(torch.float64)
    on = mask != 0
    a, b = M.to(torch.float64) >= 2.5, Gd >= 2.5
    both, ca, cb = int((a & b).sum()), int(a.sum()), int(b.sum())
    return {"rho": rho, "keep": None, "average": avg, "level": float(Gd[on].mean()),
            "dice": 2.0 * both / (ca + cb), "counts": None,
            "rmse": float(torch.sqrt(torch.mean((M.to(torch.float64) - Gd) ** 2)))}


def work(case) -> dict:
    """Inputs read once, outputs written once, and per iteration and entry the
    rebuild (2 n), the symmetric Gram (n + 1) and the elementwise step (12)."""
    kind, es = case["kind"], 4 if case["dtype"] == "f32" else 8
    if kind in ("solve", "warm", "many", "serve"):
        shapes = [(case["H"], case["W"], case["n"])] if kind in ("solve", "warm") else _shapes(case)
        words = 6 if kind == "warm" else 3
        return {"bytes": sum(words * es * h * w * n for h, w, n in shapes),
                "flops": sum(case["maxit"] * (h * w * n * (3.0 * n + 13.0) + 10.0 * n**3)
                             for h, w, n in shapes)}
    mn = case["H"] * case["W"] * case["n"]
    # correlation, selection (read, write), average (read, write), masked mean, Dice, RMSE
    return {"bytes": mn * (es * (1 + 2 + 2 + 1 + 2 + 2) + 1), "flops": 12.0 * mn}
