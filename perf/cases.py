"""Timed workloads of the deblurring library, through its Python entry points.

Each case is a dict of plain values; ``kind`` names the work:

* ``solve``      one blurred image to the deblurred image: transform, FISTA
                 iterations with float64 checks, synthesis;
* ``warm``       the same with the network's prediction as the first iterate and
                 the per-scale preconditioner;
* ``batch``      many images that share one or two operators in one call;
* ``dwt``        the wavelet transform of one image or of a stack of images;
* ``predict``    inference of the warm-start network on a batch;
* ``train``      two training steps of the network and its weights;
* ``exact``      the baseline that applies the blur itself in every iteration;
* ``calibrate``  a new PSF field: Theta_K, its norm, and the matrix on the host.

Operators, networks and their tuned layouts are what a program keeps from one
image to the next, so they are made once per process and setting; images,
noise and training batches come from the seed.
"""
import functools
import math
import types

import numpy as np
import torch

from paper_1512_08401_amd import wdb

DEV = "cuda:0"
HAAR = (0.7071067811865476, 0.7071067811865476)
DB4 = (0.2303778133088964, 0.7148465705529156, 0.6308807679298587, -0.0279837694168599,
       -0.1870348117190931, 0.0308413818355607, 0.0328830116668852, -0.0105974017850690)
TAPS = {"haar": HAAR, "db4": DB4}   # published tables; sym6 has no 64-bit reference here


# --------------------------------------------------------------------------
# cases
# --------------------------------------------------------------------------
def _solve(name, n, wavelet, levels, nnz, psf, a, b, lam, noise, iters, **kw):
    c = {"kind": "solve", "n": n, "wavelet": wavelet, "levels": levels, "nnz": nnz, "psf": psf, "a": a, "b": b,
         "lam": lam, "noise": noise, "iters": iters, "check_every": 20, "tol": 0.0, "graph": True, "values": "f32",
         "precond": "none", "rule": "naive", "l1": "uniform"}
    c.update(kw)
    if name:
        c["name"] = name
    return c


def listed():
    return [
        # the smallest problem, as an interactive preview or a test runs it: launches and latency decide
        _solve("solve 64", 64, "haar", 3, 40 * 64 * 64, "isotropic", 1.0, 3.0, 2e-3, 0.01, 200, graph=False),
        # the ordinary image: 30 entries per pixel, 500 iterations, checks recorded along the way
        _solve("solve 512", 512, "db4", 5, 30 * 512 * 512, "rotating", 4.0, 1.0, 1e-3, 0.01, 500),
        # the largest image, with the duality-gap stopping test read by the host at every check
        _solve("solve 1024", 1024, "db4", 6, 20 * 1024 * 1024, "rotating", 6.0, 1.0, 5e-4, 0.005, 400, tol=1e-4),
        # the same operator with 16-bit values, for a quick answer
        _solve("solve 1024 f16", 1024, "db4", 6, 20 * 1024 * 1024, "rotating", 6.0, 1.0, 5e-4, 0.005, 140,
               values="f16"),
        # the real-time path: transform, network, a few preconditioned iterations from its prediction, synthesis
        {"name": "warm 256", "kind": "warm", "n": 256, "wavelet": "db4", "levels": 4, "nnz": 30 * 256 * 256,
         "psf": "isotropic", "a": 1.0, "b": 3.0, "lam": 1e-3, "noise": 0.01, "iters": 60},
        # a video's or a training set's images, two cameras, a ragged count on each; every image stops by itself
        {"name": "batch 19+13", "kind": "batch", "n": 256, "count": 19, "n2": 512, "count2": 13, "wavelet": "db4",
         "px": 30, "lam": 1e-3, "noise": 0.01, "iters": 120, "tol": 2e-2},
        # one image to coefficients
        {"name": "dwt 512", "kind": "dwt", "n": 512, "wavelet": "db4", "levels": 5, "count": 1, "inverse": False},
        # a stack of solutions back to images
        {"name": "idwt 1024 x 21", "kind": "dwt", "n": 1024, "wavelet": "db4", "levels": 6, "count": 21,
         "inverse": True},
        # the network on one held-out chunk
        {"name": "predict 256 x 77", "kind": "predict", "n": 256, "wavelet": "db4", "levels": 4, "batch": 77},
        # training at the batch size the warm start is trained with
        {"name": "train 256 x 32", "kind": "train", "n": 256, "wavelet": "db4", "levels": 4, "batch": 32, "lr": 1e-3},
        # the baseline without Theta_K
        {"name": "exact 512", "kind": "exact", "n": 512, "wavelet": "db4", "levels": 5, "psf": "rotating", "a": 4.0,
         "b": 1.0, "lam": 1e-3, "noise": 0.01, "iters": 20},
        # a camera's new PSF field, offline
        {"name": "calibrate 256", "kind": "calibrate", "n": 256, "wavelet": "db4", "levels": 4, "nnz": 30 * 256 * 256,
         "psf": "rotating", "a": 3.0, "b": 1.0, "rule": "naive"},
    ]


def _log_uniform(rng, lo, hi):
    return math.exp(rng.uniform(math.log(lo), math.log(hi)))


def _psf(rng, n):
    """A PSF family of the workloads whose support fits the image."""
    top = min(5.0, (n - 1) / 6.5)
    if rng.random() < 0.5:
        return "isotropic", round(rng.uniform(1.0, top), 2), round(rng.uniform(1.0, top), 2)
    minor = round(rng.uniform(1.0, 2.0), 2)
    return "rotating", round(rng.uniform(minor, top), 2), minor


def draw(rng):
    kind = rng.choice(["solve", "solve", "warm", "batch", "dwt", "dwt", "predict", "train", "exact", "calibrate"])
    wavelet = rng.choice(["haar", "db4", "db4", "sym6"])
    if kind == "solve":
        n = rng.choice([64, 128, 256, 512])
        psf, a, b = _psf(rng, n)
        values = rng.choice(["f32", "f32", "f16", "bf16"])
        return _solve(None, n, wavelet, rng.choice([2, int(math.log2(n)) - 4]),
                      int(_log_uniform(rng, 8, 40) * n * n) + rng.randrange(64), psf, a, b,
                      _log_uniform(rng, 1e-4, 1e-2), rng.choice([0.005, 0.01]), int(_log_uniform(rng, 20, 300)),
                      check_every=rng.choice([10, 20, 50]), tol=rng.choice([0.0, 1e-4]),
                      graph=rng.random() < 0.5, values=values,
                      precond=rng.choice(["none", "none", "spai", "spai_scale", "jacobi"]),
                      rule=rng.choice(["naive", "scale"]), l1=rng.choice(["uniform", "uniform", "scale"]))
    if kind == "warm":
        n = rng.choice([64, 128, 256])
        psf, a, b = _psf(rng, n)
        return {"kind": kind, "n": n, "wavelet": wavelet, "levels": int(math.log2(n)) - 4,
                "nnz": int(_log_uniform(rng, 10, 40) * n * n), "psf": psf, "a": a, "b": b,
                "lam": _log_uniform(rng, 1e-4, 1e-2), "noise": 0.01, "iters": int(_log_uniform(rng, 10, 100))}
    if kind == "batch":
        n, n2 = rng.choice([64, 128, 256]), rng.choice([0, 64, 128, 256])
        return {"kind": kind, "n": n, "count": rng.randint(1, 20), "n2": n2,
                "count2": rng.randint(1, 12) if n2 else 0, "wavelet": wavelet, "px": rng.randint(20, 40),
                "lam": _log_uniform(rng, 1e-4, 1e-2), "noise": 0.01, "iters": 120, "tol": 2e-2}
    if kind == "dwt":
        n = rng.choice([32, 64, 128, 256, 512, 1024, 2048])
        most = max(1, 20 * 1024 * 1024 // (n * n))
        return {"kind": kind, "n": n, "wavelet": wavelet, "levels": rng.randint(1, int(math.log2(n)) - 3),
                "count": int(_log_uniform(rng, 1, min(most, 60) + 0.99)), "inverse": rng.random() < 0.5}
    if kind in ("predict", "train"):
        n = rng.choice([32, 64, 128, 256])
        most = min(64, (32 if kind == "train" else 77) * 256 * 256 // (n * n))
        c = {"kind": kind, "n": n, "wavelet": rng.choice(["haar", "db4"]),
             "levels": rng.randint(1, int(math.log2(n)) - 3), "batch": int(_log_uniform(rng, 1, most + 0.99))}
        if kind == "train":
            c["lr"] = 1e-3
        return c
    if kind == "exact":
        n = rng.choice([64, 128, 256])
        psf, a, b = _psf(rng, n)
        return {"kind": kind, "n": n, "wavelet": wavelet, "levels": int(math.log2(n)) - 4, "psf": psf, "a": a, "b": b,
                "lam": _log_uniform(rng, 1e-4, 1e-2), "noise": 0.01, "iters": rng.randint(5, 40)}
    n = rng.choice([64, 128, 256])
    psf, a, b = _psf(rng, n)
    return {"kind": kind, "n": n, "wavelet": wavelet, "levels": int(math.log2(n)) - 4,
            "nnz": int(rng.uniform(10, 30) * n * n), "psf": psf, "a": a, "b": b,
            "rule": rng.choice(["naive", "scale"])}


# --------------------------------------------------------------------------
# inputs, in plain torch (float64 on the GPU)
# --------------------------------------------------------------------------
def _field(n, psf, a, b, wobble=0.0, phase=0.0):
    """PSF parameters per source pixel; `wobble` perturbs them smoothly (a measured field)."""
    col = np.arange(n)[None, :] / n
    row = np.arange(n)[:, None] / n
    bend = 1.0 + wobble * np.sin(2 * math.pi * (row + 2 * col) + phase)
    if psf == "isotropic":
        major = minor = (a + (b - a) * col) * bend
        angle = np.zeros((n, n))
    else:
        major, minor = np.full((n, n), a) * bend, np.full((n, n), b) * bend
        angle = math.pi * col + 0.2 * wobble * row
    full = [np.array(np.broadcast_to(v, (n, n)), dtype=np.float64) for v in (major, minor, angle)]
    return types.SimpleNamespace(n=n, sig_major=full[0], sig_minor=full[1], angle=full[2], trunc=3.0)


def _calibration_field(c, seed):
    r = np.random.default_rng(seed)
    return _field(c["n"], c["psf"], c["a"] * (1 - 0.04 * r.random()), c["b"], 0.02, 6.28 * r.random())


def _offsets(f):
    """(dy, dx, weight at every source pixel) of the truncated, normalised PSFs."""
    M, m, t = (torch.as_tensor(v, device=DEV) for v in (f.sig_major, f.sig_minor, f.angle))
    c, s = torch.cos(t), torch.sin(t)
    R = int(math.floor(f.trunc * max(f.sig_major.max(), f.sig_minor.max())))

    def weight(dy, dx):
        p, q = (c * dx + s * dy) / M, (c * dy - s * dx) / m
        d = p * p + q * q
        return torch.where(d <= f.trunc ** 2, torch.exp(-0.5 * d), torch.zeros_like(d))

    near = [(dy, dx) for dy in range(-R, R + 1) for dx in range(-R, R + 1) if dy * dy + dx * dx <= (R + 1) ** 2]
    Z = torch.zeros_like(M)
    for dy, dx in near:
        Z += weight(dy, dx)
    for dy, dx in near:
        yield dy, dx, weight(dy, dx) / Z


@functools.lru_cache(maxsize=4)
def _blur_entries(n, psf, a, b):
    """The blur matrix as (row, column, value) for images that are blurred often."""
    idx = torch.arange(n * n, device=DEV).view(n, n)
    rows, cols, vals = [], [], []
    for dy, dx, w in _offsets(_field(n, psf, a, b)):
        at = w.reshape(-1).nonzero().view(-1)
        cols.append(at.to(torch.int32))
        rows.append(torch.roll(idx, (-dy, -dx), (0, 1)).reshape(-1)[at].to(torch.int32))
        vals.append(w.reshape(-1)[at])
    return torch.cat(rows).long(), torch.cat(cols).long(), torch.cat(vals)


def _spread(entries, x, adjoint=False):
    r, c, v = entries
    if adjoint:
        r, c = c, r
    return torch.zeros_like(x).index_add_(0, r, v * x[c])


def _images(n, count, seed):
    """Piecewise smooth images in [0, 1]: a ramp with eight painted disks and boxes each."""
    r = np.random.default_rng(seed)
    y, x = torch.meshgrid(torch.arange(n, device=DEV, dtype=torch.float64) / n,
                          torch.arange(n, device=DEV, dtype=torch.float64) / n, indexing="ij")
    out = []
    for _ in range(count):
        img = r.uniform(0, 0.5) + r.uniform(-0.25, 0.25) * x + r.uniform(-0.25, 0.25) * y
        for _ in range(8):
            p = r.uniform(0, 1, 4)
            if r.random() < 0.5:
                inside = (y - p[0]) ** 2 + (x - p[1]) ** 2 <= (1 / 16 + p[2] * 3 / 16) ** 2
            else:
                inside = (y >= min(p[0], p[1])) & (y <= max(p[0], p[1])) & (x >= min(p[2], p[3])) & (x <= max(p[2], p[3]))
            img = torch.where(inside, torch.full_like(img, r.uniform(0, 1)), img)
        out.append(img.clamp(0, 1))
    return torch.stack(out)


def _noise(shape, sigma, seed):
    g = torch.Generator(device=DEV)
    g.manual_seed(seed)
    return sigma * torch.randn(shape, generator=g, device=DEV, dtype=torch.float64)


def _observed(n, psf, a, b, noise, seed, count=1):
    """Blurred, noisy float32 images (count, n * n)."""
    entries = _blur_entries(n, psf, a, b)
    sharp = _images(n, count, seed).view(count, -1)
    return torch.stack([_spread(entries, s) for s in sharp]).add_(_noise(sharp.shape, noise, seed)).float()


def _high(h):
    return [(-1) ** m * v for m, v in enumerate(reversed(h))]


def _down(x, f, dim):
    """out[i] = sum_m f[m] x[2 i + m], periodic, along dim."""
    out = 0
    for m, v in enumerate(f):
        s = torch.roll(x, -m, dim)
        out = out + v * (s[..., ::2] if dim in (-1, x.dim() - 1) else s[..., ::2, :])
    return out


def _up(c, f, dim):
    shape = list(c.shape)
    shape[dim] *= 2
    z = torch.zeros(shape, device=c.device, dtype=c.dtype)
    if dim == -1:
        z[..., ::2] = c
    else:
        z[..., ::2, :] = c
    out = 0
    for m, v in enumerate(f):
        out = out + v * torch.roll(z, m, dim)
    return out


def _dwt64(u, h, levels):
    """(count, n, n) float64 images to (count, n * n) coefficients, coarse to fine."""
    g, parts = _high(h), []
    for _ in range(levels):
        lo, hi = _down(u, h, -1), _down(u, g, -1)
        parts = [_down(hi, h, -2), _down(lo, g, -2), _down(hi, g, -2)] + parts
        u = _down(lo, h, -2)
    return torch.cat([p.reshape(p.shape[0], -1) for p in [u] + parts], 1)


def _idwt64(x, h, levels):
    count, n = x.shape[0], int(round(math.sqrt(x.shape[1])))
    g, s = _high(h), n >> levels
    u = x[:, :s * s].reshape(count, s, s)
    while s < n:
        d01, d10, d11 = (x[:, k * s * s:(k + 1) * s * s].reshape(count, s, s) for k in (1, 2, 3))
        u = _up(_up(u, h, -2) + _up(d10, g, -2), h, -1) + _up(_up(d01, h, -2) + _up(d11, g, -2), g, -1)
        s *= 2
    return u


@functools.lru_cache(maxsize=8)
def _small_theta(n, wavelet, levels, nnz, psf, a, b):
    """Theta_K of a small image computed here (dense, float64), as host CSR arrays."""
    T = _dense_theta(_blur_entries(n, psf, a, b), n, wavelet, levels)
    return _largest(T, nnz)


def _dense_theta(entries, n, wavelet, levels):
    N, (r, c, v) = n * n, entries
    H = torch.zeros(N, N, device=DEV, dtype=torch.float64)
    H.index_put_((r, c), v, accumulate=True)
    h = TAPS[wavelet]
    W = _dwt64(torch.eye(N, device=DEV, dtype=torch.float64).view(N, n, n), h, levels)   # row i: transform of pixel i
    return W.t().contiguous() @ H @ W


def _largest(T, nnz):
    """The nnz largest entries (zeros never kept) as CSR, ties to the smaller index."""
    N = T.shape[0]
    mag, at = T.abs().reshape(-1).sort(descending=True, stable=True)
    at = at[:min(nnz, int((mag > 0).sum()))].sort().values
    rp = torch.zeros(N + 1, dtype=torch.int64, device=DEV)
    rp[1:] = torch.bincount(at // N, minlength=N).cumsum(0)
    return rp.cpu().numpy(), (at % N).int().cpu().numpy(), T.reshape(-1)[at].cpu().numpy()


# --------------------------------------------------------------------------
# what a program keeps
# --------------------------------------------------------------------------
@functools.lru_cache(maxsize=10)
def _operator(n, wavelet, levels, nnz, psf, a, b, rule="naive", values="f32", precond="none", l1="uniform"):
    if n <= 64 and rule == "naive" and wavelet in TAPS:   # a matrix that was computed elsewhere
        th = wdb.Theta.from_csr(n, wavelet, levels, *_small_theta(n, wavelet, levels, nnz, psf, a, b))
    else:
        th = wdb.build_theta(_field(n, psf, a, b), wavelet, levels, nnz, rule=rule)
    th.lipschitz_lanczos()
    if precond != "none":
        th.set_precond(precond, eps=1e-6 if precond == "jacobi" else 0.0, max_iters=2000)
    if l1 != "uniform":
        th.set_l1_weights(l1)
    th.set_precision(values)
    th.autotune(reps=10)
    return th


def _solve_operator(c):
    return _operator(c["n"], c["wavelet"], c["levels"], c["nnz"], c["psf"], c["a"], c["b"], c.get("rule", "naive"),
                     c.get("values", "f32"), c.get("precond", "none"), c.get("l1", "uniform"))


def _stacks(n, levels):
    """(offset, channels, side) of the network's stacks, coarse to fine."""
    s = n >> levels
    return [(0, 1, s)] + [((n >> lev) ** 2, 3, n >> lev) for lev in range(levels, 0, -1)]


@functools.lru_cache(maxsize=4)
def _weights(n, levels):
    """Parameters of a network after some training, He-normal with small biases, stack by stack."""
    r, parts = np.random.default_rng(7), []
    for _, C, _ in _stacks(n, levels):
        for shape, fan, s in (((32, C, 3, 3), 9 * C, 1.0), ((32, 32, 3, 3), 288, 1.0), ((C, 32, 3, 3), 288, 0.1)):
            parts += [r.normal(0, s * math.sqrt(2 / fan), shape).ravel(), r.normal(0, 0.01, shape[0])]
    return np.concatenate(parts).astype(np.float32)


@functools.lru_cache(maxsize=4)
def _network(n, levels):
    net = wdb.Cnn(n, levels)
    net.set_params(_weights(n, levels))
    return net


def _pairs(c, seed, batch):
    """(coefficients of blurred noisy images, of the sharp images) for the network."""
    n, h = c["n"], TAPS[c["wavelet"]]
    sharp = _images(n, batch, seed)
    k = torch.exp(-0.5 * (torch.arange(-5, 6, device=DEV, dtype=torch.float64) / 1.5) ** 2)
    k, soft = (k / k.sum()).tolist(), sharp
    for dim in (-1, -2):
        soft = sum(w * torch.roll(soft, j - 5, dim) for j, w in enumerate(k))
    return (_dwt64(soft + _noise(soft.shape, 0.01, seed), h, c["levels"]).float(),
            _dwt64(sharp, h, c["levels"]).float())


def prepare(case, seed):
    c, kind, n = case, case["kind"], case["n"]
    s = {"kind": kind, "case": c}
    if kind in ("solve", "warm"):
        s["theta"] = _solve_operator(dict(c, precond="spai_scale") if kind == "warm" else c)
        s["u"] = _observed(n, c["psf"], c["a"], c["b"], c["noise"], seed)[0]
        if kind == "warm":
            s["net"] = _network(n, c["levels"])
    elif kind == "batch":
        s["problems"] = []
        for k, (side, count, psf) in enumerate(((n, c["count"], ("isotropic", 1.0, 3.0)),
                                                (c["n2"], c["count2"], ("rotating", 4.0, 1.0)))):
            if count:
                th = _operator(side, c["wavelet"], int(math.log2(side)) - 4, c["px"] * side * side, *psf)
                lam = c["lam"] * np.exp(np.random.default_rng(seed + k).uniform(-1, 1, count))
                s["problems"] += [(th, u, float(v)) for u, v in
                                  zip(_observed(side, *psf, c["noise"], seed + k, count), lam)]
    elif kind == "dwt":
        u = _images(n, c["count"], seed) + _noise((c["count"], n, n), 0.01, seed)
        if c["inverse"]:
            u = _dwt64(u, TAPS.get(c["wavelet"], DB4), c["levels"])
        s["in"] = u.reshape(c["count"], -1).float()
    elif kind in ("predict", "train"):
        if kind == "predict":
            s["net"], s["x0"] = _network(n, c["levels"]), _pairs(c, seed, c["batch"])[0]
        else:   # the training run's own network and two of its batches
            s["net"] = wdb.Cnn(n, c["levels"])
            s["net"].set_params(_weights(n, c["levels"]))
            s["batches"] = [_pairs(c, seed + k, c["batch"]) for k in (0, 1)]
    elif kind == "exact":
        s["exact"] = _exact_handle(n, c["wavelet"], c["levels"], c["psf"], c["a"], c["b"])
        s["u"] = _observed(n, c["psf"], c["a"], c["b"], c["noise"], seed)[0]
    else:
        s["field"] = _calibration_field(c, seed)
    return s


@functools.lru_cache(maxsize=4)
def _exact_handle(n, wavelet, levels, psf, a, b):
    ex = wdb.Exact(_field(n, psf, a, b), wavelet, levels)
    ex.lipschitz()
    return ex


def run(state):
    c, kind = state["case"], state["kind"]
    if kind == "solve":
        th = state["theta"]
        x, info = th.solve(state["u"], c["lam"], c["iters"], check_every=c["check_every"], tol=c["tol"],
                           precond=c["precond"] != "none", use_graph=c["graph"])
        return {"x": x, "image": th.synthesize(x), "objective": info["objective"], "iters": info["iters"]}
    if kind == "warm":
        th = state["theta"]
        x0 = wdb.dwt(state["u"], c["wavelet"], c["levels"])
        x, info = th.solve_coeffs(x0, c["lam"], c["iters"], x_init=state["net"].predict(x0), precond=True,
                                  use_graph=True)
        return {"x": x, "image": th.synthesize(x), "objective": info["objective"]}
    if kind == "batch":
        xs, infos = wdb.solve_batched(state["problems"], c["iters"], check_every=20, tol=c["tol"], use_graph=True)
        return {"x": xs, "objective": np.array([i["objective"] for i in infos], dtype=np.float32),
                "iters": np.array([i["iters"] for i in infos])}
    if kind == "dwt":
        if c["count"] == 1:
            return wdb.dwt(state["in"][0], c["wavelet"], c["levels"], inverse=c["inverse"])
        return wdb.dwt_batched(state["in"], c["wavelet"], c["levels"], inverse=c["inverse"])
    if kind == "predict":
        return state["net"].predict(state["x0"])
    if kind == "train":
        net = state["net"]
        losses = [net.train_step(x0, t, c["lr"]) for x0, t in state["batches"]]
        return {"loss": losses, "weights": net.get_params()}
    if kind == "exact":
        x, info = state["exact"].solve(state["u"], c["lam"], c["iters"])
        return {"x": x, "objective": info["objective"]}
    th = wdb.build_theta(state["field"], c["wavelet"], c["levels"], c["nnz"], rule=c["rule"])
    L = th.lipschitz_lanczos()["L"]
    rowptr, col, val = th.export()
    return {"rowptr": rowptr, "col": col, "val": val, "L": L}


# --------------------------------------------------------------------------
# what a pass cannot do without
# --------------------------------------------------------------------------
def _conv_flops(n, levels, batch):
    return sum(2 * 9 * (C * 32 + 32 * 32 + 32 * C) * s * s for _, C, s in _stacks(n, levels)) * batch


def work(case):
    c, kind, n = case, case["kind"], case["n"]
    N = n * n
    if kind in ("solve", "warm"):
        # per iteration both products read every kept value once (an operator that is used between passes
        # cannot stay on the chip) and the vectors of the update once
        size = 4 if c.get("values", "f32") == "f32" else 2
        return {"bytes": c["iters"] * (2 * size * c["nnz"] + 28 * N) + 12 * N, "flops": c["iters"] * 4 * c["nnz"]}
    if kind == "batch":
        sides = [(n, c["count"]), (c["n2"], c["count2"])]
        return {"bytes": c["iters"] * sum(8 * c["px"] * s * s * -(-k // 8) + 28 * s * s * k for s, k in sides),
                "flops": c["iters"] * sum(4 * c["px"] * s * s * k for s, k in sides)}
    if kind == "dwt":
        taps = {"haar": 2, "db4": 8, "sym6": 12}[c["wavelet"]]
        return {"bytes": 8 * N * c["count"], "flops": 4 * taps * N * c["count"] * (1 - 0.25 ** c["levels"]) / 0.75}
    if kind == "predict":
        return {"bytes": 8 * N * c["batch"], "flops": _conv_flops(n, c["levels"], c["batch"])}
    if kind == "train":
        return {"bytes": 2 * 8 * N * c["batch"], "flops": 2 * 3 * _conv_flops(n, c["levels"], c["batch"])}
    if kind == "exact":
        per = math.pi * 9 * (((c["a"] + c["b"]) / 2) ** 2 if c["psf"] == "isotropic" else c["a"] * c["b"])
        return {"bytes": c["iters"] * 40 * N, "flops": (c["iters"] + 1) * 2 * 2 * per * N}
    per = math.pi * 9 * (((c["a"] + c["b"]) / 2) ** 2 if c["psf"] == "isotropic" else c["a"] * c["b"])
    return {"bytes": 20 * c["nnz"] + 24 * N, "flops": 2 * per * N * sum(4 ** lev for lev in range(1, c["levels"] + 1))}


# --------------------------------------------------------------------------
# the same in 64 bits
# --------------------------------------------------------------------------
def _largest_eigenvalue(mul, N):
    """lambda_max of a symmetric operator by Lanczos with full orthogonalisation, to 1e-13 of itself."""
    v = _noise((N,), 1.0, 5)
    V, alpha, beta = [v / v.norm()], [], []
    for k in range(min(N, 700)):
        u = mul(V[-1])
        alpha.append(float(u @ V[-1]))
        B = torch.stack(V)
        for _ in range(2):
            u = u - B.t() @ (B @ u)
        beta.append(float(u.norm()))
        if k % 20 == 19 or beta[-1] < 1e-14:
            T = np.diag(alpha) + np.diag(beta[:-1], 1) + np.diag(beta[:-1], -1)
            w, q = np.linalg.eigh(T)
            if beta[-1] * abs(q[-1, -1]) <= 1e-13 * w[-1]:
                return float(w[-1])
        V.append(u / beta[-1])
    return None


def _fista(forward, backward, x0, lam, L, iters):
    lam, x = float(np.float32(lam)), torch.zeros_like(x0)
    y = x
    for k in range(1, iters + 1):
        z = y - backward(forward(y) - x0) / L
        new = z.sign() * (z.abs() - lam / L).clamp_min(0)
        y, x = new + (k - 1) / (k + 2) * (new - x), new
    return x


def _net64(c, x0, params):
    """The network in float64 with bfloat16-rounded parameters (given as float64 tensors)."""
    out, at = [], 0
    for off, C, s in _stacks(c["n"], c["levels"]):
        z = x0[:, off:off + C * s * s].reshape(-1, C, s, s)
        h = z
        for layer, (o, i) in enumerate(((32, C), (32, 32), (C, 32))):
            w = params[at:at + o * i * 9].view(o, i, 9)
            b = params[at + o * i * 9:at + o * i * 9 + o]
            at += o * i * 9 + o
            acc = b
            hp = h.permute(0, 2, 3, 1)
            for d in range(9):
                acc = acc + torch.roll(hp, (1 - d // 3, 1 - d % 3), (1, 2)).reshape(-1, i) @ w[:, :, d].t().contiguous()
            h = acc.view(-1, s, s, o).permute(0, 3, 1, 2)
            h = h.relu() if layer < 2 else h
        out.append((z + h).reshape(x0.shape[0], -1))
    return torch.cat(out, 1)


def exact(case, seed):
    c, kind, n = case, case["kind"], case["n"]
    h = TAPS.get(c["wavelet"])
    if h is None:
        return None
    if kind == "solve":
        if n > 64 or c["rule"] != "naive" or c["values"] != "f32" or c["precond"] != "none" or c["l1"] != "uniform":
            return None   # Theta_K of a large image takes too long here
        rp, col, val = _small_theta(n, c["wavelet"], c["levels"], c["nnz"], c["psf"], c["a"], c["b"])
        N = n * n
        A = torch.zeros(N, N, device=DEV, dtype=torch.float64)
        A[torch.as_tensor(np.repeat(np.arange(N), np.diff(rp)), device=DEV),
          torch.as_tensor(col, device=DEV).long()] = torch.as_tensor(val.astype(np.float32), device=DEV).double()
        At = A.t().contiguous()
        L = _largest_eigenvalue(lambda v: At @ (A @ v), N)
        u = _observed(n, c["psf"], c["a"], c["b"], c["noise"], seed)[0]
        x0 = _dwt64(u.double().view(1, n, n), h, c["levels"])[0]
        if c["tol"] > 0 or L is None:
            return None   # the stopping test decides where it ends
        x = _fista(lambda v: A @ v, lambda r: At @ r, x0, c["lam"], L, c["iters"])
        E = 0.5 * float((A @ x - x0).square().sum()) + float(np.float32(c["lam"])) * float(x.abs().sum())
        return {"x": x, "image": _idwt64(x.view(1, -1), h, c["levels"])[0], "objective": E, "iters": None}
    if kind == "dwt":
        x = prepare(case, seed)["in"].double()
        y = _idwt64(x, h, c["levels"]).reshape(c["count"], -1) if c["inverse"] else \
            _dwt64(x.view(-1, n, n), h, c["levels"])
        return y[0] if c["count"] == 1 else y
    if kind == "predict":
        p = torch.as_tensor(_weights(n, c["levels"]), device=DEV).bfloat16().double()
        return torch.cat([_net64(c, x, p) for x in _pairs(c, seed, c["batch"])[0].double().split(16)])
    if kind == "train":
        master = torch.as_tensor(_weights(n, c["levels"]), device=DEV).double()
        m, v, losses = torch.zeros_like(master), torch.zeros_like(master), []
        for k in (0, 1):
            x0, t = (q.double() for q in _pairs(c, seed + k, c["batch"]))
            p = master.float().bfloat16().double().requires_grad_(True)
            loss = (_net64(c, x0, p) - t).square().mean()
            (g,) = torch.autograd.grad(loss, p)
            losses.append(float(loss.detach()))
            m, v = 0.9 * m + 0.1 * g, 0.999 * v + 0.001 * g * g
            master = master - c["lr"] * (m / (1 - 0.9 ** (k + 1))) / ((v / (1 - 0.999 ** (k + 1))).sqrt() + 1e-8)
        return {"loss": losses, "weights": master}
    if kind == "exact":
        entries = _blur_entries(n, c["psf"], c["a"], c["b"])
        L = _largest_eigenvalue(lambda x: _spread(entries, _spread(entries, x), True), n * n)
        if L is None:
            return None
        u0 = _observed(n, c["psf"], c["a"], c["b"], c["noise"], seed)[0].double()

        def blur(x):
            return _spread(entries, _idwt64(x.view(1, -1), h, c["levels"]).reshape(-1))

        def back(r):
            return _dwt64(_spread(entries, r, True).view(1, n, n), h, c["levels"])[0]

        x = _fista_image(blur, back, u0, c["lam"], L, c["iters"])
        E = 0.5 * float((blur(x) - u0).square().sum()) + float(np.float32(c["lam"])) * float(x.abs().sum())
        return {"x": x, "objective": E}
    if kind == "calibrate" and n <= 64:
        f = _calibration_field(c, seed)
        idx = torch.arange(n * n, device=DEV).view(n, n)
        H = [torch.roll(idx, (-dy, -dx), (0, 1)).reshape(-1) for dy, dx, _ in _offsets(f)]
        W = [w.reshape(-1) for _, _, w in _offsets(f)]
        T = _dense_theta((torch.cat(H), idx.reshape(-1).repeat(len(H)), torch.cat(W)), n, c["wavelet"], c["levels"])
        if c["rule"] == "naive":
            return {"rowptr": None, "col": None, "val": _largest(T, c["nnz"])[2], "L": None}
    return None


def _fista_image(blur, back, u0, lam, L, iters):
    x0 = torch.zeros_like(u0)
    lam, x, y = float(np.float32(lam)), x0, x0
    for k in range(1, iters + 1):
        z = y - back(blur(y) - u0) / L
        new = z.sign() * (z.abs() - lam / L).clamp_min(0)
        y, x = new + (k - 1) / (k + 2) * (new - x), new
    return x
