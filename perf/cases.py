"""Timed cases of the library's main paths, each one pass through the public entry points.

A case is a dict of plain values; ``listed()`` names the fixed ones, ``draw(rng)`` gives more of the
same ranges, ``prepare(case, seed)`` makes a program's inputs and handles on the GPU, ``run(state)`` is one
pass, ``work(case)`` the bytes and operations the pass cannot do without and ``exact(case, seed)`` its
result in 64 bits from plain torch.

Kinds:
  eig     standard synthesis of given eigenpairs, one instance (``collect_eig``)
  batch   the same for packed instances of one size that the program keeps (``collect_eig_batched``)
  uneven  packing and synthesis of instances of many sizes into several channels
  step    one full step from visibilities (Gram matrix, eigenproblem, levels, synthesis)
  grad    forward and backward of the differentiable image
  nufft   packing, NUFFT spread and transform
  weight  uniform weighting of visibilities and k-means energy levels
"""

import math

import numpy as np
import torch

import paper_2310_09200_amd as bb

DEV = "cuda"
LAT = math.radians(52.9)
INF = float("inf")
_CTX = []


def listed():
    return [
        # A small array and image (64 antennas, 128 x 128 pixels): the latency of one call, as in an
        # interactive look at one snapshot or a loop over snapshots that is not batched.
        dict(name="eig_64", kind="eig", n_ant=64, n_eig=64, side=128, levels=5, precision="fp32"),
        # The whole step of the same array from its visibilities, the first thing a user runs.
        dict(name="step_64", kind="step", n_ant=64, n_eig=64, side=128, levels=5, precision="fp32"),
        # One epoch of a 512-station array from visibilities to a 1024 x 1024 image, epoch by epoch.
        dict(name="step_512", kind="step", n_ant=512, n_eig=512, side=1024, levels=9, precision="fp32_3m"),
        # The main load: epochs of a 512-station array, all eigenpairs, 1024 x 1024 pixels, 8 + 1 levels.
        dict(name="batch_512", kind="batch", n_inst=16, n_ant=512, n_eig=512, side=1024, levels=9,
             precision="fp32_3m"),
        # A deep wide field: 2048 x 2048 pixels, baselines to 65 km, default precision, one epoch.
        dict(name="field_2048", kind="eig", n_ant=512, n_eig=512, side=2048, levels=9, precision="fp32"),
        # The compensated 16-bit form on sizes that are no multiple of anything: flagged stations, truncated
        # eigenpairs, an image side that is not a power of two.
        dict(name="ragged_bf16x3", kind="batch", n_inst=12, n_ant=389, n_eig=203, side=810, levels=4,
             precision="bf16x3"),
        # Channels x epochs of a flagged array in one call: 200 to 512 stations, 16 to 128 eigenpairs each.
        dict(name="uneven", kind="uneven", n_chan=16, n_step=8, l_lo=200, l_hi=512, k_lo=16, k_hi=128, side=512,
             levels=4, precision="fp32_3m"),
        # Differentiation: images and the gradients of a loss on them, 256 antennas, 64 eigenpairs.
        dict(name="grad_64", kind="grad", n_ant=256, n_eig=64, side=512, levels=4, precision="fp32"),
        # The same past 64 eigenpairs, with sizes off every tile.
        dict(name="grad_128", kind="grad", n_ant=250, n_eig=121, side=500, levels=4, precision="fp32"),
        # NUFFT synthesis of a 512-station array: 50 epochs over 6 h, 1024 x 1024 pixels of 4 arcsec.
        dict(name="nufft_1024", kind="nufft", n_inst=50, n_ant=512, n_eig=512, side=1024, levels=9, eps=1e-5),
        # NUFFT synthesis of a small array and image, where launches count.
        dict(name="nufft_128", kind="nufft", n_inst=1, n_ant=64, n_eig=64, side=128, levels=5, eps=1e-5),
        # What comes before a step: weighting one epoch's visibilities, levels from its eigenvalues.
        dict(name="weight_512", kind="weight", n_ant=512, n_eig=512, levels=9),
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    prec = rng.choice(["fp32", "fp32_3m", "fp32_3m", "bf16x3", "bf16x3_3m"])
    levels = rng.randint(1, 12)
    kind = rng.choice(["eig", "eig", "batch", "batch", "uneven", "step", "grad", "grad", "nufft", "weight"])
    if kind == "weight":
        return dict(kind=kind, n_ant=_log(rng, 24, 1024), n_eig=_log(rng, 24, 1024), levels=rng.randint(2, 12))
    if kind == "nufft":
        n = _log(rng, 32, 512)
        return dict(kind=kind, n_inst=_log(rng, 1, 24), n_ant=n, n_eig=_log(rng, 16, n), side=_log(rng, 100, 1024),
                    levels=levels, eps=rng.choice([1e-3, 1e-4, 1e-5, 1e-6]))
    if kind == "grad":
        n = _log(rng, 24, 512)
        return dict(kind=kind, n_ant=n, n_eig=_log(rng, 8, min(n, 256)), side=_log(rng, 64, 640), levels=levels,
                    precision=prec)
    if kind == "step":
        n = _log(rng, 24, 512)
        return dict(kind=kind, n_ant=n, n_eig=rng.randint(max(1, n // 4), n), side=_log(rng, 64, 1024), levels=levels,
                    precision=prec)
    if kind == "uneven":
        l_lo = _log(rng, 32, 400)
        k_hi = _log(rng, 16, min(l_lo, 224))
        return dict(kind=kind, n_chan=rng.randint(1, 16), n_step=rng.randint(1, 8), l_lo=l_lo,
                    l_hi=min(512, l_lo + rng.randint(0, 300)), k_lo=rng.randint(4, k_hi), k_hi=k_hi,
                    side=_log(rng, 100, 512), levels=levels, precision=prec)
    while True:
        n = _log(rng, 16, 1024)
        c = dict(kind=kind, n_ant=n, n_eig=_log(rng, 8, n), side=_log(rng, 48, 2048), levels=levels, precision=prec)
        if kind == "batch":
            c["n_inst"] = rng.randint(2, 24)
        if c.get("n_inst", 1) * c["n_ant"] * c["n_eig"] * c["side"] ** 2 <= 4.4e12:
            return c


# -- synthetic observations: geometry, eigenpairs, visibilities ------------------------------------------------


def _gen(case, seed):
    return np.random.default_rng([int(seed), 7919])


def _basis():
    """Image frame at declination 50 degrees: e_u, e_v and the phase centre."""
    d = math.radians(50.0)
    return np.array([[0.0, 1.0, 0.0], [-math.sin(d), 0.0, math.cos(d)], [math.cos(d), 0.0, math.sin(d)]])


def _array(n, g):
    """Stations in metres, Earth-fixed: a disk of 2 km up to 256, else a core and arms out to 32.5 km."""
    n_core = n if n <= 256 else n * 7 // 16
    r = (1000.0 if n <= 256 else 500.0) * np.sqrt(g.random(n_core))
    th = 2 * np.pi * g.random(n_core)
    m = n - n_core
    if m:
        t = g.random(m)
        r = np.concatenate([r, 600.0 * np.exp(t * math.log(32500.0 / 600.0))])
        th = np.concatenate([th, 2.5 * np.pi * t + 2 * np.pi / 3 * g.integers(0, 3, m) + g.normal(0, 0.02, m)])
    e, nn, u = r * np.cos(th), r * np.sin(th), g.normal(0.0, 2.0, n)
    return np.stack([-math.sin(LAT) * nn + math.cos(LAT) * u, e, math.cos(LAT) * nn + math.sin(LAT) * u], 1)


def _rotated(x, i, n):
    a = 0.0 if n == 1 else (i / (n - 1) - 0.5) * 2 * np.pi * 6 * 3600 / 86164.0905
    c, s = math.cos(a), math.sin(a)
    return x @ np.array([[c, s, 0.0], [-s, c, 0.0], [0.0, 0.0, 1.0]])


def _fov(case):
    """Width of the image: a field of some degrees, or for the NUFFT about 2.2 pixels per resolution element."""
    if case["kind"] == "nufft":
        return case["side"] * (2.0 / (2000.0 if case["n_ant"] <= 256 else 65000.0)) / 2.2
    return math.radians(10.0 if case["side"] >= 512 else 5.0)


def _pixels(case):
    n, h = case["side"], math.sin(_fov(case) / 2)
    c = torch.linspace(-h + h / n, h - h / n, n, dtype=torch.float64, device=DEV)
    m, l_ = torch.meshgrid(c, c, indexing="ij")
    lm = torch.stack([l_.reshape(-1), m.reshape(-1)], 1)
    lmn = torch.cat([lm, torch.sqrt(1 - lm.square().sum(1, keepdim=True))], 1)
    return lmn @ torch.from_numpy(_basis()).to(DEV)


def _eigenpairs(n_ant, n_eig, levels, g):
    """Stand-ins with the magnitudes of normalised eigenvectors, a falling spectrum, levels by energy."""
    tg = torch.Generator(device=DEV)
    tg.manual_seed(int(g.integers(1 << 62)))
    W = torch.randn(n_eig, n_ant, 2, generator=tg, device=DEV) / math.sqrt(2.0 * n_ant)
    W = W * torch.from_numpy(np.exp(g.normal(0.0, 0.5, (n_eig, 1, 1)))).to(DEV, torch.float32)
    n_neg = n_eig // 10
    lam = np.sort(np.concatenate([np.exp(g.normal(0.0, 1.5, n_eig - n_neg)), -0.05 * g.random(n_neg)]))[::-1].copy()
    lev = np.minimum((np.arange(n_eig) / max(1, n_eig) * (levels + 0.1)).astype(np.int32), levels - 1)
    # storage as an eigensolver leaves it: column-major
    return (torch.view_as_complex(W).transpose(0, 1), torch.from_numpy(lam.astype(np.float32)).to(DEV),
            torch.from_numpy(lev).to(DEV))


def _instances(case, seed):
    """[(slot, x, wavelength, W, d, level_of)] of the kinds that start from eigenpairs."""
    g = _gen(case, seed)
    out = []
    if case["kind"] == "uneven":
        x0 = _array(512, g)
        for ch in range(case["n_chan"]):
            wl = 299792458.0 / (100e6 + 100e6 * ch / max(1, case["n_chan"] - 1))
            for st in range(case["n_step"]):
                n = int(g.integers(case["l_lo"], case["l_hi"] + 1))
                k = int(g.integers(case["k_lo"], case["k_hi"] + 1))
                x = _rotated(x0[np.sort(g.choice(512, n, replace=False))], st, case["n_step"])
                out.append((ch, torch.from_numpy(x).to(DEV), wl) + _eigenpairs(n, k, case["levels"], g))
        return out
    x0 = _array(case["n_ant"], g)
    n = case.get("n_inst", 1)
    for i in range(n):
        x = torch.from_numpy(_rotated(x0, i, n)).to(DEV)
        out.append((0, x, 2.0) + _eigenpairs(case["n_ant"], case["n_eig"], case["levels"], g))
    return out


def _visibilities(case, seed):
    """x, wavelength and V of point sources in noise; V Hermitian complex128 on the GPU."""
    g = _gen(case, seed)
    n, wl = case["n_ant"], 2.0
    x = torch.from_numpy(_array(n, g)).to(DEV)
    h = math.sin(math.radians(2.5))
    n_src = 40
    lm = g.uniform(-h, h, (n_src, 2))
    dirs = np.concatenate([lm, np.sqrt(1 - (lm**2).sum(1, keepdims=True))], 1) @ _basis()
    flux = torch.from_numpy(np.exp(g.normal(0.0, 1.0, n_src))).to(DEV)
    B = _phases(x / wl, torch.from_numpy(dirs).to(DEV))
    V = (B * flux) @ B.conj().T
    tg = torch.Generator(device=DEV)
    tg.manual_seed(int(g.integers(1 << 62)))
    N = torch.view_as_complex(torch.randn(n, n, 2, generator=tg, device=DEV, dtype=torch.float64))
    N = (N + N.conj().T) / 2
    V = V + N * (V.abs().square().sum().sqrt() / N.abs().square().sum().sqrt() / 20)
    return x, wl, (V + V.conj().T) / 2


def _phases(xs, p):
    t = xs @ p.T
    return torch.polar(torch.ones_like(t), 2 * math.pi * (t - torch.round(t)))


def _solve(x, wl, V):
    """Eigenpairs of V a = lam G a with a^H G a = 1, descending, in 64 bits on the host."""
    xc, Vc = x.cpu(), V.cpu()
    G = torch.sinc(2 * (xc[:, None, :] - xc[None, :, :]).square().sum(2).sqrt() / wl).to(torch.complex128)
    C = torch.linalg.cholesky(G)
    A = torch.linalg.solve_triangular(C, Vc, upper=False)
    A = torch.linalg.solve_triangular(C, A.conj().T.contiguous(), upper=False).conj().T
    lam, U = torch.linalg.eigh((A + A.conj().T) / 2)
    W = torch.linalg.solve_triangular(C.conj().T.contiguous(), U, upper=True)
    return lam.flip(0), W.flip(1)


def _cuts(lam, n_levels):
    """Level intervals of descending eigenvalues: runs of the positive ones cut at gap midpoints, and the rest."""
    lam = np.asarray(lam.cpu(), np.float64)
    pos = lam[lam > 0]
    if n_levels == 1 or pos.size < n_levels:
        return np.array([[-INF, INF]] + [[INF, INF]] * (n_levels - 1))
    k = n_levels - 1
    at = [pos.size * i // k for i in range(1, k)]
    b = [INF] + [0.5 * (pos[i - 1] + pos[i]) for i in at]
    low = 0.5 * (pos[-1] + (lam[lam <= 0].max() if (lam <= 0).any() else 0.0))
    b.append(low)
    iv = [[b[i + 1], b[i]] for i in range(k)] + [[-INF, np.nextafter(low, -INF)]]
    return np.array(iv)


def _context():
    if not _CTX:
        _CTX.append(bb.Context(0))
    return _CTX[0]


def _synthesis(case, n_slots, n_ant_max, k_max):
    return bb.StandardSynthesis(_context(), _pixels(case), case["levels"], n_slots, max(32, n_ant_max), max(32, k_max),
                                case["precision"])


def prepare(case, seed):
    kind = case["kind"]
    st = {"case": case}
    if kind in ("eig", "batch", "uneven"):
        st["items"] = _instances(case, seed)
        n_slots = case.get("n_chan", 1)
        st["s"] = _synthesis(case, n_slots, max(i[3].shape[0] for i in st["items"]),
                             max(i[3].shape[1] for i in st["items"]))
        if kind == "batch":
            st["batch"] = bb.Batch(st["items"], DEV)
    elif kind == "step":
        x, wl, V = _visibilities(case, seed)
        st.update(x=x, wl=wl, V=V, intervals=_cuts(_solve(x, wl, V)[0], case["levels"]))
        st["s"] = _synthesis(case, 1, case["n_ant"], case["n_eig"])
    elif kind == "grad":
        _, x, wl, W, d, lev = _instances(case, seed)[0]
        tg = torch.Generator(device=DEV)
        tg.manual_seed(int(seed))
        st.update(x=x.requires_grad_(), wl=wl, W=W.requires_grad_(), d=d.requires_grad_(), lev=lev,
                  pix=_pixels(case),
                  up=torch.randn(case["levels"], case["side"] ** 2, generator=tg, device=DEV))
    elif kind == "nufft":
        st["items"] = _instances(case, seed)
        frame = _basis()
        f = torch.from_numpy(frame).to(DEV)
        far = [((c := i[1] @ f.T).amax(0) - c.amin(0)) / i[2] for i in st["items"]]
        uvw = torch.stack(far).amax(0).cpu().numpy() * 1.001
        st["s"] = bb.NufftSynthesis(_context(), _pixels(case).cpu().numpy(), case["levels"], max(32, case["n_ant"]),
                                    max(32, case["n_eig"]), case["eps"], frame, uvw)
    else:
        x, wl, V = _visibilities(case, seed)
        st.update(x=x, wl=wl, V=V, frame=_basis(), lam=_spectrum(case, seed))
        st["s"] = bb.StandardSynthesis(_context(), _pixels(dict(case, side=16)), case["levels"], 1,
                                       max(32, case["n_ant"]), 32)
    return st


def _spectrum(case, seed):
    g = _gen(case, seed + 1)
    n = case["n_eig"]
    lam = np.concatenate([np.exp(g.normal(0.0, 1.5, n - n // 3)), -np.abs(g.normal(0.0, 0.05, n // 3))])
    return torch.from_numpy(np.sort(lam)[::-1].copy()).to(DEV)


def run(state):
    kind = state["case"]["kind"]
    if kind == "grad":
        img = bb.bluebild_image(state["W"], state["d"], state["x"], state["pix"], state["lev"], state["wl"],
                                state["case"]["levels"], state["case"]["precision"])
        gW, gd, gx = torch.autograd.grad(img, (state["W"], state["d"], state["x"]), state["up"])
        return {"images": img.detach(), "W": gW, "d": gd, "x": gx}
    s = state["s"]
    if kind == "weight":
        Vw = s.uniform_weighting(state["x"], state["wl"], state["V"], state["frame"][0], state["frame"][1],
                                 math.radians(5.0))
        iv, lev = s.levels_kmeans(state["lam"])
        return {"V": Vw, "intervals": iv, "levels": lev}
    if kind == "nufft":
        s.images.zero_()
        s.collect_eig_batched(bb.Batch(state["items"], DEV))
        s.emit()
        return s.images
    s.reset()
    if kind == "eig":
        s.collect_eig(*state["items"][0])
    elif kind == "batch":
        s.collect_eig_batched(state["batch"])
    elif kind == "uneven":
        s.collect_eig_batched(bb.Batch(state["items"], DEV))
    else:
        s.collect(0, state["x"], state["wl"], state["V"], state["case"]["n_eig"], state["intervals"])
    return s.images


# -- required work ---------------------------------------------------------------------------------------------


def _products(case):
    """(sum of antennas x eigenpairs, of antennas, of eigenpairs, instances), in the mean for drawn sizes."""
    if case["kind"] == "uneven":
        n = case["n_chan"] * case["n_step"]
        ant, k = (case["l_lo"] + case["l_hi"]) / 2, (case["k_lo"] + case["k_hi"]) / 2
    else:
        n, ant, k = case.get("n_inst", 1), case["n_ant"], case["n_eig"]
    return n * ant * k, n * ant, n * k, n


def work(case):
    kind = case["kind"]
    if kind == "weight":
        n = case["n_ant"]
        return {"bytes": 32.0 * n * n + 24 * n + 12 * case["n_eig"], "flops": 12.0 * n * n}
    prod, ants, eigs, n_inst = _products(case)
    pix, slots = case["side"] ** 2, case.get("n_chan", 1)
    io = 24.0 * pix + 4 * case["levels"] * slots * pix + 24 * ants + 8 * prod + 8 * eigs
    if kind == "nufft":
        # every baseline of every level to the image: one complex value each, plus a transform of a
        # doubled grid per level
        base = n_inst * case["n_ant"] * (case["n_ant"] - 1) / 2
        m = 2.0 * case["side"]
        fft = case["levels"] * 5 * m * m * math.log2(m * m)
        return {"bytes": io + 8 * case["levels"] * m * m, "flops": 8 * base * case["n_eig"] + fft}
    if kind == "step":
        n = case["n_ant"]
        return {"bytes": io + 16.0 * n * n, "flops": 8.0 * prod * pix + 36.0 * n**3}
    if kind == "grad":
        return {"bytes": io + 8 * prod + 24 * ants + 4 * eigs + 4 * case["levels"] * pix, "flops": 24.0 * prod * pix}
    return {"bytes": io, "flops": 8.0 * prod * pix}


# -- results in 64 bits ----------------------------------------------------------------------------------------


def _images(items, pix, n_levels, n_slots):
    """Level images of eigenpairs in 64 bits, pixels in slices."""
    img = torch.zeros(n_slots, n_levels, pix.shape[0], dtype=torch.float64, device=DEV)
    for slot, x, wl, W, d, lev in items:
        Wh = W.to(torch.complex128).conj().T.contiguous()
        Q = torch.nn.functional.one_hot(lev.long() + 1, n_levels + 1)[:, 1:].T.double() * d.double()
        for a in range(0, pix.shape[0], 1 << 16):
            E = Wh @ _phases(x / wl, pix[a:a + (1 << 16)])
            img[slot, :, a:a + (1 << 16)] += Q @ (E.real.square() + E.imag.square())
    return img


def _weighted(case, seed):
    x, wl, V = (v.cpu().numpy() if torch.is_tensor(v) else v for v in _visibilities(case, seed))
    n = x.shape[0]
    dx = x[:, None, :] - x[None, :, :]
    cell = []
    for e in _basis()[:2]:
        a = ((dx[..., 0] * e[0] + dx[..., 1] * e[1]) + dx[..., 2] * e[2]) * (math.radians(5.0) / wl)
        cell.append(np.trunc(a + np.copysign(0.5, a)).astype(np.int64))
    _, inv, cnt = np.unique(cell[0] * (1 << 31) + cell[1], return_inverse=True, return_counts=True)
    return V / cnt[inv].reshape(n, n)


def _kmeans(lam, n_levels):
    """Exact one-dimensional k-means of the positive eigenvalues (descending), by dynamic programme."""
    pos = lam[lam > 0]
    n, k = pos.size, n_levels - 1
    wide = pos.astype(np.longdouble)
    s1, s2 = np.concatenate([[0], np.cumsum(wide)]), np.concatenate([[0], np.cumsum(wide**2)])
    i = np.arange(n + 1)
    with np.errstate(divide="ignore", invalid="ignore"):
        cost = (s2[None, :] - s2[:, None]) - (s1[None, :] - s1[:, None]) ** 2 / (i[None, :] - i[:, None])
    cost[i[None, :] <= i[:, None]] = INF
    cost[i[None, :] > i[:, None]] = np.maximum(cost[i[None, :] > i[:, None]], 0)
    best, back = cost[0].copy(), []
    for _ in range(1, k):
        t = best[:, None] + cost
        back.append(np.argmin(t, axis=0))
        best = t.min(axis=0)
    at, j = [], n
    for b in reversed(back):
        j = int(b[j])
        at.append(j)
    b = [INF] + [0.5 * (pos[j - 1] + pos[j]) for j in reversed(at)]
    low = 0.5 * (pos[-1] + lam[lam <= 0].max())
    b.append(low)
    return np.array([[b[j + 1], b[j]] for j in range(k)] + [[-INF, np.nextafter(low, -INF)]])


def exact(case, seed):
    kind = case["kind"]
    if kind == "weight":
        iv = _kmeans(_spectrum(case, seed).cpu().numpy(), case["levels"])
        return {"V": torch.from_numpy(_weighted(case, seed)), "intervals": torch.from_numpy(iv), "levels": None}
    pix = _pixels(case)
    if kind == "step":
        x, wl, V = _visibilities(case, seed)
        lam, W = _solve(x, wl, V)
        iv = _cuts(lam, case["levels"])
        k = case["n_eig"]
        lam, W = lam[:k], W[:, :k]
        lev = np.full(k, -1, np.int32)
        for l_ in range(case["levels"] - 1, -1, -1):
            lev[(lam.numpy() >= iv[l_, 0]) & (lam.numpy() <= iv[l_, 1])] = l_
        item = (0, x, wl, W.to(DEV), lam.to(DEV), torch.from_numpy(lev).to(DEV))
        return _images([item], pix, case["levels"], 1)
    items = _instances(case, seed)
    if kind == "nufft":
        return _images(items, pix, case["levels"], 1)[0]
    if kind != "grad":
        return _images(items, pix, case["levels"], case.get("n_chan", 1))
    _, x, wl, W, d, lev = items[0]
    tg = torch.Generator(device=DEV)
    tg.manual_seed(int(seed))
    up = torch.randn(case["levels"], case["side"] ** 2, generator=tg, device=DEV).double()
    img = _images(items, pix, case["levels"], 1)[0]
    W, d = W.to(torch.complex128), d.double()
    gW, gd, gx = torch.zeros_like(W), torch.zeros_like(d), torch.zeros_like(x)
    for a in range(0, pix.shape[0], 1 << 15):
        p = pix[a:a + (1 << 15)]
        B = _phases(x / wl, p)
        E = W.conj().T.contiguous() @ B
        c = up[lev.long(), a:a + (1 << 15)]
        gd += (c * (E.real.square() + E.imag.square())).sum(1)
        M = (d[:, None] * c) * E.conj()
        gW += 2 * (B @ M.T.contiguous())
        H = (W.conj() @ M)                                  # (L, P)
        gx += -(4 * math.pi / wl) * ((H * B).imag @ p)
    return {"images": img, "W": gW, "d": gd, "x": gx}
