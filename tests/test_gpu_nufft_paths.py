"""NUFFT synthesis at the edges of its kernels' cases, against the FP64 NUFFT oracle.

Tolerance: 1e-5 of each level's peak, as for the other comparisons of the FP32
grid and transform with this oracle, at the pixels inside the planned extents.  A
pixel at an end of an extent lies a quarter of the type-2 grid from its centre, so
that for an even kernel width its window ends on an exact tie, where rounding and
the oracle's convention may choose different windows, equally good to epsilon.
"""
import numpy as np
import pytest
import torch

import sims
from oracle import nufft_ref as nf

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def ctx(gpu):
    from paper_2310_09200_amd import Context
    c = Context(0)
    yield c
    c.close()


def _pixels(n, fov_deg, frame):
    h = np.sin(np.deg2rad(fov_deg) / 2)
    l_, m = np.meshgrid(np.linspace(-h, h, n), np.linspace(-h, h, n))
    lmn = np.stack([l_.ravel(), m.ravel(), np.sqrt(1 - l_.ravel() ** 2 - m.ravel() ** 2)], 1)
    return lmn @ frame


def _case(n_levels, extent, seed, n_inst=2, fov_deg=20.0):
    """Random eigenpairs of arrays of the given extents (wavelengths, frame axes); unused and negative ones too."""
    g = np.random.default_rng(seed)
    frame = np.array(sims.tangent_basis(40.0))
    items = []
    for i in range(n_inst):
        L, K, wl = 24 - 5 * i, max(20, n_levels), 1.5 + 0.25 * i
        x = (g.random((L, 3)) - 0.5) * np.asarray(extent) * wl @ frame
        W = g.normal(size=(L, K)) + 1j * g.normal(size=(L, K))
        d = g.normal(size=K) * (1.0 + np.arange(K))
        lev = np.concatenate([np.arange(n_levels), g.integers(-1, n_levels, K - n_levels)]).astype(np.int32)
        items.append((x, wl, W.astype(np.complex64), d.astype(np.float32), lev))
    b = np.zeros(3)
    for x, wl, *_ in items:
        b = np.maximum(b, np.max(np.abs((x[:, None] - x[None]).reshape(-1, 3) @ frame.T), axis=0) / wl)
    return _pixels(14, fov_deg, frame), items, frame, b * 1.01


def _check(ctx, n_levels, items, pix, frame, uvw, eps, calls, thick=None):
    from paper_2310_09200_amd import Batch, NufftSynthesis
    P = nf.plan_params(eps, uvw, nf.rotate(pix, frame))
    if thick:
        assert thick[0] < P["N"][2] <= thick[1], P["N"]
    c = nf.rotate(pix, frame)
    lo, hi = c.min(axis=0), c.max(axis=0)
    inside = np.all(np.abs(c - (lo + hi) / 2) < (hi - lo) / 2 * (1 - 1e-9), axis=1)
    plan = NufftSynthesis(ctx, pix, n_levels, 64, 64, eps, frame, uvw)
    for _ in range(2):  # the second pass starts from the grid that the first one left
        plan.images.zero_()
        for ch in np.array_split(np.arange(len(items)), calls):
            plan.collect_eig_batched(Batch([(0, *items[i]) for i in ch], ctx.device))
        plan.emit()
        plan.sync()
        got = plan.images.double().cpu().numpy()
        ref = [(x, wl, W.astype(np.complex128), d.astype(np.float64), np.arange(n_levels)[:, None] == lev[None])
               for x, wl, W, d, lev in items]
        want = nf.nufft_images(ref, pix, eps, X=uvw, frame=frame)
        for a, b in zip(got, want):
            assert np.max(np.abs(a - b)[inside]) <= 1e-5 * np.max(np.abs(b))
    plan.close()


# levels: below, at and beyond a product's eight, with the vector remainder (9, 11) and a second product (12, 16)
@pytest.mark.parametrize("n_levels", [1, 2, 8, 9, 11, 12, 16])
@pytest.mark.parametrize("depth", [16, 32, 64])
def test_spread_levels_and_depths(ctx, n_levels, depth):
    print(f"case nufft levels={n_levels} depth={depth}", flush=True)
    pix, items, frame, uvw = _case(n_levels, (14.0, 17.0, {16: 20.0, 32: 150.0, 64: 400.0}[depth]), 7)
    _check(ctx, n_levels, items, pix, frame, uvw, 1e-5, 1, thick={16: (0, 16), 32: (16, 32), 64: (32, 64)}[depth])


# every kernel width; grids down to twice the kernel's width (all runs wrap); one and two calls before an emit
@pytest.mark.parametrize("eps", [1e-2, 1e-3, 1e-4, 1e-5, 1e-6, 1e-7])
@pytest.mark.parametrize("extent", [(0.2, 0.2, 0.2), (2.0, 40.0, 5.0), (40.0, 3.0, 5.0)])
@pytest.mark.parametrize("calls", [1, 2])
def test_spread_widths_and_wraps(ctx, eps, extent, calls):
    print(f"case nufft eps={eps} extent={extent} calls={calls}", flush=True)
    pix, items, frame, uvw = _case(3, extent, 8)
    _check(ctx, 3, items, pix, frame, uvw, eps, calls)


_LENGTHS = sorted(m for m in (4 * 2 ** a * 3 ** b * 5 ** c for a in range(12) for b in range(8) for c in range(6))
                  if 24 <= m <= 9000)


# every transform length up to 9000: two and three passes of each radix in
# registers, and the lengths left to the in-place transform
@pytest.mark.parametrize("length", _LENGTHS)
def test_line_lengths(ctx, length):
    print(f"case nufft line length={length}", flush=True)
    eps, w = 1e-5, 6
    h = np.sin(np.deg2rad(10.0))
    extent = (length / 2 - w - 0.5) / (8 * h) / 1.01
    g = np.random.default_rng(length)
    frame = np.array(sims.tangent_basis(40.0))
    x = np.array([[0.0, 0, 0], [extent, 0, 0]] + [[e, 0, 0] for e in extent * g.random(4)])
    x[1:, 1:] = 0.3 * (g.random((5, 2)) - 0.5)
    W = (g.normal(size=(6, 6)) + 1j * g.normal(size=(6, 6))).astype(np.complex64)
    items = [(x @ frame, 1.0, W, np.ones(6, np.float32), np.zeros(6, np.int32))]
    pix = _pixels(10, 20.0, frame)
    uvw = np.array([extent * 1.01, 0.35, 0.35])
    assert nf.plan_params(eps, uvw, nf.rotate(pix, frame))["M"][0] == length
    _check(ctx, 1, items, pix, frame, uvw, eps, 1)


# Blocks of more than one part (1024 baselines), where a baseline reaches the most of them: stations on a short
# diagonal, ordered along it, so that every baseline lies just past the grid's origin, and 18 points on axes 0 and 1,
# of which the last block of 8 or 4 columns holds 2.
@pytest.mark.parametrize("eps, depth, n_ant", [(1e-7, 16, 305), (1e-6, 16, 305), (1e-7, 32, 240)])
def test_spread_parts_across_the_wrap(ctx, eps, depth, n_ant):
    from paper_2310_09200_amd import Batch, NufftSynthesis
    print(f"case nufft parts eps={eps} depth={depth} antennas={n_ant}", flush=True)
    w = nf.kernel_width(eps)
    g = np.random.default_rng(n_ant + w)
    frame = np.array(sims.tangent_basis(40.0))
    pix = _pixels(14, 20.0, frame)
    c = nf.rotate(pix, frame)
    S = 0.5 * (c.max(axis=0) - c.min(axis=0))
    uvw = np.array([(18 - w - 0.5) / (8 * S[0]), (18 - w - 0.5) / (8 * S[1]), (depth - w - 0.5) / (8 * S[2])])
    P = nf.plan_params(eps, uvw, c)
    assert list(P["N"]) == [18, 18, depth]
    x = np.sort(g.random(n_ant))[::-1, None] * (np.array([0.3, 0.3, 0.0]) * P["h"]) @ frame
    W = (g.normal(size=(n_ant, 6)) + 1j * g.normal(size=(n_ant, 6))).astype(np.complex64)
    d, lev = g.normal(size=6).astype(np.float32), np.array([0, 1, 0, 1, 0, -1], np.int32)
    plan = NufftSynthesis(ctx, pix, 2, n_ant, 6, eps, frame, uvw)
    plan.collect_eig_batched(Batch([(0, x, 1.0, W, d, lev)], ctx.device))
    plan.emit()
    plan.sync()
    got = plan.images.double().cpu().numpy()
    plan.close()
    ref = [(x, 1.0, W.astype(np.complex128), d.astype(np.float64), np.arange(2)[:, None] == lev[None])]
    want = nf.nufft_images(ref, pix, eps, X=uvw, frame=frame)
    lo, hi = c.min(axis=0), c.max(axis=0)
    inside = np.all(np.abs(c - (lo + hi) / 2) < (hi - lo) / 2 * (1 - 1e-9), axis=1)
    for a, b in zip(got, want):
        assert np.max(np.abs(a - b)[inside]) <= 1e-5 * np.max(np.abs(b))


def test_emit_under_capture(ctx):
    """A transform captured between two spreads and replayed after them images both."""
    from paper_2310_09200_amd import Batch, NufftSynthesis
    print("case nufft emit under capture", flush=True)
    pix, items, frame, uvw = _case(3, (14.0, 17.0, 20.0), 9)
    batches = [Batch([(0, *it)], ctx.device) for it in items]
    plans = [NufftSynthesis(ctx, pix, 3, 64, 64, 1e-5, frame, uvw) for _ in range(2)]
    for b in batches:
        plans[0].collect_eig_batched(b)
    plans[0].emit()
    plans[0].sync()
    want = plans[0].images.double().cpu().numpy()
    p = plans[1]
    p.collect_eig_batched(batches[0])
    p.sync()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        p.emit()
    for rnd in range(3):
        p.images.zero_()
        p.collect_eig_batched(batches[1])
        if rnd > 0:
            p.collect_eig_batched(batches[0])
        torch.cuda.synchronize()
        graph.replay()
        torch.cuda.synchronize()
        got = p.images.double().cpu().numpy()
        for a, b in zip(got, want):
            assert np.max(np.abs(a - b)) <= 1e-5 * np.max(np.abs(b)), rnd
    for q in plans:
        q.close()
