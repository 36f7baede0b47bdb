"""GPU parity of the split 16-bit products where they can go wrong: tile and block edges, columns of W
of very different magnitudes, phases too large for the fast form, non-finite inputs.

The tolerance is the sum of what the arithmetic may lose, element by element.  With S_k = sum_l |w_lk|,
of E_kp (unit phases, |b| = 1):
  the split of both operands and the dropped lo lo     4 * 2^-22 S_k
  sine and cosine of an FP32 argument in turns         (2 * 1.3e-7 + 2 pi 2^-25) S_k
  an FP64 phase of T turns                             2 pi T 2^-50 S_k
  the sums: 3 MFMAs per plane and 32 antennas, each of
  their accumulations rounded or truncated             3 * (3 ceil(L / 32) + 2) * 2^-23 S_k
and of the image sum_k d_k |E_kp|^2: 2 |E| dE + dE^2 each, (K + 8) 2^-24 |d_k| |E|^2 for its own FP32 sum.
BF16 words hold 16 bits instead of 22: 2^-16 in place of 2^-22.
"""

import numpy as np
import pytest
import torch

import oracle as ref
import sims

pytestmark = pytest.mark.gpu

PRECISIONS = ["fp32", "fp32_3m", "bf16x3", "bf16x3_3m"]


@pytest.fixture(scope="module")
def ctx(gpu):
    from paper_2310_09200_amd import Context
    return Context(0)


def images(ctx, pix, n_levels, x, wl, W, d, lev, precision, tiles=None):
    from paper_2310_09200_amd import StandardSynthesis
    L, K = W.shape
    s = StandardSynthesis(ctx, pix, n_levels, 1, L, K, precision)
    if tiles is not None:
        s.tiles = tiles
    s.collect_eig(0, x, wl, W, d, lev)
    s.sync()
    out = s.images[0].double().cpu().numpy()
    s.close()
    return out


def expected(pix, n_levels, x, wl, W, d, lev, precision):
    """(images, elementwise bound) in 64 bits, of the inputs as the library takes them."""
    W = W.astype(np.complex64).astype(np.complex128)
    d = d.astype(np.float32).astype(np.float64)
    x0 = x - x[0]
    B = ref.phases(x0, pix, wl)
    E = W.conj().T @ B
    L, K = W.shape
    S = np.abs(W).sum(axis=0)
    turns = np.abs(x0).sum(axis=1).max() / wl * max(1.0, np.abs(pix).max())
    word = 2.0**-22 if precision.startswith("fp32") else 2.0**-16
    dE = S * (4 * word + 2 * 1.3e-7 + 2 * np.pi * (2.0**-25 + turns * 2.0**-50) + 3 * (3 * -(-L // 32) + 2) * 2.0**-23)
    a = np.abs(E)
    tol = np.abs(d)[:, None] * (2 * a * dE[:, None] + dE[:, None] ** 2 + (K + 8) * 2.0**-24 * a * a)
    member = (lev[None, :] == np.arange(n_levels)[:, None]).astype(np.float64)
    return member @ (d[:, None] * a * a), member @ tol


def check(ctx, pix, n_levels, x, wl, W, d, lev, precision, tiles=None):
    want, tol = expected(pix, n_levels, x, wl, W, d, lev, precision)
    got = images(ctx, pix, n_levels, x, wl, W, d, lev, precision, tiles)
    worst = np.max(np.abs(got - want) / np.maximum(tol, 1e-300))
    print("worst error over bound", worst, flush=True)
    assert np.all(np.abs(got - want) <= tol)
    return got


def case(L, K, n_pix, n_levels, seed, diameter=2000.0):
    g = np.random.default_rng(seed)
    x = sims.disk_layout(L, diameter, g, z_sigma_m=2.0)
    pix = sims.pixel_grid(int(np.ceil(np.sqrt(n_pix))), 6.0, 60.0)[:n_pix]
    W = sims.random_eigvecs(L, K, g)
    d = np.exp(g.normal(0, 1, K))
    lev = g.integers(-1, n_levels, K).astype(np.int32)
    return x, 2.0, pix, W, d, lev


# antennas around the 32-deep step and one more chunk, eigenpairs around the 16-row blocks and each pass
# (32, 64, 128, 256 a pass), pixels around 64- and 128-pixel tiles, one level and the most
@pytest.mark.parametrize("precision", PRECISIONS)
@pytest.mark.parametrize("L,K,n_pix,n_levels", [
    (1, 1, 1, 1), (31, 16, 63, 16), (32, 17, 64, 2), (33, 33, 65, 3), (64, 48, 129, 16), (65, 65, 127, 4),
    (97, 113, 200, 2), (40, 129, 257, 3), (130, 257, 100, 16), (70, 273, 66, 2), (1024, 31, 70, 2), (20, 1024, 70, 16),
])
def test_edges(ctx, L, K, n_pix, n_levels, precision):
    print("case edges", L, K, n_pix, n_levels, precision, flush=True)
    x, wl, pix, W, d, lev = case(L, K, n_pix, n_levels, 7 * L + K)
    check(ctx, pix, n_levels, x, wl, W, d, lev, precision)


@pytest.mark.parametrize("n_pix", [128 * 256 - 1, 128 * 256, 128 * 256 + 1])
@pytest.mark.parametrize("K,precision", [(40, "fp32_3m"), (100, "fp32_3m"), (140, "fp32")])
def test_image_sizes_around_the_narrow_tiles(ctx, K, precision, n_pix):
    """A 128-pixel tile gives way to its 64-pixel sibling below one tile per compute unit."""
    print("case narrow", K, precision, n_pix, flush=True)
    x, wl, pix, W, d, lev = case(36, K, n_pix, 2, n_pix + K)
    check(ctx, pix, 2, x, wl, W, d, lev, precision)


@pytest.mark.parametrize("precision", PRECISIONS)
def test_columns_of_any_magnitude(ctx, precision):
    """Columns scaled by 2^-60 .. 2^60 (weights by the inverse square), one zero column, and entries from
    2^-40 to 1 of a column's largest: every eigenpair keeps its accuracy."""
    print("case magnitudes", precision, flush=True)
    x, wl, pix, W, d, _ = case(50, 41, 150, 41, 3)
    g = np.random.default_rng(4)
    e = np.linspace(-60, 60, 41).round()
    W = W * 2.0 ** g.integers(-40, 1, W.shape) * 2.0**e
    W[:, 20] = 0
    d = d * 2.0 ** (-2 * e)
    for k0 in range(0, 41, 16):  # at most 16 levels: every column gets one of its own in turn
        lev = np.full(41, -1, np.int32)
        lev[k0:k0 + 16] = np.arange(len(lev[k0:k0 + 16]))
        got = check(ctx, pix, 16, x, wl, W, d, lev, precision)
        assert np.all(got[lev[20]] == 0) or lev[20] < 0


@pytest.mark.parametrize("precision", ["fp32", "fp32_3m"])
@pytest.mark.parametrize("diameter,offset", [(2000.0, 6.4e6), (3.0e6, 0.0), (1.0e8, 0.0)])
def test_large_positions(ctx, precision, diameter, offset):
    """Far from the origin (fast phases after the shift to the first antenna), and beyond 2^19 turns."""
    print("case positions", precision, diameter, offset, flush=True)
    x, wl, pix, W, d, lev = case(48, 20, 130, 2, 5, diameter)
    check(ctx, pix, 2, np.round(x * 1024) / 1024 + offset, wl, W, d, lev, precision)


def test_pixels_longer_than_unit(ctx):
    """A wave with one long pixel vector takes the general phases, and all its pixels agree with the oracle."""
    print("case long pixels", flush=True)
    x, wl, pix, W, d, lev = case(48, 20, 130, 2, 6)
    x = np.round(x * 1024) / 1024 * 400.0  # with the long pixels past 2^19 turns
    pix = pix.copy()
    pix[70] *= 900.0
    pix[129] *= 3.0
    check(ctx, pix, 2, x, wl, W, d, lev, "fp32_3m")


@pytest.mark.parametrize("precision", PRECISIONS)
def test_non_finite_inputs_stay_where_they_belong(ctx, precision):
    """A NaN pixel spoils its own pixel, a non-finite column its own level, a non-finite antenna everything."""
    print("case non-finite", precision, flush=True)
    x, wl, pix, W, d, _ = case(48, 20, 130, 2, 8)
    lev = (np.arange(20) % 2).astype(np.int32)
    bad = pix.copy()
    bad[77, 1] = np.nan
    got = images(ctx, bad, 2, x, wl, W, d, lev, precision)
    clean = images(ctx, pix, 2, x, wl, W, d, lev, precision)
    ok = np.arange(130) != 77
    assert np.all(np.isnan(got[:, 77])) and np.all(np.isfinite(got[:, ok]))
    np.testing.assert_allclose(got[:, ok], clean[:, ok], rtol=1e-5, atol=1e-5 * clean.max())
    for v in (np.nan, np.inf):
        Wb = W.copy()
        Wb[3, 5] = v
        got = images(ctx, pix, 2, x, wl, Wb, d, lev, precision)
        assert not np.any(np.isfinite(got[1])) and np.array_equal(got[0], clean[0])
        xb = x.copy()
        xb[9, 0] = v
        assert not np.any(np.isfinite(images(ctx, pix, 2, xb, wl, W, d, lev, precision)))
