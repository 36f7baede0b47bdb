"""Synthesis at the sizes where the dispatch takes another tile than a K class's own: images whose tiles leave the last
round nearly empty or are fewer than the compute units, and local memory that leaves room for fewer workgroups.  Two
instances of one slot (the second adds to the first's images), a ragged last tile, against the FP64 oracle at 2000 of
the pixels, tolerances as for the other synthesis tests."""

import numpy as np
import pytest

import sims
from tests._helpers import level_errors, oracle_images

pytestmark = pytest.mark.gpu

TOL = {"fp32": 1e-5, "fp32_3m": 1e-5, "bf16x3": 1e-4, "bf16x3_3m": 1e-4}


@pytest.fixture(scope="module")
def ctx(gpu):
    from paper_2310_09200_amd import Context
    c = Context(0)
    yield c
    c.close()


@pytest.mark.parametrize("precision", list(TOL))
@pytest.mark.parametrize("n_ant, n_eig, side, n_levels", [
    (70, 60, 201, 3),    # 316 tiles of 128 pixels on 256 units
    (70, 100, 201, 3),
    (70, 200, 201, 3),
    (70, 200, 151, 3),   # 179 tiles
    (70, 60, 101, 16),   # 80
    (200, 24, 401, 5),   # 32 rows, two workgroups a unit in the three-product form
    (29, 24, 515, 10),
    (900, 60, 201, 5),   # 64 rows, one eight-wave workgroup a unit
])
def test_tiles_chosen_by_size(ctx, n_ant, n_eig, side, n_levels, precision):
    from paper_2310_09200_amd import Batch, StandardSynthesis
    print(f"case tile rules {precision} {n_ant} {n_eig} {side} {n_levels}", flush=True)
    g = np.random.default_rng(n_ant + n_eig + side)
    pix = sims.pixel_grid(side, 5.0, 70.0)
    sel = np.unique(np.concatenate([g.integers(0, side * side, 2000), np.arange(side * side - 130, side * side)]))
    items, want = [], 0.0
    for i in range(2):
        x = sims.disk_layout(n_ant, 1500.0, g, z_sigma_m=1.0)
        W = sims.random_eigvecs(n_ant, n_eig, g).astype(np.complex64)
        d = g.uniform(0.5, 2.0, n_eig).astype(np.float32)
        lev = np.concatenate([np.arange(n_levels), g.integers(-1, n_levels, n_eig - n_levels)]).astype(np.int32)
        items.append((0, x, 2.0 + 0.1 * i, W, d, lev))
        want = want + oracle_images(W.astype(np.complex128), d.astype(np.float64), lev, x, 2.0 + 0.1 * i, pix[sel],
                                    n_levels)
    s = StandardSynthesis(ctx, pix, n_levels, 1, n_ant, n_eig, precision)
    s.collect_eig_batched(Batch(items, ctx.device))
    s.sync()
    got = s.images.double().cpu().numpy().reshape(n_levels, -1)[:, sel]
    s.close()
    assert np.all(level_errors(got, want)[:, 0] <= TOL[precision])
