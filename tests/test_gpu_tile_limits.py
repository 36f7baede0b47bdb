"""Every tile shape at the sizes where local memory is scarcest: many antennas, many levels.  Images against the
FP64 oracle, tolerances as for the other synthesis tests."""

import numpy as np
import pytest

import sims
from tests._helpers import level_errors, oracle_images

pytestmark = pytest.mark.gpu

TOL = {"fp32": 1e-5, "fp32_3m": 1e-5, "bf16x3": 1e-4, "bf16x3_3m": 1e-4}
KS = [20, 50, 100, 140]  # one instance per K class


@pytest.fixture(scope="module")
def ctx(gpu):
    from paper_2310_09200_amd import Context
    c = Context(0)
    yield c
    c.close()


def case(n_ant, n_levels):
    g = np.random.default_rng(n_ant + n_levels)
    pix = sims.pixel_grid(12, 5.0, 70.0)
    wl, items, want = 2.0, [], []
    for slot, K in enumerate(KS):
        x = sims.disk_layout(n_ant, 1500.0, g, z_sigma_m=1.0)
        W = sims.random_eigvecs(n_ant, K, g).astype(np.complex64)
        d = g.uniform(0.5, 2.0, K).astype(np.float32)
        lev = np.concatenate([np.arange(n_levels), g.integers(0, n_levels, K - n_levels)]).astype(np.int32)
        items.append((slot, x, wl, W, d, lev))
        want.append(oracle_images(W.astype(np.complex128), d.astype(np.float64), lev, x, wl, pix, n_levels))
    return pix, items, np.array(want)


@pytest.mark.parametrize("precision", list(TOL))
@pytest.mark.parametrize("n_ant, n_levels", [(64, 16), (512, 13), (1024, 9), (1024, 16)])
def test_tiles_where_local_memory_is_scarce(ctx, n_ant, n_levels, precision):
    from paper_2310_09200_amd import Batch, StandardSynthesis, tile_shapes
    pix, items, want = case(n_ant, n_levels)
    b = Batch(items, ctx.device)
    s = StandardSynthesis(ctx, pix, n_levels, len(KS), n_ant, max(KS), precision)
    shapes = tile_shapes(precision)
    allowed = [[t for t, *_, cl in shapes if c in cl] for c in range(4)]
    for j in range(max(len(a) for a in allowed)):
        s.tiles = [a[j % len(a)] for a in allowed]
        print(f"case tiles {precision} {n_ant} antennas {n_levels} levels {s.tiles}", flush=True)
        s.reset()
        s.collect_eig_batched(b)
        s.sync()
        for got, w in zip(s.images.double().cpu().numpy(), want):
            assert np.all(level_errors(got, w)[:, 0] <= TOL[precision]), s.tiles
    ms = s.autotune_batched(b, reps=1)
    assert all(min(row.values()) > 0 for row in ms.values())
    s.close()
