"""k-means levels and uniform weighting at the edges of their kernels: one
workgroup (at most 64 values), the chip-wide sweeps, and the fallback of a handle
whose workspace holds no table of costs, against the CPU oracle.  Level ids are
whole numbers and interval bounds are single roundings of sums of two inputs, so
both have to be equal."""
import numpy as np
import pytest
import torch

import sims
from oracle import levels_ref as lv
from oracle import weighting_ref as uw

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n_ant_max", [16, 1024])
@pytest.mark.parametrize("n", [2, 63, 64, 65, 128, 341, 1024])
@pytest.mark.parametrize("k", [1, 2, 8])
def test_kmeans_paths(gpu, n, k, n_ant_max):
    from paper_2310_09200_amd import Context, StandardSynthesis
    print(f"case kmeans n={n} k={k} n_ant_max={n_ant_max}", flush=True)
    if k > n:
        pytest.skip("fewer values than levels")
    g = np.random.default_rng(1000 * n + k)
    # clusters far wider apart than they are wide: one best partition, found by
    # any order of the sums; -1 values interleaved beyond the first k
    centres = 4.0 ** np.arange(k)
    lam = centres[np.arange(n) % k] * (1 + 1e-3 * g.random(n))
    lam[k:][g.random(n - k) < 0.25] = -1.0
    lam = lam[g.permutation(n)]
    ctx = Context(0)
    s = StandardSynthesis(ctx, sims.pixel_grid(16, 5.0), k + 1, 1, n_ant_max, 16, "fp32")
    iv, lev = s.levels_kmeans(torch.as_tensor(lam), negative_level=True)
    s.sync()
    want = lv.kmeans_intervals(lam, k, negative_level=True)
    np.testing.assert_array_equal(iv.cpu().numpy(), want)
    np.testing.assert_array_equal(lev.cpu().numpy(), lv.level_of(lam, want))
    s.close()
    ctx.close()


@pytest.mark.parametrize("L", [1, 2, 255, 256, 257])
def test_uniform_weighting_mirrored_cells(gpu, L):
    """Coincident antennas (pairs at the origin) and many pairs per cell."""
    from paper_2310_09200_amd import Context, StandardSynthesis
    print(f"case uniform weighting mirrored cells L={L}", flush=True)
    g = np.random.default_rng(L)
    x = np.round(g.normal(0.0, 3.0, (L, 3))) * 2.0
    x[L // 2:L // 2 + 2] = x[0]
    V = g.normal(size=(L, L)) + 1j * g.normal(size=(L, L))
    e_u, e_v = np.array([1.0, 0.0, 0.0]), np.array([0.0, 1.0, 0.0])
    ctx = Context(0)
    s = StandardSynthesis(ctx, sims.pixel_grid(16, 5.0), 2, 1, 512, 16, "fp32")
    out = s.uniform_weighting(torch.as_tensor(x), 2.0, torch.as_tensor(V), e_u, e_v, 0.7)
    s.sync()
    np.testing.assert_array_equal(out.cpu().numpy(), uw.apply_uniform_weighting(V, x, 2.0, e_u, e_v, 0.7))
    s.close()
    ctx.close()
