"""dW of the backward at the edges of its tiles (32 and 128 antennas, 64 and 128
eigenpairs, 64 pixels) and over weights of very different sizes, against the CPU
oracle.  Tolerance per eigenpair: 2e-5 of its largest |dW|, ten times the rounding
of FP32 phases and fields (about 1e-6 of a sum over random terms)."""
import numpy as np
import pytest

import oracle as ref
import sims

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("L,K,n_pix", [(1, 1, 1), (2, 2, 63), (31, 63, 64), (32, 64, 65), (33, 65, 129), (127, 128, 193),
                                       (128, 129, 200), (129, 40, 1000), (257, 200, 67)])
@pytest.mark.parametrize("spread", [0.0, 25.0])
def test_dw_edges(gpu, L, K, n_pix, spread):
    from paper_2310_09200_amd import Context, StandardSynthesis
    print(f"case dW edges L={L} K={K} n_pix={n_pix} spread={spread}", flush=True)
    g = np.random.default_rng(1000 * L + K)
    n_levels = 3
    x = sims.disk_layout(L, 2000.0, g, z_sigma_m=1.0)
    wl = sims.wavelength_m(150e6)
    pix = sims.pixel_grid(int(np.ceil(np.sqrt(n_pix))), 5.0, 90.0)[:n_pix]
    W = sims.random_eigvecs(L, K, g).astype(np.complex64)
    d = (g.choice([-1.0, 1.0], K) * 10.0 ** (spread * (g.random(K) - 0.5))).astype(np.float32)
    lev = g.integers(-1, n_levels, K).astype(np.int32)
    lev[0] = 0
    wts = g.standard_normal((n_levels, n_pix)).astype(np.float32)
    ctx = Context(0)
    s = StandardSynthesis(ctx, pix, n_levels, 1, max(L, 2), K)
    dW, dd, dx = s.eig_backward(x, wl, W, d, lev, wts)
    s.sync()
    dW = dW.cpu().numpy()
    s.close()
    ctx.close()
    rW, _, _ = ref.grad_ref.grad(W.astype(np.complex128), d.astype(np.float64), x, ref.membership_from_level_of(lev, n_levels),
                                 wts.astype(np.float64), pix, wl)
    for k in range(K):
        if lev[k] < 0:
            assert np.all(dW[:, k] == 0)
        else:
            assert np.max(np.abs(dW[:, k] - rW[:, k])) <= 2e-5 * np.max(np.abs(rW[:, k])), k
