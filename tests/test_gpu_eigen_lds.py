"""The pre-step eigenproblem after kernels that leave NaN in local memory: its exchange between workgroups must not
read rows that no workgroup published.  Tolerance: as for the eigenvalues of well conditioned problems elsewhere,
1e-12 of the largest."""

import numpy as np
import pytest

import sims
from scipy import linalg

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n", [65, 129, 160, 200, 256, 257])
def test_after_nan_in_local_memory(gpu, n):
    from paper_2310_09200_amd import Context, StandardSynthesis
    print("case NaN in local memory, size", n, flush=True)
    ctx = Context(0)
    g = np.random.default_rng(n)
    L, K = 256, 64
    pix = sims.pixel_grid(96, 5.0, 90.0)
    b = StandardSynthesis(ctx, pix, 1, 1, L, K)
    x = sims.disk_layout(L, 2000.0, g, z_sigma_m=1.0)
    W = sims.random_eigvecs(L, K, g).astype(np.complex64)
    nan = np.full((1, pix.shape[0]), np.nan, np.float32)
    s = StandardSynthesis(ctx, np.array([[0.0, 0.0, 1.0]]), 1, 1, n, n, gram="identity")
    V = g.normal(size=(n, n)) + 1j * g.normal(size=(n, n))
    V = V + V.conj().T
    want = linalg.eigh(V, eigvals_only=True)[::-1]
    for _ in range(4):
        _, _, dx = b.eig_backward(x, 2.0, W, np.ones(K, np.float32), np.zeros(K, np.int32), nan)
        b.sync()
        assert np.all(np.isnan(dx.cpu().numpy()))
        _, lam, _, _ = s.prestep(sims.disk_layout(n, 400.0, g), 2.0, V, n, np.array([[-np.inf, np.inf]]))
        assert np.max(np.abs(lam.cpu().numpy() - want)) <= 1e-12 * np.max(np.abs(want)) * max(1.0, n / 64)
    s.close()
    b.close()
    ctx.close()
