"""The pre-step eigenproblem when its workgroups give up waiting for each other: the library's solver answers, over a
workspace that held NaN.  Tolerance: eigenvalues as elsewhere, 1e-12 of the largest (n / 64, and cond(G) below 10)."""

import numpy as np
import pytest
from scipy import linalg

import oracle as ref
import sims

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("gram", ["sinc", "identity"])
@pytest.mark.parametrize("n", [129, 256, 300, 512])
def test_late_workgroups(gpu, monkeypatch, n, gram):
    from paper_2310_09200_amd import Context, StandardSynthesis
    print("case late workgroups, size", n, gram, flush=True)
    monkeypatch.setenv("BB_DEBUG_FILL", "1")
    monkeypatch.setenv("BB_DEBUG_TRD_LATE", "1")
    ctx = Context(0)
    g = np.random.default_rng(n)
    x = sims.disk_layout(n, 400.0 * np.sqrt(n), g, z_sigma_m=2.0)
    V = g.normal(size=(n, n)) + 1j * g.normal(size=(n, n))
    V = V + V.conj().T
    G = ref.gram(x, 2.0) if gram == "sinc" else np.eye(n)
    want = linalg.eigh(V, G.astype(np.complex128), eigvals_only=True)[::-1]
    s = StandardSynthesis(ctx, np.array([[0.0, 0.0, 1.0]]), 1, 1, n, n, gram=gram)
    for late in ("1", "0"):  # and the handle's own kernels after it
        monkeypatch.setenv("BB_DEBUG_TRD_LATE", late)
        _, lam, _, _ = s.prestep(x, 2.0, V, n, np.array([[-np.inf, np.inf]]))
        assert np.max(np.abs(lam.cpu().numpy() - want)) <= 1e-11 * max(1.0, n / 64) * np.max(np.abs(want))
    s.close()
    ctx.close()


@pytest.mark.parametrize("n", [20, 100, 200, 300])
def test_columns_whose_squares_underflow(gpu, n):
    """A matrix in two blocks with a coupling below the range of squares, and one that lies there whole (accepted; the
    solvers' own thresholds leave no accuracy there)."""
    from paper_2310_09200_amd import Context, StandardSynthesis
    print("case underflow, size", n, flush=True)
    ctx = Context(0)
    g = np.random.default_rng(n)
    x = sims.disk_layout(n, 400.0 * np.sqrt(n), g, z_sigma_m=2.0)
    V = g.normal(size=(n, n)) + 1j * g.normal(size=(n, n))
    V = V + V.conj().T
    k = n // 3
    V[:k, k:], V[k:, :k] = 1e-170j, -1e-170j
    V[:k, :k] = np.diag(np.arange(1.0, k + 1))
    s = StandardSynthesis(ctx, np.array([[0.0, 0.0, 1.0]]), 1, 1, n, n, gram="identity")
    want = linalg.eigh(V, eigvals_only=True)[::-1]
    _, lam, _, _ = s.prestep(x, 2.0, V, n, np.array([[-np.inf, np.inf]]))
    assert np.max(np.abs(lam.cpu().numpy() - want)) <= 1e-12 * max(1.0, n / 64) * np.max(np.abs(want))
    _, lam, _, _ = s.prestep(x, 2.0, V * 1e-160, n, np.array([[-np.inf, np.inf]]))
    assert np.all(np.isfinite(lam.cpu().numpy()))
    s.close()
    ctx.close()
