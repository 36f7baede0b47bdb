"""GPU pre-step eigenproblem V a = lambda G a against LAPACK in 64 bits, at the sizes where its kernels change
(panels of 64, one or several workgroups, the library beyond 512) and for degenerate inputs.

Tolerances.  Eigenvalues: FP64 backward error of reduction and tridiagonalisation, a few n eps of the largest
times the conditioning of G: 1e-12 max |lambda| cond(G) n / 64.  Eigenvectors leave as complex64 (2^-24 a component):
a column of norm |a| is off by 2^-23 |a| at most, so ||V a - lambda G a|| <= 2^-22 (||V|| + |lambda| ||G||) |a| and
|a^H G a' - delta| <= 2^-21 ||G|| |a| |a'|; both beside an FP64 error of the size of the eigenvalues' own.
"""

import numpy as np
import pytest
import torch
from scipy import linalg

import oracle as ref
import sims

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def ctx(gpu):
    from paper_2310_09200_amd import Context
    return Context(0)


def prestep(ctx, x, wl, V, gram="sinc", n_eig=None):
    from paper_2310_09200_amd import StandardSynthesis
    n = x.shape[0]
    s = StandardSynthesis(ctx, np.array([[0.0, 0.0, 1.0]]), 1, 1, n, n, gram=gram)
    W, lam, _, _ = s.prestep(x, wl, V, n_eig or n, np.array([[-np.inf, np.inf]]))
    out = W.cpu().numpy().astype(np.complex128), lam.cpu().numpy()
    s.close()
    return out


def check(ctx, x, wl, V, gram="sinc"):
    n = x.shape[0]
    G = ref.gram(x, wl).astype(np.complex128) if gram == "sinc" else np.eye(n, dtype=np.complex128)
    want = linalg.eigh(V, G, eigvals_only=True)[::-1]
    W, lam = prestep(ctx, x, wl, V, gram)
    top = max(np.abs(want).max(), 1e-300)
    ev = np.linalg.eigvalsh(G)
    f64 = 1e-12 * ev[-1] / ev[0] * max(1.0, n / 64)
    print("n", n, gram, "eigenvalues off by", np.abs(lam - want).max() / top, "allowed", f64, flush=True)
    assert np.all(np.diff(lam) <= 0) and np.abs(lam - want).max() <= f64 * top
    norm = np.linalg.norm(W, axis=0)
    res = np.linalg.norm(V @ W - (G @ W) * lam, axis=0)
    nv, ng = np.linalg.norm(V, 2), ev[-1]
    assert np.all(res <= (2.0**-22 + f64) * (nv + top * ng) * norm)
    orth = np.abs(W.conj().T @ G @ W - np.eye(n))
    assert np.all(orth <= (2.0**-21 + f64) * ng * norm[:, None] * norm[None, :])


def layout(n, seed):
    g = np.random.default_rng(seed)
    return sims.disk_layout(n, 400.0 * np.sqrt(n), g, z_sigma_m=2.0), g


def hermitian(n, g):
    A = g.standard_normal((n, n)) + 1j * g.standard_normal((n, n))
    return (A + A.conj().T) / 2


@pytest.mark.parametrize("gram", ["sinc", "identity"])
@pytest.mark.parametrize("n", [1, 2, 3, 5, 63, 64, 65, 127, 128, 129, 200, 255, 256, 257, 511, 512, 513])
def test_sizes(ctx, n, gram):
    print("case size", n, gram, flush=True)
    x, g = layout(n, n)
    check(ctx, x, 2.0, hermitian(n, g), gram)


@pytest.mark.parametrize("n", [20, 64, 130, 300])
@pytest.mark.parametrize("kind", ["zero", "diagonal", "tridiagonal", "rank2", "real", "scaled"])
def test_degenerate(ctx, n, kind):
    """No reflector at all, equal eigenvalues, one that is already tridiagonal, real and badly scaled matrices."""
    print("case", kind, n, flush=True)
    x, g = layout(n, 7 * n)
    V = hermitian(n, g)
    if kind == "zero":
        V = np.zeros_like(V)
    elif kind == "diagonal":
        V = np.diag(np.repeat([3.0, -1.0], [n - n // 2, n // 2])).astype(np.complex128)
    elif kind == "tridiagonal":
        V = np.triu(np.tril(V, 1), -1)
    elif kind == "rank2":
        u = V[:, :2]
        V = u @ u.conj().T
        V = (V + V.conj().T) / 2
    elif kind == "real":
        V = V.real.astype(np.complex128)
    else:
        s = 10.0 ** g.uniform(-6, 0, n)
        V = s[:, None] * V * s[None, :]
        V = (V + V.conj().T) / 2
    check(ctx, x, 2.0, V, "identity")
    check(ctx, x, 2.0, V)


@pytest.mark.parametrize("n", [3, 64, 65, 150, 512])
def test_singular_gram_is_refused(ctx, n):
    """Two antennas in one place: the Cholesky factorisation fails, also in a later panel."""
    from paper_2310_09200_amd import BluebildError, _lib
    print("case singular", n, flush=True)
    x, g = layout(n, 11 * n)
    x[-1] = x[n // 2]
    with pytest.raises(BluebildError) as e:
        prestep(ctx, x, 2.0, hermitian(n, g))
    assert e.value.status == _lib.BB_ERR_NOT_POSDEF


def test_repeated_calls_are_bitwise_equal(ctx):
    for n in (64, 300):
        print("case repeat", n, flush=True)
        x, g = layout(n, 13)
        V = hermitian(n, g)
        a, b = prestep(ctx, x, 2.0, V), prestep(ctx, x, 2.0, V)
        assert np.array_equal(a[0], b[0]) and np.array_equal(a[1], b[1])
