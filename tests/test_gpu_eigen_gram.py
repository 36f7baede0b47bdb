"""Arrays whose Gram matrix is singular to rounding without two antennas in one place: the call answers as the library's
factorisation does (the sign that its last pivots round to), whichever solver runs first.  The arrays and answers are
those of rocSOLVER's one-call solver on them."""

import numpy as np
import pytest

import sims

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("kind, n, accepted", [("pair", 65, True), ("pair", 512, True), ("dense", 100, True),
                                               ("pair", 10, False), ("pair", 150, False), ("denser", 100, False)])
def test_gram_singular_to_rounding(gpu, kind, n, accepted):
    from paper_2310_09200_amd import BluebildError, Context, StandardSynthesis, _lib
    print("case Gram", kind, n, flush=True)
    ctx = Context(0)
    if kind == "pair":  # two antennas 1e-9 wavelengths apart
        g = np.random.default_rng(11 * n)
        x = sims.disk_layout(n, 400.0 * np.sqrt(n), g, z_sigma_m=2.0)
        x[-1] = x[n // 2] + np.array([2.0e-9, 0.0, 0.0])
    else:  # many antennas within a wavelength or two
        g = np.random.default_rng(n)
        x = sims.disk_layout(n, 2.0 if kind == "dense" else 1.0, g, z_sigma_m=0.1)
    V = g.standard_normal((n, n)) + 1j * g.standard_normal((n, n))
    V = (V + V.conj().T) / 2
    s = StandardSynthesis(ctx, np.array([[0.0, 0.0, 1.0]]), 1, 1, n, n)
    status = _lib.BB_OK
    try:
        _, lam, _, _ = s.prestep(x, 2.0, V, n, np.array([[-np.inf, np.inf]]))
        assert np.all(np.isfinite(lam.cpu().numpy()))
    except BluebildError as e:
        status = e.status
    s.close()
    ctx.close()
    assert status == (_lib.BB_OK if accepted else _lib.BB_ERR_NOT_POSDEF)
