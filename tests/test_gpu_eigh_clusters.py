"""Clustered spectra: off the diagonal a Jacobi sweep then converges linearly, and neither form of the eigensolver may take
that for the rounding floor.  Residual bound 5e-14 of the norm (the solver's threshold, an off-diagonal norm of 1e-15 to
3e-15 of it, and a few roundings of products with the matrix)."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

import paper_2511_05897_amd as adc  # noqa: E402


def spectrum(kind, n, rng):
    if kind == "multiple":  # one eigenvalue of multiplicity 3 n / 4 among a spread spectrum
        return np.concatenate([np.full(3 * n // 4, 1.0), rng.uniform(0.05, 3.0, n - 3 * n // 4)])
    if kind == "half":      # half of them within 1e-14 of each other
        return np.concatenate([1.0 + 1e-14 * rng.standard_normal(n // 2), rng.uniform(0.05, 3.0, n - n // 2)])
    return 1.0 + 1e-11 * rng.standard_normal(n)  # "all"


@pytest.mark.parametrize("kind", ["multiple", "half", "all"])
@pytest.mark.parametrize("n", [40, 64, 96, 97, 200, 600])
def test_clustered_spectrum(n, kind):
    rng = np.random.default_rng(n)
    lam = spectrum(kind, n, rng)
    Q, _ = np.linalg.qr(rng.standard_normal((n, n)))
    A = (Q * lam) @ Q.T
    A = 0.5 * (A + A.T)
    w, V = adc.adc3_eigh(torch.as_tensor(A, device="cuda"))
    w, V = w.cpu().numpy(), V.cpu().numpy()
    nrm = np.linalg.norm(A)
    assert np.linalg.norm(A @ V - V * w) <= 5e-14 * nrm
    assert np.abs(w - np.linalg.eigvalsh(A)).max() <= 1e-13 * nrm
    assert np.abs(V.T @ V - np.eye(n)).max() <= 1e-12
