"""Loose clusters (eigenvalues within 1e-5 to 1e-10 of each other): every pair then takes a small rotation in the vectors'
correction against the input, and their squares add up over the cluster.  Evaluated in extended precision, with the bounds of
the spread spectra: V^T A V off its diagonal 12 eps ||A||_F, V^T V - I at most n eps / 2."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

import paper_2511_05897_amd as adc  # noqa: E402

EPS = np.finfo(np.float64).eps


@pytest.mark.parametrize("width", [1e-5, 1e-6, 1e-7, 1e-8, 1e-9, 1e-10])
@pytest.mark.parametrize("n", [97, 200, 400])
def test_loose_cluster(n, width):
    rng = np.random.default_rng(n)
    lam = 1.0 + width * rng.standard_normal(n)
    Q, _ = np.linalg.qr(rng.standard_normal((n, n)))
    A = (Q * lam) @ Q.T
    A = 0.5 * (A + A.T)
    _, V = adc.adc3_eigh(torch.as_tensor(A, device="cuda"))
    X = V.cpu().numpy().astype(np.longdouble)
    S = X.T @ (A.astype(np.longdouble) @ X)
    off = S - np.diag(np.diag(S))
    G = X.T @ X - np.eye(n)
    assert np.sqrt((off ** 2).sum()) <= 12 * EPS * np.linalg.norm(A)
    assert np.sqrt((G ** 2).sum()) <= 0.5 * n * EPS
