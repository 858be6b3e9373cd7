"""Eigenvectors of the block eigensolver (n > 96) against the input matrix, evaluated in extended precision: the rotations'
accumulated rounding is corrected once, so what is left is the rounding of a few products with the input.

Bounds: V^T A V off its diagonal 12 eps ||A||_F (the residual's rounding: about eps times the norm of A V, a few times
over), V^T V - I at most n eps / 2 in the Frobenius norm (the storage's and the Gram matrix's rounding, about sqrt(n) eps).
Close pairs (a gap of 1e-6, where an error of eps in V^T A V shows as 1e-10 in the vectors) are part of each spectrum."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

import paper_2511_05897_amd as adc  # noqa: E402

EPS = np.finfo(np.float64).eps


def spectrum_matrix(n, seed):
    rng = np.random.default_rng(seed)
    lam = rng.uniform(0.05, 3.0, n)
    lam[1] = lam[0] + 1e-6
    Q, _ = np.linalg.qr(rng.standard_normal((n, n)))
    A = (Q * lam) @ Q.T
    return 0.5 * (A + A.T)


def check(A, w, V):
    n = len(A)
    X = V.astype(np.longdouble)
    S = X.T @ (A.astype(np.longdouble) @ X)
    off = S - np.diag(np.diag(S))
    assert np.sqrt((off ** 2).sum()) <= 12 * EPS * np.linalg.norm(A)
    G = X.T @ X - np.eye(n)
    assert np.sqrt((G ** 2).sum()) <= 0.5 * n * EPS
    assert np.abs(w - np.linalg.eigvalsh(A)).max() <= 1e-14 * np.linalg.norm(A)


@pytest.mark.parametrize("n", [97, 113, 200, 333, 600])
def test_vectors_to_the_rounding_of_the_input(n):
    A = spectrum_matrix(n, n)
    w, V = adc.adc3_eigh(torch.as_tensor(A, device="cuda"))
    check(A, w.cpu().numpy(), V.cpu().numpy())


def test_vectors_of_a_batch():
    A = np.stack([spectrum_matrix(130, 7 + b) for b in range(3)])
    w, V = adc.adc3_eigh_batched(torch.as_tensor(A, device="cuda"))
    for b in range(3):
        check(A[b], w[b].cpu().numpy(), V[b].cpu().numpy())
