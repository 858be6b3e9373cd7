"""The eigensolver at the edges of its forms (adc3_eigh): thread counts of the one-workgroup form (a thread per
2x2 block up to n = 64, three above), odd orders (a padding row and column), and for n > 96 a last block of
1, 15 and 16 rows with even and odd block counts; and matrices scaled far from 1.

Tolerances as for the eigensolver's other tests: rounding in the matrix norm."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

import paper_2511_05897_amd as adc  # noqa: E402


@pytest.mark.parametrize("scale", [1.0, 1e-100, 1e100])
@pytest.mark.parametrize("n", [3, 32, 33, 44, 45, 64, 65, 95, 98, 111, 112, 113, 127, 128, 129, 161])
def test_eigh_edges(n, scale):
    rng = np.random.default_rng(n)
    A = rng.standard_normal((n, n))
    A = 0.5 * (A + A.T) * scale
    w, V = adc.adc3_eigh(torch.as_tensor(A, device="cuda"))
    w, V = w.cpu().numpy(), V.cpu().numpy()
    nrm = np.linalg.norm(A / scale) * scale
    assert np.all(np.diff(w) >= 0)
    assert np.abs(w - np.linalg.eigvalsh(A / scale) * scale).max() <= 1e-12 * nrm
    assert np.abs(V.T @ V - np.eye(n)).max() <= 1e-12
    assert np.abs(A @ V - V * w).max() <= 1e-11 * nrm
    assert np.all(V[np.argmax(np.abs(V), axis=0), np.arange(n)] > 0)
