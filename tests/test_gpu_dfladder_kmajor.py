"""The FP64 assembled ladder on its k-major kernel: even and odd v around the tile edges (the padded factor copy),
row counts that leave short row and column tiles, one or several chunks of auxiliary functions and K chunks of the
second product (workspace fractions), against the contraction in numpy.

Tolerance: 1e-12 of the largest element (FP64 sums of X v^2 terms in another order)."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

import paper_2511_05897_amd as adc  # noqa: E402


@pytest.mark.parametrize("frac", [1.0, 0.4])
@pytest.mark.parametrize("M,v,X", [(7, 48, 31), (5, 61, 30), (3, 64, 90), (8, 127, 17), (4, 128, 12), (5, 129, 21),
                                   (1, 130, 33), (2, 255, 9)])
def test_assembled_ladder_k_major(M, v, X, frac):
    rng = np.random.default_rng(1000 * v + M)
    B = rng.standard_normal((X, v, v))
    B = 0.5 * (B + B.transpose(0, 2, 1))
    Z = rng.standard_normal((M, v, v))
    ref = np.zeros_like(Z)
    for Q in range(X):
        ref += B[Q] @ Z @ B[Q]
    lo = adc.adc3_ladder_workspace_bytes(v, X, M, 0)
    C = adc.adc3_ladder_apply(torch.as_tensor(B, device="cuda"), torch.as_tensor(Z, device="cuda"),
                              workspace_bytes=int(lo * (1 + frac * (X - 1))) + 512)
    torch.cuda.synchronize()
    assert np.abs(C.cpu().numpy() - ref).max() <= 1e-12 * np.abs(ref).max()
