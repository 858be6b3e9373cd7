"""A reduced-precision phase whose new directions all lie in the subspace goes on in the next precision.

The factor couples virtuals 0 and 1 among themselves and everything else by 1e-10, so the doubles of that pair are an
invariant space of four up to 1e-10.  Started with four generic vectors of it (and a decoupled high one), the BF16 phase sees
a residual of the vectors' rounding, some 4e-2 and above its threshold of 5e-4, that lies in the subspace; the FP64 phase then
finds the lowest root of the four at once, with a residual near 1e-10.  Reference: the oracle's secular matrix, dense."""
import numpy as np
import pytest

from oracle.adc_cs import Problem

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

import paper_2511_05897_amd as adc  # noqa: E402


def test_directions_inside_the_subspace():
    o, v, X = 1, 8, 2
    eo, ev = np.array([-1.0]), np.linspace(0.1, 3.0, v)
    B = np.zeros((X, o + v, o + v))
    B[0, 1:3, 1:3] = [[5.0, 4.0], [4.0, 3.3]]  # a ladder of norm 70, nearly singular: the roots of the pair start near 1.2
    B[1, 1:3, 1:3] = [[0.2, 0.1], [0.1, -0.3]]
    B[:, 1, 3] = B[:, 3, 1] = 1e-10
    P = Problem(eo, ev, B)
    M = P.dense(3)
    pair = [v + a * v + b for a in (0, 1) for b in (0, 1)]
    rng = np.random.default_rng(3)
    guess = np.zeros((5, P.dim()))
    guess[:4, pair] = np.linalg.qr(rng.standard_normal((4, 4)))[0]
    guess[4, P.dim() - 1] = 1.0
    d = lambda x: torch.as_tensor(x, dtype=torch.float64, device="cuda")  # noqa: E731
    ctx = adc.Context(d(eo), d(ev), d(B), 3, nroots=1, precision=2)
    w, _, rn, it, st = ctx.davidson(1, 1e-8, precision=2, guess=d(guess))
    lowest = np.linalg.eigvalsh(M[np.ix_(pair, pair)])[0]
    assert st == adc.ADC3_OK and rn[0] <= 1e-8
    assert abs(w[0] - lowest) <= 1e-8
