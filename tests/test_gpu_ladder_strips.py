"""The k-major FP64 product at row counts that end in one or two 4-row strips (20, 36, 40, 52, 56, 68, 72, 84, 100, 104, 116,
120 rows and their neighbours, and several row tiles), through the ladder and particle-hole products of a sigma, against
the oracle.

Tolerance: 1e-11 of the largest element, as for the other FP64 products."""
import numpy as np
import pytest

import synth
from oracle.adc_cs import Problem

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

import paper_2511_05897_amd as adc  # noqa: E402


def dev(x):
    return torch.as_tensor(np.ascontiguousarray(x), dtype=torch.float64, device="cuda")


@pytest.mark.parametrize("o,v", [(4, 21), (5, 24), (7, 18), (9, 17), (13, 20)])
def test_sigma_row_strips(o, v):
    eo, ev, B = synth.make_instance(o, v, 30, 3 * v + o, scale=0.3)
    P = Problem(eo, ev, B)
    r = np.random.default_rng(o).standard_normal((16, P.dim()))
    ref = P.sigma(r, 3)
    ctx = adc.Context(dev(eo), dev(ev), dev(B), 3)
    for nv in range(1, 17):
        out = ctx.sigma(dev(r[:nv])).cpu().numpy()
        assert np.abs(out - ref[:nv]).max() <= 1e-11 * np.abs(ref[:nv]).max(), nv
    ctx.close()
