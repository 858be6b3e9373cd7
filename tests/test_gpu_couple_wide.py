"""The 1p <-> 2p1h coupling kernels at the widest virtual spaces they take (v up to 256 and just past it): the widest LDS slab
(v > 192) with rows filling it and not, odd v (element-aligned rows, through registers), and the separate products beyond; 1, 8 and 9
vectors (one and two copies of vector rows); against the oracle's ADC(2) sigma.

Tolerances as for the other sigma tests: 1e-11 of the largest element in FP64, 2e-5 with the FP32 copy of the block."""
import numpy as np
import pytest

import synth
from oracle.adc_cs import Problem

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

import paper_2511_05897_amd as adc  # noqa: E402


@pytest.mark.parametrize("o,v", [(1, 192), (1, 193), (2, 194), (1, 200), (1, 254), (1, 255), (2, 256), (1, 257), (1, 258)])
def test_wide_coupling(o, v):
    eo, ev, B = synth.make_instance(o, v, 6, v, scale=0.3)
    P = Problem(eo, ev, B)
    r = np.random.default_rng(v).standard_normal((9, P.dim()))
    ref = P.sigma(r, 2)
    d = lambda x: torch.as_tensor(np.ascontiguousarray(x), dtype=torch.float64, device="cuda")  # noqa: E731
    for prec, tol in ((0, 1e-11), (1, 2e-5)):
        ctx = adc.Context(d(eo), d(ev), d(B), 2, precision=prec)
        for nv in (1, 8, 9):
            out = ctx.sigma(d(r[:nv]), precision=prec).cpu().numpy()
            assert np.abs(out - ref[:nv]).max() <= tol * np.abs(ref[:nv]).max(), (prec, nv)
        ctx.close()
