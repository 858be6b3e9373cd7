"""The stored ladder for up to 20 rows from half of each symmetric pair block (blocks of 4096 pairs and up): 1 to 20 rows, odd
and even, column blocks that end at different places (v = 91 to 113), against the ladder assembled from the DF factor, an
independent kernel that the other tests hold against the oracle.

Tolerance: 1e-11 of the largest element, as for the other FP64 products."""
import numpy as np
import pytest

import synth

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

import paper_2511_05897_amd as adc  # noqa: E402


def dev(x):
    return torch.as_tensor(np.ascontiguousarray(x), dtype=torch.float64, device="cuda")


@pytest.mark.parametrize("o,v", [(1, 91), (3, 92), (8, 95), (10, 91), (9, 101), (16, 100), (17, 96), (20, 113)])
def test_sigma_half_stream(o, v):
    eo, ev, B = synth.make_instance(o, v, 12, v + o, scale=0.3)
    stored = adc.Context(dev(eo), dev(ev), dev(B), 3)
    assembled = adc.Context(dev(eo), dev(ev), dev(B), 3, ladder=2)
    r = torch.as_tensor(np.random.default_rng(v).standard_normal((3, stored.N)), device="cuda")
    for nv in (1, 2, 3):
        a, b = stored.sigma(r[:nv].contiguous()), assembled.sigma(r[:nv].contiguous())
        assert float((a - b).abs().max()) <= 1e-11 * float(b.abs().max()), nv
    stored.close()
    assembled.close()
