"""Setup products of more than 1024 tiles (dealt to the XCDs in patches; row strips that do and do not fill a patch) against the
same context built in chunks of a few virtuals, whose small products the other tests hold against the oracle.

Tolerance: 1e-11 of the largest element, as for the other FP64 intermediates."""
import numpy as np
import pytest

import synth

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

import paper_2511_05897_amd as adc  # noqa: E402


def dev(x):
    return torch.as_tensor(np.ascontiguousarray(x), dtype=torch.float64, device="cuda")


@pytest.mark.parametrize("o,v", [(10, 121), (12, 128), (20, 110)])
def test_setup_patched_tiles(o, v):
    eo, ev, B = synth.make_instance(o, v, 20, v, scale=0.3)
    whole = adc.Context(dev(eo), dev(ev), dev(B), 3)
    u = whole.intermediate(1).clone()
    whole.close()
    old = adc.adc3_set_chunk_elems(0)
    try:
        adc.adc3_set_chunk_elems(o * v * v * 7)
        parts = adc.Context(dev(eo), dev(ev), dev(B), 3)
        w = parts.intermediate(1)
        assert float((u - w).abs().max()) <= 1e-11 * float(w.abs().max())
        parts.close()
    finally:
        adc.adc3_set_chunk_elems(old)
