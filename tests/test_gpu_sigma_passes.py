"""The sigma pass's data passes, coupling kernels and shared ladder launch at the edges of their tiles: v around 16, 32,
64 and 128 (16 x 16 and 32 x 32 tile pairs, 64-row slabs, odd rows aligned to 8 bytes only), one occupied orbital, 1 to 16
vectors, aligned and odd vector strides, the assembled ladder, and tile offsets limited so that the two pair blocks' partial sums
no longer fit one launch; against the oracle.

Tolerance: 1e-11 of the largest element, as for the other FP64 intermediates.  FP32 coupling: 2e-5, the bound of the
reduced-precision sigma."""
import numpy as np
import pytest

import synth
from oracle.adc_cs import Problem

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

import paper_2511_05897_amd as adc  # noqa: E402


def dev(x):
    return torch.as_tensor(np.ascontiguousarray(x), dtype=torch.float64, device="cuda")


def err(a, b):
    return np.abs(a.detach().cpu().numpy() - b).max() / np.abs(b).max()


SIZES = [(1, 1, 2), (1, 2, 3), (3, 15, 8), (2, 16, 9), (1, 17, 5), (2, 31, 12), (3, 32, 7), (2, 33, 20), (2, 48, 11),
         (1, 64, 9), (2, 65, 10), (1, 66, 10), (1, 128, 8), (1, 130, 9)]


@pytest.mark.parametrize("o,v,X", SIZES)
def test_sigma_tile_edges(o, v, X):
    eo, ev, B = synth.make_instance(o, v, X, 7 * v + o, scale=0.3)
    P = Problem(eo, ev, B)
    r = np.random.default_rng(v).standard_normal((16, P.dim()))
    for level in (2, 3):
        ctx = adc.Context(dev(eo), dev(ev), dev(B), level)
        for nv in (1, 2, 5, 16):
            assert err(ctx.sigma(dev(r[:nv])), P.sigma(r[:nv], level)) <= 1e-11, (level, nv)
        ctx.close()
    ctx = adc.Context(dev(eo), dev(ev), dev(B), 3, ladder=2)
    assert err(ctx.sigma(dev(r[:3])), P.sigma(r[:3], 3)) <= 1e-11
    ctx.close()
    ctx = adc.Context(dev(eo), dev(ev), dev(B), 2, precision=1)
    assert err(ctx.sigma(dev(r[:3]), precision=1), P.sigma(r[:3], 2)) <= 2e-5
    ctx.close()


@pytest.mark.parametrize("rows", [64, 128, 512])
def test_sigma_limited_offsets(rows):
    """Tiles of at most `rows` rows of G within the offset limit: many K chunks in one launch, then one launch per block,
    then the row-major kernel, as the partial sums' room runs out."""
    o, v, X = 2, 60, 12
    eo, ev, B = synth.make_instance(o, v, X, 3, scale=0.3)
    P = Problem(eo, ev, B)
    r = np.random.default_rng(1).standard_normal((16, P.dim()))
    lp = (v * (v + 1) // 2 + 7) // 8 * 8
    try:
        adc.adc3_debug_ladder_offset_limit(8 * lp * rows)
        ctx = adc.Context(dev(eo), dev(ev), dev(B), 3)
        for nv in (1, 3, 9, 16):
            assert err(ctx.sigma(dev(r[:nv])), P.sigma(r[:nv], 3)) <= 1e-11, nv
        ctx.close()
    finally:
        adc.adc3_debug_ladder_offset_limit(0)
