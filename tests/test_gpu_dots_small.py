"""The small inner-product kernel (row counts 1 to 16, vectors shorter than a step, ending on odd elements, and rows
aligned to 8 bytes only) through the solver that consists of it: Davidson roots against the dense matrix, and the
orthonormality of its vectors.

Tolerances: a root lies within its residual norm (conv, 1e-8) of an eigenvalue; orthonormality is kept to 1e-10 by the
second orthonormalisation pass, whose inner products are rounded at 1e-15."""
import numpy as np
import pytest

import synth

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

import paper_2511_05897_amd as adc  # noqa: E402


def dev(x):
    return torch.as_tensor(np.ascontiguousarray(x), dtype=torch.float64, device="cuda")


@pytest.mark.parametrize("nroots", [1, 2, 3, 4, 5, 8, 9])
@pytest.mark.parametrize("o,v", [(1, 4), (1, 16), (2, 16), (1, 23), (3, 21)])
def test_davidson_small_blocks(o, v, nroots):
    eo, ev, B = synth.make_instance(o, v, 9, 5 * v + o, scale=0.3)
    ctx = adc.Context(dev(eo), dev(ev), dev(B), 3, nroots=nroots)
    w = np.linalg.eigvalsh(ctx.dense().cpu().numpy())
    roots, vecs, _, _, status = ctx.davidson(nroots, 1e-8, want_vectors=True)
    assert status == 0
    assert np.abs(roots[:, None] - w[None, :]).min(axis=1).max() <= 1e-8
    V = vecs.cpu().numpy().reshape(nroots, -1)
    assert np.abs(V @ V.T - np.eye(nroots)).max() <= 1e-10
    ctx.close()
