"""A solve that keeps v - 1 of an even number of virtuals, without NAF truncation, runs in the workspace queried for it
(its bases have odd row strides throughout, which the untruncated size has not)."""
import numpy as np
import pytest
import torch

import paper_2511_05897_amd as adc
import synth

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("lockstep", [0, 1, 2])
def test_odd_kept_count_in_the_queried_workspace(lockstep):
    o, v, X, nr = 2, 120, 360, 2
    eo, ev, B = synth.make_instance(o, v, X, 5, scale=0.1)
    d = lambda x: torch.as_tensor(x, dtype=torch.float64, device="cuda:0")  # noqa: E731
    opts = adc.adc3_default_opts()
    opts.lockstep = lockstep
    opts.fno_keep_frac = (v - 1) / v
    opts.fno_correction = 0
    roots, reps, st = adc.adc3_ea_solve(d(eo), d(ev), d(B), nr, 0.0, 0.0, 1e-8, opts)
    assert st == adc.ADC3_OK
    assert [r["nvir_kept"] for r in reps] == [v - 1] * nr and [r["naux_kept"] for r in reps] == [X] * nr
    # one virtual of the least occupation less: near the untruncated roots
    full, _, st = adc.adc3_ea_solve(d(eo), d(ev), d(B), nr, 0.0, 0.0, 1e-8)
    assert st == adc.ADC3_OK
    assert np.abs(roots - full).max() < 1e-3
