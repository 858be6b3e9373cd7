"""The tuner's choice between one launch for both pair blocks of a small stored ladder and one launch each, kept in the cache
file: either choice is read back, not measured and appended again by the next process."""
import os
import subprocess
import sys

import pytest

pytestmark = pytest.mark.gpu

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CODE = """
import sys; sys.path.insert(0, %r)
import numpy as np, torch
import paper_2511_05897_amd as adc, synth
eo, ev, B = (torch.as_tensor(x, dtype=torch.float64, device="cuda") for x in synth.make_instance(3, 40, 60, 8, scale=0.5))
ctx = adc.Context(eo, ev, B, 3)
r = np.random.default_rng(3).standard_normal((2, 40 + 3 * 40 * 40))
np.save(sys.argv[1], ctx.sigma(torch.as_tensor(r, device="cuda")).cpu().numpy())
""" % ROOT


def run(cache, out):
    env = dict(os.environ, ADC3_TUNE_CACHE=str(cache))
    r = subprocess.run([sys.executable, "-c", CODE, str(out)], env=env, capture_output=True, text=True, timeout=100)
    assert r.returncode == 0, r.stderr[-2000:]


def test_either_choice_is_kept(tmp_path):
    import numpy as np
    cache = tmp_path / "tune.txt"
    run(cache, tmp_path / "a.npy")
    lines = cache.read_text().splitlines()
    at = [i for i, l in enumerate(lines) if " launches " in l]
    assert len(at) == 1 and lines[at[0]].split()[-1] in ("1", "2")
    ref = np.load(tmp_path / "a.npy")
    for choice in ("1", "2"):
        lines[at[0]] = " ".join(lines[at[0]].split()[:-1] + [choice])
        cache.write_text("\n".join(lines) + "\n")
        run(cache, tmp_path / "b.npy")
        assert cache.read_text().splitlines() == lines
        assert np.abs(np.load(tmp_path / "b.npy") - ref).max() <= 1e-11 * np.abs(ref).max()
