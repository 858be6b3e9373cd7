"""The workspace plan of a truncating solve covers every kept count, odd ones among them (no GPU needed): a basis of
v - 1 virtuals takes copies with even row strides that one of v (even) does not."""
import os

import pytest

import paper_2511_05897_amd as adc

# o, v, X, roots
SHAPES = [(4, 120, 360, 5), (20, 200, 600, 5), (20, 199, 600, 3), (14, 120, 360, 4), (6, 110, 330, 2), (9, 83, 249, 3),
          (3, 66, 67, 2), (1, 65, 9, 1), (2, 7, 15, 2), (1, 2, 1, 1), (30, 400, 1200, 2)]


@pytest.fixture(scope="module", autouse=True)
def lib():
    if not os.path.exists(adc.LIB_PATH):
        pytest.skip("library not built")
    return adc.load()


@pytest.mark.parametrize("lockstep", [0, 1, 2])
@pytest.mark.parametrize("chunk", [None, 1 << 22])
@pytest.mark.parametrize("shape", SHAPES)
def test_plan_covers_every_kept_count(lib, shape, chunk, lockstep):
    o, v, X, nr = shape
    opts = adc.adc3_default_opts()
    opts.lockstep = lockstep
    before = lib.adc3_set_chunk_elems(0)
    try:
        if chunk:
            lib.adc3_set_chunk_elems(chunk)
        plan = adc.adc3_ea_solve_workspace_bytes(o, v, X, nr, opts)
        assert plan > 0
        for vk in sorted({v, v - 1, v - 2, v - 3} | set(range(1, v, max(1, v // 16)))):
            if vk < 1 or nr > vk + o * vk * vk:
                continue
            for xk, naf in ((0, False), (0, True), (max(1, X - 1), True)):
                need = adc.adc3_debug_kept_workspace_bytes(o, v, X, nr, vk, xk, naf, opts)
                assert 0 < need <= plan, (vk, xk, naf)
    finally:
        lib.adc3_set_chunk_elems(before)
