"""Steps between refills from one to the largest the call accepts give the same bits in the 1D walks (the
count in pairs of steps, and twice it, stay in an int)."""
import numpy as np
import pytest

from paper_1709_10187_amd import media, rddmc

pytestmark = pytest.mark.gpu

CASES = {
    "static": media.slab(300.0, 1e4, 8, 16, n_packets=2000),
    "moving": media.sphere(300.0, 1e4, 8, 24, x_max=9.0, v_max=60.0, n_packets=2000),
    "hybrid": media.slab(300.0, 1e4, 12, 24, n_packets=1000, tau_threshold=10.0),
}


@pytest.mark.parametrize("chunk", [1, (1 << 31) - 2, (1 << 31) - 1])
@pytest.mark.parametrize("name", list(CASES))
def test_chunk_does_not_change_the_bits(name, chunk):
    print(f"[chunk] {name} {chunk}", flush=True)
    out = []
    for kw in ({}, {"chunk": chunk}):
        p = rddmc.Problem(CASES[name])
        p.run(seed=3, **kw)
        out.append(p.results()[0])
    for k in ("spectrum", "time_hist", "step_hist"):
        np.testing.assert_array_equal(getattr(out[0], k), getattr(out[1], k), err_msg=k)
    assert out[0].steps_total == out[1].steps_total and out[1].capped == 0
