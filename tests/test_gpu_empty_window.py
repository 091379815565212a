"""A cloud without window states (no sub-walk long enough for the exit kernel, no cell in the learned
surrogate's domain) is walked as without a surrogate, alone and beside a cloud that has a window, by the
lanes and cooperatively."""
import numpy as np
import pytest

from paper_1709_10187_amd import media, rddmc
from paper_1709_10187_amd import surrogate as sg

pytestmark = pytest.mark.gpu

MEDIA = {
    "slab": media.slab(1e4, 1e4, 12, 24, n_packets=3000),
    "leaky": media.slab(300.0, 1e4, 40, 9, n_packets=3000),
    "outflow": media.sphere(3e3, 1e4, 12, 32, v_max=60.0, n_packets=3000),
}


def _run(p, **kw):
    p.reset()
    p.run(seed=31, max_steps=50001, **kw)
    return p.results()


def _same(a, b):
    for k in ("spectrum", "time_hist", "step_hist"):
        np.testing.assert_array_equal(getattr(a, k), getattr(b, k), err_msg=k)
    for k in ("launched", "escaped", "capped", "steps_total", "steps_max", "t_mean", "t_var", "surrogate_calls"):
        assert getattr(a, k) == getattr(b, k), k


@pytest.mark.parametrize("tail", [0, -1])
@pytest.mark.parametrize("name", list(MEDIA))
def test_no_window_is_the_plain_walk(name, tail):
    p = rddmc.Problem(MEDIA[name])
    ref = _run(p, tail_lanes=tail)[0]
    print(f"[empty window] {name} tail_lanes {tail}", flush=True)
    ek = rddmc.ExitKernel(p, min_steps=1e15)
    assert ek.n_states == 0
    _same(_run(p, tail_lanes=tail, surrogate=ek.buffer)[0], ref)
    at = sg.Attached(p, rddmc.Mdn(max_batch=32, seed=1), sg.Domain(tau_min=1e14, tau_max=1e15))
    assert at.n_states == 0
    _same(_run(p, tail_lanes=tail, surrogate=at.buffer)[0], ref)


def test_empty_window_beside_another():
    thick, leaky = media.slab(1e6, 1e4, 12, 96, n_packets=2000), MEDIA["leaky"]
    both = rddmc.Problem([leaky, thick])
    print("[empty window] batch", flush=True)
    ek = rddmc.ExitKernel(both, min_steps=1e3)
    assert ek.windows[0][1] < ek.windows[0][0] and ek.windows[1][1] >= ek.windows[1][0]
    got = _run(both, surrogate=ek.buffer)
    assert got[0].surrogate_calls == 0 and got[1].surrogate_calls > 0
    _same(got[0], _run(rddmc.Problem([leaky]))[0])
