"""The cooperative tail walk's mixed blocks (windows of cells x bins) against the lane walk: the same
packets walked by lanes alone, with the automatic hand-over and with everything handed over give the
same bits, at grid sizes where a window is cut by the grid (one cell, one bin, fewer or more than a
window holds), in static and moving media, on non-uniform bins, near the step cap and with the exact
exit kernel."""
import numpy as np
import pytest

from paper_1709_10187_amd import media, rddmc

pytestmark = pytest.mark.gpu

_E = np.sort(np.concatenate([np.random.default_rng(3).uniform(-9.0, 9.0, 40), [0.0]]))

CASES = {
    "slab_8x16": (media.slab(300.0, 1e4, 8, 16, n_packets=6000), {}),
    "slab_1x7": (media.slab(50.0, 1e4, 1, 7, n_packets=2000), {}),
    "slab_9x1": (media.slab(50.0, 1e4, 9, 1, n_packets=2000), {}),
    "slab_100x3": (media.slab(1e3, 1e4, 100, 3, n_packets=1000), {}),
    "slab_3x100": (media.slab(1e3, 1e4, 3, 100, n_packets=1000), {}),
    "slab_nonuniform": (media.slab(1e3, 1e4, 15, 40, n_packets=1500).replace(bin_edges=_E), {}),
    "sphere_static": (media.sphere(2e3, 1e4, 40, 50, n_packets=1500), {}),
    "sphere_moving": (media.sphere(1e3, 1e4, 24, 64, x_max=8.0, v_max=60.0, n_packets=1500), {}),
    "sphere_fast": (media.sphere(300.0, 3e2, 17, 33, x_max=60.0, v_max=150.0, n_packets=1000), {}),
    "sphere_moving_nonuniform": (media.sphere(300.0, 1e4, 15, 40, v_max=50.0, n_packets=1000).replace(bin_edges=_E), {}),
    "cap_odd": (media.sphere(2e3, 1e4, 24, 64, x_max=8.0, v_max=60.0, n_packets=2000), {"max_steps": 3333}),
    "cap_short": (media.slab(300.0, 1e4, 8, 16, n_packets=2000), {"max_steps": 67}),
    "slab_3x300": (media.slab(1e3, 1e4, 3, 300, n_packets=600), {}),        # bands move, windows at their edges
    "slab_2x64": (media.slab(1e3, 1e4, 2, 64, n_packets=600), {}),          # one band covers the grid
    "slab_2x31": (media.slab(1e3, 1e4, 2, 31, n_packets=600), {}),          # a window and one bin
    "sphere_moving_wide": (media.sphere(1e3, 1e4, 3, 200, v_max=5.0, n_packets=600), {}),
    "grid_ends_in_the_core": (media.slab(1e3, 1e4, 4, 101, x_max=2.0, n_packets=600), {"max_steps": 20001}),
    "cap_in_block": (media.slab(1e4, 1e4, 3, 300, n_packets=600), {"max_steps": 1001}),
    "cap_in_block_moving": (media.sphere(1e4, 1e4, 3, 200, v_max=5.0, n_packets=600), {"max_steps": 130}),
    "several_waves_per_simd": (media.slab(20.0, 1e4, 8, 16, n_packets=(1 << 18) + 5), {}),
    "one_wave_per_simd": (media.slab(50.0, 1e4, 8, 16, n_packets=(1 << 16) - 3), {}),
    "exit_kernel": (media.sphere(1e5, 1e4, 32, 64, n_packets=2000), {"exit": True}),
    "exit_kernel_moving": (media.sphere(1e5, 1e4, 32, 64, x_max=40.0, v_max=50.0, n_packets=2000), {"exit": True}),
    "exit_kernel_wide": (media.sphere(1e5, 1e4, 16, 300, n_packets=600), {"exit": True}),
    "exit_kernel_cap": (media.sphere(1e5, 1e4, 32, 64, n_packets=2000), {"exit": True, "max_steps": 301}),
}


@pytest.mark.parametrize("name", list(CASES))
def test_tail_modes_give_the_same_bits(name):
    m, kw = CASES[name]
    kw = dict(kw)
    p = rddmc.Problem(m)
    if kw.pop("exit", False):
        kw["surrogate"] = rddmc.ExitKernel(p).buffer
    out = []
    for tail in (-1, 0, 64):
        print(f"[tail] {name} tail_lanes={tail}", flush=True)
        p.reset()
        p.run(seed=11, tail_lanes=tail, **kw)
        r = p.results()[0]
        assert r.launched == m.n_packets == r.escaped + r.capped
        out.append(r)
    for r in out[1:]:
        for k in ("spectrum", "time_hist", "step_hist"):
            np.testing.assert_array_equal(getattr(r, k), getattr(out[0], k))
        assert (r.steps_total, r.steps_max, r.t_mean, r.t_var, r.surrogate_calls) == (
            out[0].steps_total, out[0].steps_max, out[0].t_mean, out[0].t_var, out[0].surrogate_calls)
