"""The hybrid 1D walk's cooperative walk against its lane walk: the same packets with (tail_lanes = 0)
and without it (-1) give the same bits, for every kind of state and estimator it carries: continuous-MC
and group states, dust by absorption and by weights, census estimators, emission windows, moving media
on uniform and other grids, windows cut by the grid, the step cap, and a work area with too few export
slots."""
import numpy as np
import pytest

from paper_1709_10187_amd import media, rddmc

pytestmark = pytest.mark.gpu

_E = np.sort(np.concatenate([np.random.default_rng(3).uniform(-9.0, 9.0, 40), [0.0]]))
_D = dict(dust_abs=np.full(24, 0.05), dust_sca=np.full(24, 0.03))
_C = np.linspace(0.0, 4.0, 7)


def _cases():
    out = {}
    for name, F in (("slab", media.slab), ("sphere", media.sphere)):
        out[name + "_mc"] = F(1e3, 1e4, 24, 40, n_packets=1500, tau_threshold=10.0)
        out[name + "_groups"] = F(1e3, 1e4, 16, 64, n_packets=1500, tau_threshold=10.0).replace(flags=media.GROUP_MC)
        out[name + "_dust"] = F(1e3, 1e4, 24, 40, n_packets=1500, tau_threshold=10.0).replace(**_D)
        out[name + "_weights"] = F(1e3, 1e4, 24, 40, n_packets=1000, tau_threshold=10.0).replace(
            flags=media.DUST_WEIGHT, **_D)
        out[name + "_census"] = F(1e3, 1e4, 24, 40, n_packets=1500, tau_threshold=10.0).replace(census=_C, **_D)
        out[name + "_census_weights"] = F(1e3, 1e4, 24, 40, n_packets=1000, tau_threshold=10.0).replace(
            census=_C, flags=media.DUST_WEIGHT, **_D)
        out[name + "_census_pure"] = F(1e3, 1e4, 24, 40, n_packets=1500).replace(census=_C,
                                                                                src_t=np.array([[0.0, 1.0]]))
    out["slab_1x9"] = media.slab(60.0, 1e4, 1, 9, n_packets=1000, tau_threshold=10.0)
    out["slab_3x100"] = media.slab(300.0, 1e4, 3, 100, n_packets=500, tau_threshold=10.0)
    out["slab_100x3"] = media.slab(3e3, 1e4, 100, 3, n_packets=500, tau_threshold=5.0)
    out["sphere_moving"] = media.sphere(2e3, 1e4, 24, 64, x_max=9.0, v_max=60.0, n_packets=1000, tau_threshold=10.0)
    out["sphere_moving_census"] = out["sphere_moving"].replace(census=_C)
    out["sphere_moving_other_grid"] = media.sphere(1e3, 1e4, 15, 40, v_max=50.0, n_packets=1000,
                                                   tau_threshold=5.0).replace(bin_edges=_E)
    out["slab_moving"] = media.slab(1e3, 1e4, 24, 64, x_max=9.0, vel=np.linspace(-40.0, 40.0, 24), n_packets=1000,
                                    tau_threshold=10.0)
    return out


CASES = _cases()


def _run(m, slots=None, **kw):
    p = rddmc.Problem(m)
    if slots is not None:
        p.work = p.work[:32 + 13 * slots]
    p.run(seed=13, **kw)
    return p.results()[0]


def _same(a, b):
    for k in ("spectrum", "time_hist", "step_hist", "census_bin", "census_path", "census_accel", "spectrum_w",
              "spectrum_w2"):
        if getattr(a, k) is not None:
            np.testing.assert_array_equal(getattr(a, k), getattr(b, k), err_msg=k)
    for k in ("launched", "escaped", "capped", "absorbed", "steps_total", "steps_max", "to_mc", "to_ddmc", "reflected",
              "mc_steps", "t_mean", "t_var", "escaped_w", "t_mean_w", "t_var_w"):
        assert getattr(a, k) == getattr(b, k), k


@pytest.mark.parametrize("name", list(CASES))
def test_cooperative_walk_gives_the_same_bits(name):
    m = CASES[name]
    print(f"[hybrid tail] {name}", flush=True)
    ref = _run(m, tail_lanes=-1)
    assert ref.launched == m.n_packets == ref.escaped + ref.capped + ref.absorbed
    _same(ref, _run(m))
    _same(_run(m, tail_lanes=-1, max_steps=301), _run(m, max_steps=301))


def test_few_export_slots():
    """Packets that find no slot are walked by their lanes."""
    m = CASES["sphere_census"]
    ref = _run(m, tail_lanes=-1)
    for slots in (0, 1, 100):
        print(f"[hybrid tail] {slots} slots", flush=True)
        _same(ref, _run(m, slots=slots))
