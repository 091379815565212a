"""Clouds at rest whose cells differ in temperature: a leak between thick cells takes the frequency to the
neighbour's Doppler units, x' = x sqrt(T/T'), as in moving clouds.  The rates and the interface flags are
built for that image of the bin, so a walk that kept the bin met states without a record: in the media
below some thick states have a neighbour that is thin in the same bin and thick over the bin's image."""
import math

import numpy as np
import pytest

from oracle import chain, tables, walk, walk1dh, walk3d
from paper_1709_10187_amd import media, rddmc
from tests._stats import assert_spectrum_matches, compare_exact, compare_two_samples

_E = np.sort(np.concatenate([np.random.default_rng(3).uniform(-6.0, 6.0, 45), [-6.0, 0.0, 6.0]]))


def _steps(m):
    """Cells from 0.3 to 3.3 times the temperature, with the line-centre opacity ~ T^(-1/2)."""
    t = np.exp(1.2 * np.cos(np.arange(m.k0.size) * 1.9))
    return m.replace(temp=m.temp * t, k0=m.k0 / np.sqrt(t))


CASES = {
    "slab": _steps(media.slab(900.0, 1e4, 9, 48, x_max=6.0, tau_threshold=5.0)),
    "slab_other_grid": _steps(media.slab(900.0, 1e4, 9, 47, x_max=6.0, tau_threshold=5.0)).replace(bin_edges=_E),
    "sphere": _steps(media.sphere(900.0, 1e4, 9, 48, x_max=6.0, tau_threshold=5.0)),
    "cube": _steps(media.cube(n=4, seed=7, mean_tau_cell=30.0, sigma_v=0.0, n_bins=40, dv_bin=5.0, tau_threshold=5.0,
                              n_sources=2, packets_per_source=1, name="cube")),
}


def _run(m, n, **kw):
    print(f"[temperature steps] {m.name} packets={n} {kw}", flush=True)
    p = rddmc.Problem(m.with_packets(n))
    p.run(seed=3, **kw)
    return p.results()[0]


@pytest.mark.parametrize("name", sorted(CASES))
def test_media_have_neighbours_thin_in_the_same_bin(name):
    t = tables.build(CASES[name])
    assert any(t.nbr[c, f] >= 0 and not t.face_is_mc[c, j, f] and not t.thick[t.nbr[c, f], j]
               for c, j in np.argwhere(t.thick) for f in range(t.nf))


@pytest.mark.gpu
@pytest.mark.parametrize("name", sorted(CASES))
def test_hybrid_walk_matches_oracle_walker(name):
    m = CASES[name]
    ng, no = 1 << 16, 1 << 14
    g = _run(m, ng)
    o = (walk3d if m.geometry == media.CART3D else walk1dh).run(m.with_packets(no), n_packets=no, seed=5)
    assert g.escaped == ng and o.escaped == no and g.to_mc > 0
    assert_spectrum_matches(compare_two_samples(g.spectrum.ravel(), o.spectrum.ravel()))
    assert abs(g.t_mean - o.t_mean) < 4.5 * math.sqrt(g.t_var / ng + o.t_var / no)
    assert abs(g.steps_mean - o.steps_mean) < 4.5 * math.sqrt(o.steps_var * (1.0 / ng + 1.0 / no))


@pytest.mark.gpu
def test_pure_3d_walk_matches_exact_chain():
    m = media.cube(n=4, seed=7, mean_tau_cell=300.0, sigma_v=0.0, n_bins=16, dv_bin=25.0, tau_threshold=0.0,
                   n_sources=2, packets_per_source=1, name="cube_pure")
    m = m.replace(temp=1e4 * np.where(np.arange(64) % 3 == 0, 4.0, 1.0))
    n = 100000
    ref, g = chain.solve(m), _run(m, n)
    r = compare_exact(g.spectrum, ref.spectrum, n)
    assert_spectrum_matches(r, l1_max=max(0.01, 2.5 * r["expected_noise_L1"]))
    assert abs(g.steps_mean - ref.steps) < 4 * math.sqrt(ref.steps_var / n)
    assert abs(g.t_mean - ref.t_mean) < 4 * math.sqrt(ref.t_var / n)


_TWO = 1e4 * np.where(np.arange(9) % 3 == 0, 4.0, 1.0)
_EP = np.sort(np.concatenate([np.random.default_rng(5).uniform(-3.0, 3.0, 20), [-3.0, 3.0]]))
PURE = {
    "slab": media.slab(300.0, 1e4, 9, 24, x_max=3.0).replace(temp=_TWO),
    "slab_other_grid": media.slab(300.0, 1e4, 9, 21, x_max=3.0).replace(temp=_TWO, bin_edges=_EP),
    "sphere": media.sphere(500.0, 1e4, 9, 24, x_max=3.0).replace(temp=_TWO),
}


@pytest.mark.parametrize("name", sorted(PURE))
def test_pure_oracle_walker_matches_exact_chain(name):
    m, n = PURE[name], 10000
    ref, o = chain.solve(m), walk.run(m, n_packets=n, seed=3)
    r = compare_exact(o.spectrum, ref.spectrum, n)
    assert_spectrum_matches(r, l1_max=2.5 * r["expected_noise_L1"])
    assert abs(o.steps_mean - ref.steps) < 4 * math.sqrt(ref.steps_var / n)


@pytest.mark.gpu
@pytest.mark.parametrize("name", sorted(PURE))
def test_pure_1d_walk_matches_exact_chain(name):
    m, n = PURE[name], 100000
    ref, g = chain.solve(m), _run(m, n)
    assert g.escaped == n
    r = compare_exact(g.spectrum, ref.spectrum, n)
    assert_spectrum_matches(r, l1_max=max(0.01, 2.5 * r["expected_noise_L1"]))
    assert abs(g.steps_mean - ref.steps) < 4 * math.sqrt(ref.steps_var / n)
    assert abs(g.t_mean - ref.t_mean) < 4 * math.sqrt(ref.t_var / n)
    # lanes alone, and beside a cloud without steps: the same packets
    for meds, kw in (([m], dict(tail_lanes=-1)), ([m, media.slab(300.0, 1e4, 9, 24, x_max=3.0)
                                                   if m.geometry == media.SLAB else
                                                   media.sphere(500.0, 1e4, 9, 24, x_max=3.0)], {})):
        p = rddmc.Problem([q.with_packets(3000) for q in meds])
        p.run(seed=3, **kw)
        a, b = p.results()[0], _run(m, 3000)
        np.testing.assert_array_equal(a.spectrum, b.spectrum)
        assert (a.steps_total, a.t_mean) == (b.steps_total, b.t_mean)


@pytest.mark.gpu
@pytest.mark.parametrize("census", [False, True])
@pytest.mark.parametrize("name", sorted(CASES))
def test_cooperative_walk_gives_the_same_bits(name, census):
    m = CASES[name]
    if census:
        if m.geometry == media.CART3D:
            pytest.skip("census estimators are tallied on 1D grids")
        m = m.replace(census=np.linspace(0.0, 12.0, 6))
    # few packets: they are handed over early and walked in windows
    a, b = _run(m, 300, tail_lanes=0), _run(m, 300, tail_lanes=-1)
    for k in ("spectrum", "census_bin", "census_path", "census_accel"):
        if getattr(a, k) is not None:
            np.testing.assert_array_equal(getattr(a, k), getattr(b, k), err_msg=k)
    for k in ("escaped", "steps_total", "steps_max", "to_mc", "to_ddmc", "reflected", "mc_steps", "t_mean", "t_var"):
        assert getattr(a, k) == getattr(b, k), k
