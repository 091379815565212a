"""The 3D walk's cooperative walk against its lane walk: the same packets with (tail_lanes = 0) and
without it (-1) give the same bits, in static and moving cubes, with fewer and more bins than a band
holds, on non-uniform bins, in thin and in purely diffusive cubes, in a batch, at a step cap, and with
too few export slots."""
import numpy as np
import pytest

from paper_1709_10187_amd import media, rddmc

pytestmark = pytest.mark.gpu

_E = np.sort(np.concatenate([np.random.default_rng(3).uniform(-30.0, 30.0, 48), [0.0]]))

CASES = {
    "moving": [media.cube(8, n_bins=64, dv_bin=60.0, n_sources=5, packets_per_source=400)],
    "static": [media.cube(8, n_bins=64, dv_bin=60.0, n_sources=5, packets_per_source=400, sigma_v=0.0)],
    "fine_bins": [media.cube(5, n_bins=200, dv_bin=5.0, n_sources=3, packets_per_source=100, mean_tau_cell=300.0)],
    "wide_bins": [media.cube(6, n_bins=9, dv_bin=100.0, n_sources=3, packets_per_source=300)],
    "other_grid": [media.cube(7, n_bins=48, n_sources=3, packets_per_source=300).replace(bin_edges=_E)],
    "thin": [media.cube(6, n_bins=32, dv_bin=60.0, mean_tau_cell=3.0, n_sources=3, packets_per_source=300)],
    "pure": [media.cube(5, n_bins=32, dv_bin=60.0, mean_tau_cell=50.0, n_sources=3, packets_per_source=200,
                        tau_threshold=0.0)],
    "batch": [media.cube(5, n_bins=32, dv_bin=60.0, n_sources=3, packets_per_source=300),
              media.cube(6, seed=9, n_bins=48, dv_bin=50.0, n_sources=2, packets_per_source=300)],
}


def _run(meds, slots=None, **kw):
    p = rddmc.Problem(meds)
    if slots is not None:
        p.work = p.work[:32 + 11 * slots]
    p.run(seed=17, **kw)
    return p.results()


def _same(a, b):
    for x, y in zip(a, b):
        for k in ("spectrum", "time_hist", "step_hist", "pixels"):
            np.testing.assert_array_equal(getattr(x, k), getattr(y, k), err_msg=k)
        for k in ("launched", "escaped", "capped", "steps_total", "steps_max", "to_mc", "to_ddmc", "reflected",
                  "mc_steps", "t_mean", "t_var"):
            assert getattr(x, k) == getattr(y, k), k


@pytest.mark.parametrize("name", list(CASES))
def test_cooperative_walk_gives_the_same_bits(name):
    meds = CASES[name]
    print(f"[3D tail] {name}", flush=True)
    ref = _run(meds, tail_lanes=-1)
    assert all(r.launched == m.n_packets == r.escaped + r.capped for r, m in zip(ref, meds))
    _same(ref, _run(meds))
    _same(_run(meds, tail_lanes=-1, max_steps=301), _run(meds, max_steps=301))


def test_few_export_slots():
    """Packets that find no slot are walked by their lanes."""
    meds = CASES["moving"]
    ref = _run(meds, tail_lanes=-1)
    for slots in (0, 1, 100):
        print(f"[3D tail] {slots} slots", flush=True)
        _same(ref, _run(meds, slots=slots))


@pytest.mark.parametrize("chunk", [1, 1000, (1 << 31) - 1])
def test_steps_between_refills_do_not_change_the_bits(chunk):
    """The hand-over rule counts the passes since a refill, up to the longest the call accepts."""
    meds = CASES["moving"]
    print(f"[3D tail] chunk {chunk}", flush=True)
    _same(_run(meds, tail_lanes=-1), _run(meds, chunk=chunk))


def test_batches_that_leak_or_scatter_stay_in_the_lanes():
    """No hand-over (counted in the work area) in a batch with a cloud that is diffusive in every state, and
    none from waves with many continuous-MC events; packets of thick clouds are handed over."""
    given = {}
    for name in ("pure", "thin", "moving"):
        p = rddmc.Problem(CASES[name])
        p.run(seed=17)
        given[name] = int(p.work[8])
    mixed = rddmc.Problem(CASES["moving"] + CASES["pure"])
    mixed.run(seed=17)
    print(f"[3D tail] handed over {given}", flush=True)
    assert given["pure"] == 0 and given["thin"] == 0 and int(mixed.work[8]) == 0
    assert given["moving"] > 0
