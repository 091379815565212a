"""Pure frequency-group batches take a walk of their own; a cloud's results do not depend on its batch,
so the same cloud beside a hybrid one (which the general hybrid walk takes) gives the same bits: slab
and shells, one cell, with dust, emission windows, several clouds, and a step cap."""
import numpy as np
import pytest

from paper_1709_10187_amd import media, rddmc

pytestmark = pytest.mark.gpu


def _grp(F, tau0, cells, bins, n, dust=0.0, **kw):
    m = F(tau0, 1e4, cells, bins, n_packets=n, tau_threshold=media.ALL_THIN).replace(flags=media.GROUP_MC, **kw)
    return m.replace(dust_abs=np.full(cells, dust), dust_sca=np.full(cells, 3 * dust)) if dust else m


CASES = {
    "slab": [_grp(media.slab, 800.0, 12, 64, 2000)],
    "sphere": [_grp(media.sphere, 500.0, 9, 50, 2000)],
    "one_cell": [_grp(media.slab, 30.0, 1, 33, 2000)],
    "one_bin": [_grp(media.sphere, 30.0, 4, 1, 500)],
    "dust": [_grp(media.slab, 500.0, 10, 40, 2000, dust=0.05)],
    "dusty_shells": [_grp(media.sphere, 300.0, 10, 40, 2000, dust=0.2, src_t=np.array([[0.1, 0.7]]))],
    "batch": [_grp(media.slab, 300.0, 7, 40, 700), _grp(media.slab, 200.0, 5, 21, 900, dust=0.1)],
}


@pytest.mark.parametrize("cap", [1 << 62, 97])
@pytest.mark.parametrize("name", list(CASES))
def test_alone_and_beside_a_hybrid_cloud(name, cap):
    meds = CASES[name]
    F = media.slab if meds[0].geometry == media.SLAB else media.sphere
    other = F(200.0, 1e4, 6, 24, n_packets=300, tau_threshold=5.0)
    print(f"[groups] {name} cap {cap}", flush=True)
    p = rddmc.Problem(meds)
    p.run(seed=3, max_steps=cap)
    q = rddmc.Problem(meds + [other])
    q.run(seed=3, max_steps=cap)
    for m, a, b in zip(meds, p.results(), q.results()):
        assert a.launched == m.n_packets == a.escaped + a.capped + a.absorbed
        for k in ("spectrum", "time_hist", "step_hist"):
            np.testing.assert_array_equal(getattr(a, k), getattr(b, k), err_msg=k)
        for k in ("steps_total", "steps_max", "mc_steps", "absorbed", "t_mean", "t_var"):
            assert getattr(a, k) == getattr(b, k), k
