"""The tuner's candidates hold the automatic schedule and the automatic hand-over, so that a tuned schedule is
not worse than none."""
import inspect

import numpy as np
import pytest

from paper_1709_10187_amd import autotune, media, rddmc


def test_automatic_choices_are_candidates():
    assert (0, 0, 0) in list(autotune.default_candidates(256))
    assert 0 in inspect.signature(autotune.tune).parameters["tail_candidates"].default
    assert autotune.prefers_automatic(9.0, 0.96, 10.0, 1.0)
    assert not autotune.prefers_automatic(10.0, 1.0, 9.0, 1.0)
    assert not autotune.prefers_automatic(9.0, 0.9, 10.0, 1.0)


@pytest.mark.gpu
def test_tuned_schedule_is_the_automatic_one_or_no_slower_on_the_sample():
    m = media.slab(2e3, 1e4, 32, 64, n_packets=4000)
    p = rddmc.Problem(m)
    print("[autotune] 32 x 64 slab", flush=True)
    best = autotune.tune(p, sample_packets=4000, trial_steps=2000, use_cache=False, tail_packets_per_cloud=2000)
    assert {t["tail_lanes"] for t in best["tail_trials"]} == {0, 16, -1, 8, 32}
    assert any(t["block"] == t["grid"] == t["chunk"] == 0 for t in best["trials"])
    s = autotune.schedule(best)
    if s["grid"]:
        tuned = min(t["ms"] for t in best["tail_trials"])
        auto = next(t for t in best["trials"] if t["grid"] == 0)
        assert not autotune.prefers_automatic(best["automatic_ms"], auto["steps_per_s"], tuned, best["steps_per_s"])
    p.reset()
    p.run(seed=5, **s)
    q = rddmc.Problem(m)
    q.run(seed=5)
    np.testing.assert_array_equal(p.results()[0].spectrum, q.results()[0].spectrum)
