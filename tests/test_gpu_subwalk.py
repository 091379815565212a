"""Sub-walks of the surrogate's training data: sample q is a function of (seed, q) alone, however many
samples share its wave (few: taken cooperatively one by one; many: side by side first), in static and
moving cells, with and without a step cap."""
import numpy as np
import pytest

from paper_1709_10187_amd import surrogate as sg

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("shift,cap", [(0.0, 1 << 30), (-0.2, 1 << 30), (-0.2, 37), (0.0, 64)])
def test_sample_does_not_depend_on_the_number_of_samples(shift, cap):
    m = sg.probe_medium(2e3, 4.7e-4, 0.9, shift, None if shift == 0.0 else 20.0, odd_bins=True)
    j = m.n_bins // 2
    dom = sg.Domain(x_core=1e9)
    big = sg.generate([m], 300000, dom, seed=5, max_steps=cap, bins=[j])
    bx, by, bs = (v.cpu().numpy() for v in (big.x, big.y, big.steps))
    assert np.all(bs <= cap) and (cap < 1 << 20 or len(bs) == 300000)
    for n in (1, 5, 64, 20001):
        print(f"[sub-walk] shift {shift} cap {cap} n {n}", flush=True)
        d = sg.generate([m], n, dom, seed=5, max_steps=cap, bins=[j])
        k = d.n   # rows cut by the cap are dropped, in order
        np.testing.assert_array_equal(d.x.cpu().numpy(), bx[:k])
        np.testing.assert_array_equal(d.y.cpu().numpy(), by[:k])
        np.testing.assert_array_equal(d.steps.cpu().numpy(), bs[:k])
