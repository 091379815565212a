"""Exact-law training samples at grids around the 64 bins that a wave holds at a time, against the
exact single-cell exit law O5: face split, exit bins, mean time."""
import math

import numpy as np
import pytest

from oracle import exitlaw
from oracle import tables as tb
from paper_1709_10187_amd import surrogate as sg
from tests._stats import assert_spectrum_matches, compare_exact
from tests.test_gpu_surrogate import DOM, _coarse, _exit_hist, _scale

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("nb", [16, 63, 64, 65, 66, 130])
def test_samples_on_partial_and_whole_chunks(nb):
    m = sg.probe_medium(5.0e5, 1.0e-3, 0.8, 0.0, 12.0, False)
    m = m.replace(bin_edges=np.linspace(-9.0, 9.0, nb + 1))
    n = 20000
    print(f"[exit samples] {nb} bins", flush=True)
    d = sg.generate_exact([m], n, DOM, seed=9, bins_per_probe=1)
    x, y = d.x.cpu().numpy(), d.y.cpu().numpy().astype(np.float64)
    e = np.asarray(m.bin_edges)
    j = int(np.argmin(np.abs(0.5 * (e[:-1] + e[1:]) - 3.0 * float(x[0, 2]))))
    ex = exitlaw.exit_law(tb.build(m), 1, j)
    H = _exit_hist(m, y[:, 0], _scale(m) * np.sinh(y[:, 1]))
    p0 = ex.prob[0].sum()
    assert abs(H[0].sum() - p0) < 4.5 * math.sqrt(p0 * (1 - p0) / n)
    assert_spectrum_matches(compare_exact(np.round(_coarse(H) * n).ravel(), _coarse(ex.prob).ravel(), n))
    dt = np.exp(y[:, 2]) * (m.faces[0][2] - m.faces[0][1])
    assert abs(dt.mean() - ex.t_mean) < 4.5 * math.sqrt(ex.t_var / n)
