"""Lanes of a wave that exchange values through LDS order them by wave_sync (a wavefront fence on either
side of the barrier): __builtin_amdgcn_wave_barrier alone orders no memory, so a lane could keep the value
that it stored itself in place of what the others added."""
import glob
import os
import re

import numpy as np
import pytest

from paper_1709_10187_amd import media

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
SYNC = re.compile(r'__builtin_amdgcn_fence\(__ATOMIC_RELEASE, "wavefront"\);\s*__builtin_amdgcn_wave_barrier\(\);\s*'
                  r'__builtin_amdgcn_fence\(__ATOMIC_ACQUIRE, "wavefront"\);')


def test_wave_barriers_stand_between_fences():
    for path in glob.glob(os.path.join(ROOT, "paper_1709_10187_amd", "csrc", "*")):
        src = re.sub(r"//[^\n]*", "", open(path).read())
        assert "__builtin_amdgcn_wave_barrier" not in SYNC.sub("", src), path


# many spatial leaks: most lanes of a block hold a face pair or lie past its end, and add nothing
LEAKY = {
    "slab_60x3": media.slab(3e3, 1e4, 60, 3, n_packets=400, tau_threshold=5.0),
    "sphere_40x5": media.sphere(2e3, 1e4, 40, 5, n_packets=400, tau_threshold=5.0),
    "moving_40x24": media.sphere(1e3, 1e4, 40, 24, x_max=9.0, v_max=60.0, n_packets=400, tau_threshold=5.0),
}


@pytest.mark.gpu
@pytest.mark.parametrize("weights", [False, True])
@pytest.mark.parametrize("name", list(LEAKY))
def test_residence_sums_where_few_lanes_add(name, weights):
    from paper_1709_10187_amd import rddmc
    n = LEAKY[name].n_cells_total
    m = LEAKY[name].replace(census=np.linspace(0.0, 6.0, 4), dust_abs=np.full(n, 0.05), dust_sca=np.full(n, 0.03),
                            flags=media.DUST_WEIGHT if weights else 0)
    out = []
    for lanes in (-1, 0):
        print(f"[wave sync] {name} weights {weights} tail_lanes {lanes}", flush=True)
        p = rddmc.Problem(m)
        p.run(seed=29, tail_lanes=lanes)
        out.append(p.results()[0])
    for k in ("census_bin", "census_path", "census_accel", "spectrum", "step_hist"):
        np.testing.assert_array_equal(getattr(out[0], k), getattr(out[1], k), err_msg=k)
    assert out[1].census_path.sum() > 0
