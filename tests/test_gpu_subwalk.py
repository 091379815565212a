"""Sub-walks of the surrogate's training data: sample q is a function of (seed, q) alone, however many
samples share its wave (few: taken cooperatively one by one; many: side by side first), in static and
moving cells, with and without a step cap."""
import numpy as np
import pytest

from paper_1709_10187_amd import rddmc
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


@pytest.mark.parametrize("n", [1, 4, 64, 300000])
def test_capped_rows_keep_the_entry_bin(n):
    """The rows of the C call itself, those the cap cut among them (face -1): x_out lies in the entry
    bin however many samples share a wave (up to four: cooperatively; 300 000: side by side), and the
    first rows are those of a single call.  x_out = S sinh(y1) with y1 in float32 (2^-24 relative, so
    1e-5 bin widths at |y1| < 12 and x < 100 bins)."""
    import torch
    cap = 40
    m = sg.probe_medium(2e6, 4.7e-4, 0.9, -0.2, 20.0, odd_bins=True)
    j = m.n_bins // 2 + 3
    b = rddmc.Batch([m])
    tables = torch.empty(rddmc.table_bytes(b), dtype=torch.uint8, device="cuda")
    rddmc.build_leakage(b, tables)

    def rows(k):
        print(f"[sub-walk] raw rows, n {k} cap {cap}", flush=True)
        c = np.zeros(k, dtype=np.int32)
        s = np.full(k, m.n_bins + j, dtype=np.int32)
        x = torch.empty((k, 16), dtype=torch.float32, device="cuda")
        y = torch.empty((k, 3), dtype=torch.float32, device="cuda")
        st = torch.empty(k, dtype=torch.int64, device="cuda")
        scratch = torch.empty(2 * k, dtype=torch.int32, device="cuda")
        P = rddmc.C.c_void_p
        rddmc._check(rddmc.load().rddmc_surrogate_samples(
            b.ref(), P(tables.data_ptr()), c.ctypes.data, s.ctypes.data, k, 5, cap, P(scratch.data_ptr()), 8 * k,
            P(x.data_ptr()), P(y.data_ptr()), P(st.data_ptr()), rddmc._stream(None)))
        return y.cpu().numpy(), st.cpu().numpy()

    y, st = rows(n)
    cut = y[:, 0] < 0
    assert cut.mean() > 0.9 and np.all(st[cut] == cap)
    a_tau = 4.7e-4 * 2e6
    x = np.cbrt(a_tau) * np.sinh(y[cut, 1].astype(np.float64))
    e = m.bin_edges
    w = e[j + 1] - e[j]
    assert np.all((x > e[j] - 1e-4 * w) & (x < e[j + 1] + 1e-4 * w))
    few, few_st = rows(min(n, 5))
    np.testing.assert_array_equal(few, y[:len(few)])
    np.testing.assert_array_equal(few_st, st[:len(few)])
