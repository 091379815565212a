"""The surrogate buffer holds its header, the clouds' windows and one 512-byte record per window state, and
nothing that grows with the network's batch; the argument's range is checked as before."""
import ctypes as C

import pytest

from paper_1709_10187_amd import media, rddmc
from paper_1709_10187_amd import surrogate as sg


def _bytes(batch, max_batch):
    n, states = C.c_size_t(), C.c_uint64()
    rddmc._check(rddmc.load().rddmc_surrogate_bytes(batch.ref(), C.byref(sg.use_domain().cfg()), max_batch, C.byref(n),
                                                    C.byref(states)))
    return n.value, states.value


def test_buffer_is_header_windows_and_records():
    m = media.sphere(3e7, 1e4, 64, 256, x_max=80.0)
    for meds in ([m], [m, media.sphere(10.0, 1e4, 8, 16)]):
        b = rddmc.Batch(meds)
        size, states = _bytes(b, 32)
        assert states > 0 and size == 256 + 256 + 512 * states
        assert _bytes(b, 1) == _bytes(b, 1 << 20) == (size, states)
    for bad in (0, -5, (1 << 24) + 1):
        with pytest.raises(rddmc.RddmcError):
            _bytes(b, bad)
