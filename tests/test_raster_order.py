"""sd_get_spikes gives (step, neuron) pairs in slice order, whatever the order
in which the blocks of a persistent launch recorded them and however the raster
is drained.  Host code, no device."""
from __future__ import annotations

import pytest

from host_hip import run


@pytest.mark.parametrize("cap", [1, 3, 7, 1000])
def test_slice_order(cap):
    run(f"""
    D = 4
    cfg = dict(W.tiny(model=0, n=128, k=10, seed=1, d_lo=D, d_hi=7), record_spikes=1)
    h = create(cfg)
    hip.host_record(1)

    def drain(limit=10 ** 9):
        out = []
        while len(out) < limit:
            st, ix, n = np.zeros({cap}, np.int64), np.zeros({cap}, np.uint32), C.c_int64()
            assert L.sd_get_spikes(h, C.c_void_p(st.ctypes.data), C.c_void_p(ix.ctypes.data),
                                   {cap}, C.byref(n)) == 0
            if n.value == 0:
                break
            out += list(zip(st[:n.value].tolist(), ix[:n.value].tolist()))
        return out

    assert L.sd_simulate_steps(h, 10 * D) == 0
    got = drain(7)  # in part, then more slices, then the rest
    assert L.sd_simulate_steps(h, 6 * D) == 0
    got += drain()
    assert drain() == []
    assert got == [(k * D, 64 * b) for k in range(16) for b in range(2)], got
    """)
