"""A persistent launch that ends early has advanced its net part of the way.
Where nobody asked for the launch, the calls that read the net back say so and
those that advance it refuse, until a checkpoint is loaded; where it was asked
for, the overflow flags tell, as documented.  Host code, no device."""
from __future__ import annotations

from host_hip import run

SETUP = """
    OVERFLOW = -4
    cfg = dict(W.tiny(model=1, n=100, k=10, seed=1, d_lo=2, d_hi=3), record_spikes=1)
    h = create(cfg)
    D = 2
    n = C.c_size_t()
    assert L.sd_save_state(h, None, 0, C.byref(n)) == 0
    saved = C.create_string_buffer(n.value)
    assert L.sd_save_state(h, saved, n.value, C.byref(n)) == 0

    ring = np.zeros((4, 100), np.float32)
    st = sdeliver.sd_stats()
    m, t0 = C.c_int64(), C.c_int64()
    READS = dict(
        state=lambda: read(h, 100)[0],
        none=lambda: L.sd_read_state(h, None, None, None, None),
        ring=lambda: L.sd_read_ring(h, C.c_void_p(ring.ctypes.data), 4),
        spikes=lambda: L.sd_get_spikes(h, None, None, 0, C.byref(m)),
        pending=lambda: L.sd_get_pending(h, None, None, 0, C.byref(m), C.byref(t0)),
        save=lambda: L.sd_save_state(h, None, 0, C.byref(n)),
        stats=lambda: L.sd_get_stats(h, C.byref(st)))

    def calls():
        return {k: f() for k, f in READS.items()}
"""


def test_unasked_launch():
    run(SETUP + """
    assert L.sd_simulate_steps(h, 8 * D) == 0
    assert (launches()[:, 0] == 1).all()
    assert set(calls().values()) == {0}
    for first in READS:  # whichever call looks first
        hip.host_end_early(1)
        assert L.sd_simulate_steps(h, 8 * D) == 0
        hip.host_end_early(0)
        assert L.sd_simulate_steps(h, 8 * D) == 0  # queued before anybody looked
        assert READS[first]() == OVERFLOW, first
        got = calls()
        assert set(got.values()) == {OVERFLOW}, got
        assert b"ended early" in L.sd_last_error(h)
        t, seen = L.sd_t_now(h), len(launches())
        assert L.sd_simulate_steps(h, 8 * D) == OVERFLOW
        assert L.sd_simulate_steps(h, 1) == OVERFLOW
        assert L.sd_update_neurons(h, 1) == OVERFLOW
        assert L.sd_deliver_pending(h) == OVERFLOW
        assert L.sd_deliver_spikes(h, None, None, 0, t) == OVERFLOW
        assert L.sd_t_now(h) == t and len(launches()) == seen
        assert L.sd_load_state(h, saved, n.value) == 0
        assert set(calls().values()) == {0}
        assert L.sd_simulate_steps(h, 8 * D) == 0
        assert set(calls().values()) == {0}
    """)


def test_launch_asked_for():
    run(SETUP + """
    assert L.sd_set_persistent(h, 8) == 0
    hip.host_end_early(1)
    assert L.sd_simulate_steps(h, 8 * D) == 0
    got = calls()
    assert got.pop("stats") == OVERFLOW and set(got.values()) == {0}, got
    assert L.sd_simulate_steps(h, 8 * D) == 0
    """)
