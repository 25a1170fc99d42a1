"""Which stretches run as persistent (cooperative) launches by default when nets
live on several streams: such launches queue one behind another, so small nets
of three and more streams take one launch per slice.  Host code, no device."""
from __future__ import annotations

import pytest

from host_hip import run

SETUP = """
    def cfg(n):
        return dict(W.tiny(model=0, n=n, k=10, seed=1, d_lo=2, d_hi=3))
    def kinds(h):
        hip.host_clear()
        assert L.sd_simulate_steps(h, 16) == 0, L.sd_last_error(h)
        return set(launches()[:, 0].tolist())  # 1 persistent, 2 one slice
    PERSISTENT, SLICE = {1}, {2}
"""


def test_small_nets_on_several_streams():
    run(SETUP + """
    s = [hip.host_stream(0) for _ in range(4)]
    h = [create(cfg(1250), s[0]), create(cfg(1250), s[0]), create(cfg(1250), s[1])]
    assert [kinds(x) for x in h] == [PERSISTENT] * 3  # two streams
    h.append(create(cfg(100), s[2]))
    assert [kinds(x) for x in h] == [SLICE] * 4
    assert L.sd_set_persistent(h[0], 8) == 0  # asked for
    assert [kinds(x) for x in h] == [PERSISTENT] + [SLICE] * 3
    big = create(cfg(64 * 129), s[3])  # more than half the compute units
    assert kinds(big) == PERSISTENT
    L.sd_destroy(h.pop())
    assert [kinds(x) for x in h] == [PERSISTENT] * 3
    L.sd_destroy(h.pop(0))
    more = [create(cfg(100), x) for x in s]
    assert kinds(more[3]) == SLICE
    for x in more + h:
        L.sd_destroy(x)
    assert kinds(create(cfg(100), s[3])) == PERSISTENT
    """)


def test_other_devices_and_kinds_of_nets_do_not_count():
    run(SETUP + """
    hs = []
    for d in (1, 1, 1, 0):
        hip.host_device(d)
        hs.append(create(cfg(100), hip.host_stream(d)))
    assert kinds(hs[3]) == PERSISTENT and kinds(hs[0]) == SLICE
    for over in (dict(layout=2), dict(block_neurons=1088)):  # never persistent
        hs.append(create(dict(cfg(3000), **over), hip.host_stream(0), build=False))
    hs.append(create(W.plastic(cfg(3000)), hip.host_stream(0), build=False))
    assert kinds(hs[3]) == PERSISTENT
    """)


@pytest.mark.parametrize("n", [64 * 128, 64 * 128 + 1])
def test_half_the_compute_units(n):
    run(SETUP + f"""
    hs = [create(cfg({n}), hip.host_stream(0)) for _ in range(3)]
    assert kinds(hs[0]) == (SLICE if {n} == 64 * 128 else PERSISTENT)
    """)
