"""A launch that nobody asked for and that gives up waiting (forced from the
host: no polls allowed) is reported by the next read, later launches queued
behind it leave too, and a loaded checkpoint runs on as if nothing happened."""
from __future__ import annotations

import numpy as np
import pytest

from paper_2109_12855_amd import sdeliver
from paper_2109_12855_amd import workloads as W

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("queued", [0, 3])
def test_default_launch_ends_early(queued):
    cfg = dict(W.tiny(model=1, n=2111, k=300, seed=8, d_lo=10, d_hi=20), record_spikes=1)
    a, b = (sdeliver.Net(cfg).build() for _ in range(2))
    b.set_persistent(0)
    for net in (a, b):
        net.simulate_steps(200)
    saved = a.save_state()
    a.set_barrier_spin(0)
    a.simulate_steps(80)
    a.set_barrier_spin(-1)
    for _ in range(queued):
        a.simulate_steps(80)
    with pytest.raises(sdeliver.SdError) as e:
        a.state()
    assert e.value.status == sdeliver.SD_EOVERFLOW
    assert a.stats()["overflow"] & 16
    for call in (lambda: a.simulate_steps(80), a.pending, a.spikes, a.save_state):
        with pytest.raises(sdeliver.SdError) as e:
            call()
        assert e.value.status == sdeliver.SD_EOVERFLOW
    a.load_state(saved)
    for net in (a, b):
        net.simulate_steps(400)
    for k, v in a.state().items():
        assert np.array_equal(v, b.state()[k]), k
    for x, y in zip(a.pending(), b.pending()):
        assert np.array_equal(x, y)
    assert a.stats()["overflow"] == 0
