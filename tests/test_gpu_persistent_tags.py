"""Persistent launches of one or two slices write no or one exchange line per
launch, and longer ones wait for the lines' 16-bit tags: the results stay those
of one launch per slice past 65,536 such slices."""
from __future__ import annotations

import numpy as np
import pytest

from paper_2109_12855_amd import sdeliver
from paper_2109_12855_amd import workloads as W

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("per,slices", [(1, 65_534), (2, 65_534)])
def test_tags_past_the_wrap(per, slices):
    cfg = dict(W.tiny(model=0, n=200, k=20, seed=5, d_lo=2, d_hi=5), record_spikes=1,
               record_cap=1 << 24)
    a, b = (sdeliver.Net(cfg).build() for _ in range(2))
    a.set_persistent(0)
    b.set_persistent(per)
    for net in (a, b):
        net.simulate_steps(slices * cfg["d_min"])
        assert net.stats()["overflow"] == 0
    b.set_persistent(8)
    for net in (a, b):
        net.simulate_steps(64 * cfg["d_min"])
    assert a.stats()["spikes_emitted"] > 1000
    assert a.stats() == b.stats()
    for k, v in a.state().items():
        assert np.array_equal(v, b.state()[k]), k
    for x, y in zip(a.spikes(), b.spikes()):
        assert np.array_equal(x, y)
    for x, y in zip(a.pending(), b.pending()):
        assert np.array_equal(x, y)
