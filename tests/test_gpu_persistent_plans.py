"""Persistent slices at the ends of what their plan covers, bit for bit as one
launch per slice: block sizes and delays whose window leaves no room for whole
drive chunks (drive counts drawn per slice, carried rows in the HBM ring), and
as many blocks as a launch holds lines for."""
from __future__ import annotations

import numpy as np
import pytest

from paper_2109_12855_amd import sdeliver
from paper_2109_12855_amd import workloads as W

pytestmark = pytest.mark.gpu


def _net(n, b, d_min, d_max, model):
    return dict(W.tiny(model=model, n=n, k=150, seed=6, d_lo=d_min, d_hi=d_max),
                block_neurons=b, ring_len=64, record_spikes=1, record_cap=1 << 22)


@pytest.mark.parametrize("wform", [0, 3])
@pytest.mark.parametrize("n,b,d_min,d_max,model", [
    (2500, 1024, 2, 18, 1), (2500, 960, 11, 18, 0), (2000, 640, 10, 28, 1), (1700, 832, 3, 22, 0),
    (256 * 64, 64, 4, 9, 1), (255 * 64 + 1, 64, 4, 9, 0)])
def test_same_bits(n, b, d_min, d_max, model, wform):
    cfg = dict(_net(n, b, d_min, d_max, model), wform=wform)
    nets = [sdeliver.Net(cfg).build() for _ in range(2)]
    nets[0].set_persistent(0)
    nets[1].set_persistent(9)
    for net in nets:
        net.simulate_steps(41 * d_min + 1)
        net.simulate_steps(13 * d_min)
    a, b = nets
    assert a.stats()["spikes_emitted"] > 100
    assert a.stats() == b.stats() and a.stats()["overflow"] == 0
    for k, v in a.state().items():
        assert np.array_equal(v, b.state()[k]), k
    assert np.array_equal(a.ring(d_max), b.ring(d_max))
    for x, y in zip(a.spikes(), b.spikes()):
        assert np.array_equal(x, y)
    for x, y in zip(a.pending(), b.pending()):
        assert np.array_equal(x, y)


def test_more_blocks_than_lines():
    net = sdeliver.Net(_net(257 * 64, 64, 4, 9, 1)).build()
    with pytest.raises(sdeliver.SdError) as e:
        net.set_persistent(8)
    assert e.value.status == sdeliver.SD_EUNSUPPORTED
    net.simulate_steps(40)
    assert net.stats()["overflow"] == 0
