"""Plastic nets over block sizes: the row of a window slot, which picks the
target's spike history, and the weights and slots behind every synapse.  The
pair rule depends on neither the blocks nor their order, so spikes, state,
ring and weights are the same bit for bit at every block size."""
from __future__ import annotations

import numpy as np
import pytest

from paper_2109_12855_amd import sdeliver
from paper_2109_12855_amd import workloads as W


def test_slot_row_reciprocal_is_exact():
    slot = np.arange(20480 + 1024, dtype=np.uint64)
    for B in range(64, 1025, 64):
        inv = np.uint64(0xFFFFFFFF // B + 1)
        assert np.array_equal((slot * inv) >> np.uint64(32), slot // np.uint64(B)), B


def _run(block):
    cfg = W.plastic(W.tiny(model=1, n=2111, k=300, seed=8, d_lo=4, d_hi=9))
    net = sdeliver.Net(dict(cfg, record_spikes=1, block_neurons=block)).build()
    net.simulate_steps(400)
    out = net.spikes(), net.ring(), net.state(), net.connections()
    net.close()
    return out


@pytest.mark.gpu
@pytest.mark.parametrize("block", [64, 192, 448, 960, 1024])
def test_same_at_every_block_size(block):
    s0, r0, x0, c0 = _run(0)
    s1, r1, x1, c1 = _run(block)
    assert len(s0[0]) > 50
    assert np.array_equal(s0[0], s1[0]) and np.array_equal(s0[1], s1[1])
    assert np.array_equal(np.asarray(r0).view(np.uint32), np.asarray(r1).view(np.uint32))
    for k in x0:
        assert np.array_equal(x0[k], x1[k]), k
    for a, b in zip(c0, c1):
        assert np.array_equal(a, b)
