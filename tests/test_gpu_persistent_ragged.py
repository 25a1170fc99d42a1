"""Persistent slices of nets whose last block holds few neurons: the same bits
as one launch per slice, in about the time of a net with whole blocks (the
drive of a short block is shared out over all threads)."""
from __future__ import annotations

import time

import numpy as np
import pytest
import torch

from paper_2109_12855_amd import sdeliver
from paper_2109_12855_amd import workloads as W

pytestmark = pytest.mark.gpu


def _cfg(n, model=0, **over):
    return dict(W.tiny(model=model, n=n, k=100, seed=4, **(over or dict(d_lo=15, d_hi=15))))


@pytest.mark.parametrize("last", [1, 2, 3, 5, 63])
@pytest.mark.parametrize("over", [dict(d_lo=15, d_hi=15), dict(d_lo=1, d_hi=20),
                                  dict(d_lo=10, d_hi=20, block_neurons=768)])
def test_same_bits(last, over):
    b = over.get("block_neurons", 64)
    cfg = dict(_cfg(3 * b + last, model=1, **over), record_spikes=1)
    nets = [sdeliver.Net(cfg).build() for _ in range(2)]
    nets[0].set_persistent(0)
    for net in nets:
        net.simulate_steps(30 * cfg["d_min"])
    for k, v in nets[0].state().items():
        assert np.array_equal(v, nets[1].state()[k]), k
    for x, y in zip(nets[0].spikes(), nets[1].spikes()):
        assert np.array_equal(x, y)
    assert nets[0].stats() == nets[1].stats()


def test_time_of_a_short_last_block():
    def us(n):
        net = sdeliver.Net(_cfg(n)).build()
        best = 1e9
        for _ in range(8):
            torch.cuda.synchronize()
            t = time.perf_counter()
            net.simulate_steps(100 * 15)
            torch.cuda.synchronize()
            best = min(best, time.perf_counter() - t)
        return best * 1e4

    whole, ragged = us(64 * 40), us(64 * 40 + 1)
    assert ragged < 1.5 * whole, (whole, ragged)
