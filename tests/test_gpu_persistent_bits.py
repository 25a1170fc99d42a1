"""Persistent slices give the results of one launch per slice bit for bit
(Alg. REF, Sec. 3.2: a delivery's window sums are rounded to FP32 once).

The nets cover the exchange's edges: spikes of a block and slice within the
first poll of its line, past it, past the line (list buffer), and past the
LDS list; more spikes than a walk chunk holds; one-step slices; delays equal
to the minimum; minimum delays over whole drive chunks; a ragged last block;
one block; block sizes whose carried rows stay in the HBM ring.
"""
from __future__ import annotations

import numpy as np
import pytest

from paper_2109_12855_amd import sdeliver
from paper_2109_12855_amd import workloads as W

pytestmark = pytest.mark.gpu


def _busy(n, **over):
    """Every neuron driven over threshold within a step or two: about
    n * d_min / (1 + t_ref / h) spikes per slice."""
    d = W.tiny(model=0, n=n, k=20, seed=11)
    d.update(drive_w=30.0, drive_rate_hz=9000.0, t_ref=0.0, w_exc=0.01)
    d.update(over)
    return d


NETS = {
    "alpha_2111_ragged": W.tiny(model=1, n=2111, k=300, seed=8, d_lo=10, d_hi=20),
    "alpha_1000_dmin1": W.tiny(model=1, n=1000, k=100, seed=9, d_lo=1, d_hi=20),
    "delta_equal_delays": W.tiny(model=0, n=1250, k=125, seed=3, d_lo=15, d_hi=15),
    "alpha_dmin8": W.tiny(model=1, n=900, k=90, seed=4, d_lo=8, d_hi=13),
    "alpha_dmin17": W.tiny(model=1, n=500, k=90, seed=4, d_lo=17, d_hi=18, ring_len=40),
    "one_block": W.tiny(model=0, n=50, k=20, seed=5, d_lo=3, d_hi=7),
    "line_and_buffer": _busy(3000, d_lo=5, d_hi=9, d_min=5, d_max=9, block_neurons=128),
    "lds_list_full": _busy(4100, d_lo=6, d_hi=9, d_min=6, d_max=9, block_neurons=1024),
    # 100 blocks of seven waves, some of whose columns another wave flushes
    "wide_blocks": W.tiny(model=1, n=44_452, k=100, seed=7, d_lo=10, d_hi=20, block_neurons=448),
    "wide_blocks_dmin1": W.tiny(model=1, n=44_452, k=100, seed=7, d_lo=1, d_hi=20,
                                block_neurons=448),
    "ring_in_hbm": W.tiny(model=1, n=2400, k=200, seed=6, d_lo=10, d_hi=20, block_neurons=768),
}


def _same(a, b):
    for k, v in a.state().items():
        assert np.array_equal(v, b.state()[k]), k
    n = a.cfg["d_max"]
    assert np.array_equal(a.ring(n), b.ring(n))
    for x, y in zip(a.spikes(), b.spikes()):
        assert np.array_equal(x, y)
    for x, y in zip(a.pending(), b.pending()):
        assert np.array_equal(x, y)
    sa, sb = a.stats(), b.stats()
    assert sa == sb and sa["overflow"] == 0


@pytest.mark.parametrize("wform", [0, 1, 2, 3])
@pytest.mark.parametrize("name", list(NETS))
def test_same_bits(name, wform):
    cfg = dict(NETS[name], wform=wform, record_spikes=1, record_cap=1 << 22)
    a = sdeliver.Net(cfg).build()
    b = sdeliver.Net(cfg).build()
    a.set_persistent(0)
    for i, (per, steps) in enumerate([(None, 9 * cfg["d_min"]), (7, 10 * cfg["d_min"]),
                                      (1, 3 * cfg["d_min"] + 1), (None, 8 * cfg["d_min"] + 2)]):
        if per:
            b.set_persistent(per)
        a.simulate_steps(steps)
        b.simulate_steps(steps)
        assert a.t_now == b.t_now
    assert a.stats()["spikes_emitted"] > 20
    _same(a, b)
    a.close()
    b.close()


def test_after_external_list():
    """A list delivered ahead of the carried rows: fused slices until the ring
    is back within them, then persistent ones."""
    import torch
    cfg = dict(W.tiny(model=1, n=1500, k=150, seed=2, d_lo=4, d_hi=9), record_spikes=1,
               ring_len=48)
    nets = [sdeliver.Net(cfg).build() for _ in range(2)]
    src, lag = W.replay_spikes(1500, 60, 4, seed=4)
    s, l = torch.from_numpy(src.view(np.int32)).cuda(), torch.from_numpy(lag).cuda()
    nets[0].set_persistent(0)
    for net in nets:
        net.simulate_steps(40)
        net.deliver(s, l, net.t_now + 12)
        net.simulate_steps(80)
    _same(*nets)


def test_two_streams():
    """Persistent launches queued on two streams at once give what each net
    gives alone."""
    import torch
    cfgs = [dict(W.tiny(model=1, n=2111, k=300, seed=s, d_lo=10, d_hi=20), record_spikes=1)
            for s in (8, 9)]
    alone = []
    for cfg in cfgs:
        net = sdeliver.Net(cfg).build()
        net.set_persistent(0)
        net.simulate_steps(600)
        alone.append(net)
    streams = [torch.cuda.Stream() for _ in cfgs]
    both = [sdeliver.Net(cfg, stream=s).build() for cfg, s in zip(cfgs, streams)]
    for net in both:
        net.set_barrier_spin(1 << 22)  # bounded, whatever the order of the launches
    for _ in range(10):
        for net in both:
            net.simulate_steps(60)
    for a, b in zip(alone, both):
        _same(a, b)
