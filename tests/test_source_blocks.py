"""Automatic block size of the source-major layout: as many rounds of 256
blocks as the largest block that fits needs, in the smallest blocks that keep
that number (at least 192 neurons).  The results do not depend on it."""
from __future__ import annotations

import numpy as np
import pytest

from paper_2109_12855_amd import sdeliver
from paper_2109_12855_amd import workloads as W

ALPHA = dict(W.ALPHA_112K, layout=2)  # window of 20 rows: at most 896 neurons


def _sizes(n, **over):
    cfg = dict(ALPHA, n_exc=n - n // 5, n_inh=n // 5, k_exc=80, k_inh=20)
    return sdeliver.query_sizes(dict(cfg, **over))


@pytest.mark.parametrize("n", [40, 192, 193, 3000, 49152, 49153, 229376, 229377, 281250, 458752,
                               500000, 1125000])
def test_rounds(n):
    s = _sizes(n)
    most = min(896, -(-n // 64) * 64)
    rounds = -(-(-(-n // most)) // 256)
    b = s["block_neurons"]
    assert b % 64 == 0 and b <= most
    assert -(-s["n_blocks"] // 256) == rounds
    if b > 192 and b < most:  # one size less takes another round
        assert -(-(-(-n // (b - 64))) // 256) > rounds
    assert _sizes(n, block_neurons=most)["block_neurons"] == most  # as asked for


def test_large_region_keeps_the_block():
    """Regions of 1,024 records: what the largest block needs is not exceeded
    past the binned records' limit."""
    for n in (281250, 2_000_000):
        assert _sizes(n, bin_cap=1024)["bin_cap"] == 1024


@pytest.mark.gpu
@pytest.mark.parametrize("wform", [0, 1, 2, 3])
@pytest.mark.parametrize("name,over", [
    ("closed", dict(W.tiny(model=1, n=3001, k=300, seed=4, d_lo=10, d_hi=20), layout=2)),
    ("open", dict(W.tiny(model=1, n=5000, k=200, seed=5, d_lo=10, d_hi=20), layout=2,
                  n_src_exc=3200, n_src_inh=800, src_rate_hz=40.0)),
    ("spills", dict(W.tiny(model=0, n=3001, k=400, seed=6, d_lo=3, d_hi=7), layout=2,
                    bin_cap=1))])
def test_same_results(name, over, wform):
    cfg = dict(over, wform=wform, record_spikes=1)
    nets = [sdeliver.Net(cfg).build()]
    most = 896 if cfg["d_max"] == 20 else 1024
    nets.append(sdeliver.Net(dict(cfg, block_neurons=most)).build())
    assert nets[0].sizes["block_neurons"] == 192
    steps = 6 * cfg["d_min"]
    for net in nets:
        if cfg["n_src_exc"]:
            net.prepare_input(steps + 2 * cfg["d_min"])
        net.simulate_steps(steps)
    a, b = nets
    for k, v in a.state().items():
        assert np.array_equal(v, b.state()[k]), k
    n = cfg["d_max"] - cfg["d_min"]
    assert np.array_equal(a.ring(n), b.ring(n))
    for x, y in zip(a.spikes(), b.spikes()):
        assert np.array_equal(x, y)
    sa, sb = a.stats(), b.stats()
    assert sa == sb and sa["overflow"] == 0 and sa["events_delivered"] > 0
