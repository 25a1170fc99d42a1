"""Lanes per segment of the block-major walk: 16 or 32 where the mean segment,
K B / n_src synapses, and two standard deviations more fit them, in closed loop
(n_src = N) and with virtual sources in any number.  Host code, no device."""
from __future__ import annotations

import math

import pytest

from host_hip import run

LOOPS = [None, 400, 3000, 30_000]  # sources: closed loop, or this many virtual ones


@pytest.mark.parametrize("n_src", LOOPS)
def test_lanes(n_src):
    out = run(f"""
    for k in (10, 100, 250, 500, 1000, 2900):
        for b in (64, 320, 1024):
            cfg = dict(W.tiny(model=1, n=3000, k=k, seed=1, d_lo=4, d_hi=9), layout=1,
                       block_neurons=b, ring_len=64)
            if {n_src}:
                cfg.update(n_src_exc={n_src or 0} * 4 // 5, n_src_inh={n_src or 0} // 5,
                           src_rate_hz=8.0)
            h = create(cfg)
            hip.host_clear()
            if {n_src}:
                assert L.sd_prepare_input(h, 8) == 0
            assert L.sd_simulate_steps(h, 8) == 0, L.sd_last_error(h)
            print(k, b, *set(launches()[:, 4].tolist()))
            L.sd_destroy(h)
    """)
    rows = [tuple(map(int, x.split())) for x in out.splitlines()]
    assert len(rows) == 18
    for k, b, lanes in rows:
        m = k * b / (n_src or 3000)
        top = m + 2 * math.sqrt(m)
        assert lanes == (16 if top <= 16 else 32 if top <= 32 else 64), (k, b, lanes, m)
    assert len({r[2] for r in rows}) > 1
