"""Tags of the persistent slices' exchange lines (host code, no device).

A launch of S slices writes the lines of its slices 0 .. S-2; slice k+1 waits
until every line carries slice k's tag.  A line that already holds the tag
before it is written would be taken for a block without spikes, so at every
write the line's tag must be another one -- also after the 16-bit tags wrapped
around in launches of one or two slices, which write none or one."""
from __future__ import annotations

import pytest

from host_hip import run

MODEL = """
    def check(log):
        line = [0, 0]  # tags of one block's two lines, cleared by the build
        for _, _, S, first, *_ in log[log[:, 0] == 1].tolist():
            for k in range(S - 1):
                tag = (first + k) & 0xffff
                assert line[tag & 1] != tag, tag
                line[tag & 1] = tag
"""


@pytest.mark.parametrize("per,slices", [(1, 65534), (1, 65535), (1, 131070), (2, 65534), (3, 98301),
                                        (5, 66000)])
def test_no_line_holds_a_tag_before_it_is_written(per, slices):
    run(MODEL + f"""
    cfg = dict(W.tiny(model=0, n=100, k=10, seed=1, d_lo=2, d_hi=3))
    h = create(cfg)
    for S, n in (({per}, {slices}), (8, 80)):
        assert L.sd_set_persistent(h, S) == 0, L.sd_last_error(h)
        assert L.sd_simulate_steps(h, n * 2) == 0
    log = launches()
    assert len(log) == -(-{slices} // {per}) + 10 and (log[:, 0] == 1).all()
    check(log)
    """)


def test_default_stretches():
    run(MODEL + """
    cfg = dict(W.tiny(model=0, n=100, k=10, seed=1, d_lo=2, d_hi=3))
    h = create(cfg)
    for n in [4, 7, 4, 5, 1024, 3000] * 20:
        assert L.sd_simulate_steps(h, n * 2) == 0
    log = launches()
    assert log[log[:, 0] == 1][:, 2].sum() > 65536
    check(log)
    """)
