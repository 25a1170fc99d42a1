"""Segment walk with 16, 32 and 64 lanes per segment (Alg. REF, Sec. 3.2):
in-degrees on both sides of the rule's lines, segments longer than their
lanes, and list lengths around a group and a chunk.  Counts per ring cell
equal the oracle's; weights hold the per-cell bound 1e-6 sum |w|."""
from __future__ import annotations

import numpy as np
import pytest
import torch

import oracle
from paper_2109_12855_amd import sdeliver
from paper_2109_12855_amd import workloads as W

pytestmark = pytest.mark.gpu

N, B = 640, 64
# mean segment K / 10: 3, 9 and 9.4 (16 | 32 lanes at m + 2 sqrt(m) = 16), 22
# and 23.5 (32 | 64 at 32), 70 (past a wave)
KS = [30, 90, 94, 220, 235, 700]


@pytest.mark.parametrize("wform", [0, 1, 3])
@pytest.mark.parametrize("k", KS)
def test_counts_and_sums(k, wform):
    cfg = W.tiny(model=1, n=N, k=k, seed=k, d_lo=4, d_hi=9, wform=wform, block_neurons=B)
    net, cnt = sdeliver.Net(cfg).build(), sdeliver.Net(cfg).build()
    cnt.set_count_mode(True)
    ocfg = dict(cfg, wform=W.ORACLE_WFORM[wform])
    row, tgt, dly, w = oracle.Net(ocfg).source_major()
    # the busiest sources hold segments past two standard deviations
    length = max(int(np.bincount(tgt[row[s]:row[s + 1]] // B).max()) for s in range(N))
    assert length > {30: 8, 90: 16, 94: 16, 220: 32, 235: 32, 700: 64}[k]
    ring = np.zeros((cfg["ring_len"], N))
    size = np.zeros_like(ring)
    hits = np.zeros(ring.shape, np.int64)
    for i, n in enumerate((1, 11, 12, 13, 16, 17, 250, 1023, 1025, 2300)):
        src, lag = W.replay_spikes(N, n, 4, seed=i)
        d = torch.from_numpy(src.view(np.int32)).cuda(), torch.from_numpy(lag).cuda()
        for x in (net, cnt):
            x.deliver(*d, 0)
        for s, l in zip(src.tolist(), lag.tolist()):
            e = slice(row[s], row[s + 1])
            at = ((l + dly[e]) % cfg["ring_len"], tgt[e])
            np.add.at(ring, at, w[e])
            np.add.at(size, at, np.abs(w[e]))
            np.add.at(hits, at, 1)
    assert np.array_equal(cnt.ring().astype(np.int64), hits)
    assert np.all(np.abs(net.ring() - ring) <= 1e-6 * size + 1e-30)
    assert cnt.stats()["overflow"] == 0
    net.close()
    cnt.close()
