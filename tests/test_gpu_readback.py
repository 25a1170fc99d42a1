"""Read-back through the pinned staging halves: neuron state and ring rows
equal the checkpoint's plain copies, for sizes within one transfer, at both
halves, and past them (several transfers, ranges split between them), with
rows that wrap around the ring, some arrays left out, and contexts of several
host threads reading at once."""
from __future__ import annotations

import ctypes as C
import threading

import numpy as np
import pytest

from paper_2109_12855_amd import sdeliver
from paper_2109_12855_amd import workloads as W

pytestmark = pytest.mark.gpu

HEADER = 8 + 8 + 7 * 8 + 4 * 4 + 4 * 8  # checkpoint header (bytes)


def _net(n, seed=3):
    cfg = W.tiny(model=1, n=n, k=5, seed=seed, d_lo=4, d_hi=9)
    net = sdeliver.Net(cfg).build()
    net.simulate_steps(31)  # ring rows t_now .. wrap around slot 32
    return net


def _plain(net):
    n, L = net.n_local, net.ring_len
    raw = np.frombuffer(net.save_state(), np.uint8)[HEADER:]
    a = raw[: (4 + L) * n * 4].view(np.float32).reshape(4 + L, n)
    return a[0], a[1], a[2], a[3].view(np.int32), a[4:]


def _check(net):
    V, y1, y2, r, ring = _plain(net)
    st = net.state()
    for k, v in (("V", V), ("y1", y1), ("y2", y2), ("r", r)):
        assert np.array_equal(st[k], v), k
    got = net.ring()
    for s in range(net.cfg["d_max"] - net.cfg["d_min"]):
        assert np.array_equal(got[s], ring[(net.t_now + s) % net.ring_len]), s
    only = np.full(net.n_local + 2, -7.0, np.float32)  # y2 alone, its neighbours untouched
    L = sdeliver.lib()
    assert L.sd_read_state(net._h, None, None, C.c_void_p(only[1:].ctypes.data), None) == 0
    assert np.array_equal(only[1:-1], y2) and only[0] == only[-1] == -7.0
    both = np.zeros((2, net.n_local), np.float32)  # V and y2: a gap wider than padding
    assert L.sd_read_state(net._h, C.c_void_p(both[0].ctypes.data), None,
                           C.c_void_p(both[1].ctypes.data), None) == 0
    assert np.array_equal(both[0], V) and np.array_equal(both[1], y2)


# 4 x 131072 x 4 B = 2 MiB: the largest single transfer
@pytest.mark.parametrize("n", [40, 65, 70001, 131072, 131136, 400003])
def test_matches_checkpoint(n):
    net = _net(n)
    _check(net)
    net.close()


def test_threads():
    nets = [_net(n, seed=n) for n in (50, 3000, 150001, 150001 + 64)]
    errors = []

    def work(net):
        try:
            for _ in range(5):
                _check(net)
        except BaseException as e:  # noqa: BLE001 - reported by the test
            errors.append(e)

    t = [threading.Thread(target=work, args=(x,)) for x in nets]
    for x in t:
        x.start()
    for x in t:
        x.join()
    assert not errors, errors
