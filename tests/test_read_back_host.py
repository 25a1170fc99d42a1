"""Host side of the read-back calls on a stand-in HIP runtime: the staging's
pinned memory, transfers and waits, without a device."""
from __future__ import annotations

from host_hip import run

# a net whose state is past both staging halves (2 MiB), its state written so
# that reads can be told from zeros
SETUP = """
    N = 131136
    cfg = dict(W.tiny(model=1, n=N, k=5, seed=1, d_lo=4, d_hi=9))
    rng = np.random.default_rng(1)
    V = rng.standard_normal(N).astype(np.float32)
    R = rng.integers(0, 9, N).astype(np.int32)

    def net(stream=None):
        h = create(cfg, stream, build=False)
        assert L.sd_write_state(h, C.c_void_p(V.ctypes.data), None, None,
                                C.c_void_p(R.ctypes.data)) == 0
        return h

    def right(h):
        rc, (v, _, _, r) = read(h, N)
        return rc == 0 and np.array_equal(v, V) and np.array_equal(r, R)
"""


def test_another_device_is_current():
    """Each context's reads go by its own stream, whatever device is current,
    and leave the shared staging usable for the next device's contexts."""
    run(SETUP + """
    hs = []
    for d in (0, 1):
        hip.host_device(d)
        hs.append(net(hip.host_stream(d)))
    for d in (1, 0, 0, 1):
        hip.host_device(d)
        for h in hs:
            assert right(h), (d, L.sd_last_error(h))
    """)


def test_no_pinned_memory():
    """Where no pinned memory is to be had the arrays come by plain copies."""
    run(SETUP + """
    h = net()
    hip.host_no_pinned(1)
    for _ in range(8):
        assert right(h), L.sd_last_error(h)
    ring = np.ones((3, N), np.float32)
    assert L.sd_read_ring(h, C.c_void_p(ring.ctypes.data), 3) == 0 and not ring.any()
    hip.host_no_pinned(0)
    for _ in range(8):
        assert right(h)
    """)


def test_longest_ring():
    """All rows of the longest ring at once: a list delivered as far ahead as
    the ring allows."""
    run("""
    cfg = dict(W.tiny(model=0, n=40, k=5, seed=1, d_lo=4, d_hi=9), ring_len=512)
    h = create(cfg)
    assert L.sd_deliver_spikes(h, None, None, 0, 512 - 13) == 0
    assert L.sd_simulate_steps(h, 8) == 0
    ring = np.ones((512, 40), np.float32)
    assert L.sd_read_ring(h, C.c_void_p(ring.ctypes.data), 512) == 0, L.sd_last_error(h)
    """)


def test_under_capture():
    """A read on a stream that is being captured is refused before anything of
    it is recorded, and reads work again afterwards."""
    run(SETUP + """
    stream = hip.host_stream(0)
    h = net(stream)
    for _ in range(5):
        assert right(h)
    hip.host_capture(stream, 1)
    for _ in range(2):
        assert read(h, N)[0] == -3  # SD_EHIP
    assert hip.host_recorded() == 0
    hip.host_capture(stream, 0)
    assert right(h)
    """)


def test_pinned_memory_where_it_pays():
    """A program that reads a small net a few times takes no pinned memory, one
    that goes on takes it once; a large net's first read does."""
    run(SETUP + """
    small = W.tiny(model=1, n=1250, k=5, seed=1, d_lo=4, d_hi=9)
    h = create(small, build=False)
    for _ in range(3):
        assert read(h, 1250)[0] == 0
    assert hip.host_pinned() == 0
    for _ in range(50):
        assert read(h, 1250)[0] == 0
    assert hip.host_pinned() == 1
    """)
    run(SETUP + """
    cfg["n_exc"] = 8 * N - cfg["n_inh"]  # 16 MiB of state
    h = create(cfg, build=False)
    for _ in range(3):
        assert read(h, 8 * N)[0] == 0
        assert hip.host_pinned() == 1
    """)
