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
