"""The read-back checks once a process's first, plain reads are over: every
size and range through the pinned halves."""
from __future__ import annotations

import pytest

from test_gpu_readback import _check, _net

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n", [40, 65, 70001, 131072, 131136, 400003])
def test_matches_checkpoint_staged(n):
    net = _net(n)
    for _ in range(4):
        net.state()
    _check(net)
    net.close()
