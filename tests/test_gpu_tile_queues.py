"""Queues of a tile list made on the device: those of the host's split, also
for short uneven lists. The grid of such a launch has a wavefront for every
tile of its longest queue (four to a workgroup, eight queues), so it shows that
queue's length."""

import numpy as np
import pytest

from paper_2102_12739_amd import workload as wl
from tests.gpu_common import announce, plan_for, upload

pytestmark = pytest.mark.gpu


def split(counts):
    """Tiles per queue: a queue closes with the tile that fills its share, at most one per tile."""
    nq = min(8, len(counts))
    ends, acc = [], 0
    for i, c in enumerate(counts):
        acc += c
        if len(ends) < nq - 1 and acc * nq >= sum(counts) * (len(ends) + 1):
            ends.append(i + 1)
    ends += [len(counts)] * (nq - len(ends))
    return np.diff([0] + ends)


@pytest.mark.parametrize("counts", [
    [64] + [1] * 7, [1] * 7 + [64], [64] + [1] * 31, [64, 64, 64] + [1] * 40, [5], [3, 3], [1] * 8, [1] * 9,
    [64] * 5 + [2] * 60, [2] * 60 + [64] * 5,
])
def test_device_queues_are_the_hosts(counts):
    announce(f"queues {len(counts)}")
    p = wl.make_problem("queues", counts, seed=1, kind="line", n_v=16, n_u=16)
    p.uvw[:] = [8.5, 8.5, 1.5]          # every tile fits its box: one per subgrid
    t = upload(p)
    plan = plan_for(p).sort(t["uvw"])
    plan.set_kernel(4, 64)
    i = plan.info()
    assert i["n_tiles"] == len(counts) and i["n_queues"] == min(8, len(counts))
    assert i["grid_blocks"] == i["n_queues"] * -(-int(split(counts).max()) // 4)
