"""Where the device cuts the work order into tiles: against the rule itself,
followed here visibility by visibility (order along the Hilbert curve, chunks of
2048, the longest run of at most n_b whose box fits, 24 or n_b where fewer
fit). Outputs are the same for any cut, so the number of tiles and the length of
the longest queue are compared: both change with every box judged wrongly."""

import numpy as np
import pytest

from paper_2102_12739_amd import workload as wl
from tests.gpu_common import announce, plan_for, upload
from tests.test_gpu_tile_queues import split

pytestmark = pytest.mark.gpu

CHUNK, MIN_FIT = 2048, 24
BOX = {1: 8192, 2: 12288, 3: 16384, 4: 18432}     # bytes of the kernel variants' boxes


def hilbert(x, y, bits):
    d = 0
    for b in range(bits - 1, -1, -1):
        rx, ry = (x >> b) & 1, (y >> b) & 1
        d += (1 << (2 * b)) * ((3 * rx) ^ ry)
        if ry == 0:
            if rx == 1:
                x, y = (1 << bits) - 1 - x, (1 << bits) - 1 - y
            x, y = y, x
    return d


def cut(first, cell_bytes, box, n_b):
    """Tile sizes of one subgrid's ordered first taps (None: out of range)."""
    cells, sizes = box // (4 * cell_bytes), []
    for c0 in range(0, len(first), CHUNK):
        chunk = first[c0:c0 + CHUNK]
        at = 0
        while at < len(chunk):
            n = min(n_b, len(chunk) - at)
            xs, ys, k = [], [], 0
            while k < n:
                if chunk[at + k] is not None:
                    xs.append(chunk[at + k][0])
                    ys.append(chunk[at + k][1])
                    if (max(xs) - min(xs) + 8) * (max(ys) - min(ys) + 8) > cells:
                        break
                k += 1
            if at + k < len(chunk):
                k = min(n, max(k, min(MIN_FIT, n_b)))
            sizes.append(max(k, 1))
            at += sizes[-1]
    return sizes


@pytest.mark.parametrize("counts,n_v,n_u,kind,grid", [
    ((1, 63, 64, 65, 300), 64, 64, "uniform", "c64"), ((2047, 2049, 0, 4097), 96, 80, "mixed", "c64"),
    ((6000,), 512, 512, "uniform", "c64"), ((3000, 10), 200, 333, "line", "cf16"), ((5000, 700), 40, 33, "uniform", "cbf16"),
])
def test_tiles_end_where_the_box_does(counts, n_v, n_u, kind, grid):
    announce(f"tile cut {counts} {n_v}x{n_u} {kind} {grid}")
    p = wl.make_problem("cut", counts, seed=sum(counts), kind=kind, n_v=n_v, n_u=n_u)
    p.uvw[::37] = [np.nan, 5.0, 1.5]
    t = upload(p, grid)
    plan = plan_for(p, grid_dtype=grid).sort_forward(t["uvw"])
    bits = 1
    while (1 << bits) <= max(n_u, n_v) - 8:
        bits += 1
    ordered = []
    for a, b in zip(p.offsets, p.offsets[1:]):
        taps = []
        for u, v, w in p.uvw[a:b]:
            x, y = (int(np.floor(u)) - 3, int(np.floor(v)) - 3) if np.isfinite(u) else (-1, -1)
            ok = 0 <= x <= n_u - 8 and 0 <= y <= n_v - 8 and 1.0 <= w < 2.0
            taps.append((x, y) if ok else None)
        ordered.append(sorted(taps, key=lambda t: hilbert(*t, bits) if t else 1 << (2 * bits)))
    cell = 8 if grid == "c64" else 4
    for kernel, n_b in ((1, 32), (2, 32), (3, 9), (4, 64), (4, 24), (4, 1)):
        plan.set_kernel(kernel, n_b)
        sizes = [k for taps in ordered for k in cut(taps, cell, BOX[kernel], n_b)]
        i = plan.info()
        assert i["n_tiles"] == len(sizes), (kernel, n_b)
        blocks = i["n_queues"] * -(-int(split(sizes).max()) // 4)
        assert i["grid_blocks"] == blocks or blocks > 2 * 256, (kernel, n_b)
