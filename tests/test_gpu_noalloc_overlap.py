"""degrid_execute_noalloc calls of different sizes that ask for the out-of-range
count while they overlap on two streams: whatever their own counts, every later
call's is right."""

import numpy as np
import pytest
import torch

from paper_2102_12739_amd import workload as wl
from paper_2102_12739_amd.degrid import degrid_noalloc
from tests.gpu_common import announce, device, upload

pytestmark = pytest.mark.gpu


def test_counts_after_overlapping_calls():
    announce("noalloc overlap")
    probs = []
    for k, n in enumerate((6000, 40000)):
        p = wl.make_problem("overlap", [n, 100 + k], seed=k, kind="uniform", n_v=64, n_u=64)
        p.uvw[:: 50 + k] = np.nan
        t = upload(p)
        out = torch.empty(p.n_vis, dtype=torch.complex64, device=device())
        probs.append((p, t, out, int(np.isnan(p.uvw[:, 0]).sum())))

    def call(k):
        p, t, out, _ = probs[k]
        oob = torch.full((), -1, dtype=torch.int64, device=device())
        degrid_noalloc(t["sub"], t["g_uv"], t["g_w"], t["uvw"], p.offsets, out=out, oob_count=oob)
        return oob

    streams = [torch.cuda.Stream(), torch.cuda.Stream()]
    torch.cuda.synchronize()
    counts = [[], []]
    for _ in range(60):
        for k, s in enumerate(streams):
            with torch.cuda.stream(s):
                counts[k].append(call(k))
    torch.cuda.synchronize()
    for k in (0, 1):
        assert all(int(c) == probs[k][3] for c in counts[k])
    for k in [0, 1] * 20:      # through every control block
        oob = call(k)
        torch.cuda.synchronize()
        assert int(oob) == probs[k][3]
