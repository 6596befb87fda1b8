"""degrid_execute_noalloc over thousands of subgrids, up to its limit: every
tile finds its subgrid, among empty ones, runs of empty ones and heavy ones."""

import numpy as np
import pytest
import torch

from paper_2102_12739_amd import workload as wl
from paper_2102_12739_amd.degrid import degrid_noalloc
from tests.gpu_common import announce, device, plan_for, upload

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("s,kind", [(193, "even"), (4097, "sparse"), (4225, "ends"), (16383, "even"),
                                    (16384, "sparse"), (16384, "ends")])
def test_noalloc_finds_the_subgrid_of_every_tile(s, kind):
    announce(f"noalloc {s} {kind}")
    rng = np.random.default_rng(s)
    counts = rng.integers(0, 9, s)
    if kind == "sparse":
        counts[rng.random(s) < 0.95] = 0
        counts[rng.integers(0, s, 5)] = 700
    elif kind == "ends":
        counts[1:-1] = 0
        counts[0], counts[-1] = 3000, 2999
    p = wl.make_problem("many", counts, seed=s, kind="uniform", n_v=9, n_u=10, os_uv=4, os_w=4)
    t = upload(p)
    plan = plan_for(p)
    ref = plan.execute(t["sub"], t["g_uv"], t["g_w"], t["uvw"])
    for n_b in (0, 64, 1):
        out = torch.full((p.n_vis,), float("nan"), dtype=torch.complex64, device=device())
        oob = torch.full((), -1, dtype=torch.int64, device=device())
        degrid_noalloc(t["sub"], t["g_uv"], t["g_w"], t["uvw"], p.offsets, out=out, oob_count=oob, n_b=n_b)
        assert torch.equal(torch.view_as_real(out), torch.view_as_real(ref)), n_b
        assert int(oob) == plan.oob_count()
