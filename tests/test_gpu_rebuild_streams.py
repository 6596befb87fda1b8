"""A plan that is sorted again, or given another tile size, from another stream
than that of its last call: the lists are written in place, so the rebuild has
to wait for the launches that read them."""

import pytest
import torch

from paper_2102_12739_amd import workload as wl
from tests.gpu_common import announce, device, plan_for, upload

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("rebuild", ["set_kernel", "sort"])
def test_rebuilding_waits_for_launches_on_other_streams(rebuild):
    announce(f"rebuild {rebuild}")
    p = wl.make_problem("rebuild", [3000, 500, 4000], seed=5, kind="mixed", n_v=96, n_u=80)
    t = upload(p)
    other = t["uvw"].flip(0).contiguous()
    v = torch.from_numpy(wl.complex_noise(4, p.n_vis, 1.0)).to(device())
    plan = plan_for(p)
    plan.set_kernel(4, 40)
    plan.sort(t["uvw"])
    ref = plan.execute(t["sub"], t["g_uv"], t["g_w"], t["uvw"])
    ref_g = plan.adjoint(v, t["g_uv"], t["g_w"], t["uvw"])
    out, grid = torch.zeros_like(ref), torch.zeros_like(ref_g)
    busy, s2 = torch.cuda.Stream(), torch.cuda.Stream()
    torch.cuda.synchronize()
    with torch.cuda.stream(busy):
        torch.cuda._sleep(20_000_000)   # the calls below are still waiting when the rebuild comes
        plan.execute(t["sub"], t["g_uv"], t["g_w"], t["uvw"], out=out)
        plan.adjoint(v, t["g_uv"], t["g_w"], t["uvw"], out=grid)
    with torch.cuda.stream(s2):
        if rebuild == "sort":
            plan.sort(other)
        else:
            plan.set_kernel(4, 56)
    torch.cuda.synchronize()
    assert torch.equal(torch.view_as_real(out), torch.view_as_real(ref))
    assert torch.equal(torch.view_as_real(grid), torch.view_as_real(ref_g))
    again = plan.execute(t["sub"], t["g_uv"], t["g_w"], t["uvw"])
    assert torch.equal(torch.view_as_real(again), torch.view_as_real(ref))
