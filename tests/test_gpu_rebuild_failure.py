"""A failed change of kernel or tile size leaves a plan whose kernel and tiles
still belong together: tiles of 64 visibilities never meet a kernel that takes
32."""

import pytest
import torch

from paper_2102_12739_amd import workload as wl
from paper_2102_12739_amd.degrid import DegridError
from tests.gpu_common import announce, plan_for, upload

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("sort", [False, True])
def test_a_failed_change_of_kernel_changes_nothing(monkeypatch, sort):
    announce(f"rebuild failure sort={sort}")
    p = wl.make_problem("fail", [3000, 900], seed=9, kind="mixed", n_v=60, n_u=64)
    t = upload(p)
    plan = plan_for(p)
    if sort:
        plan.sort(t["uvw"])
    plan.set_kernel(4, 64)
    before = plan.info()
    ref = plan.execute(t["sub"], t["g_uv"], t["g_w"], t["uvw"])
    for kernel, n_b in ((1, 0), (0, 8), (6, 64)):
        monkeypatch.setenv("DG_FAULT_INJECT", "alloc")
        with pytest.raises(DegridError) as e:
            plan.set_kernel(kernel, n_b)
        assert e.value.status == 3
        with pytest.raises(DegridError):
            plan.tune(t["sub"], t["g_uv"], t["g_w"], t["uvw"])
        monkeypatch.delenv("DG_FAULT_INJECT")
        assert plan.info() == before
        got = plan.execute(t["sub"], t["g_uv"], t["g_w"], t["uvw"])
        assert torch.equal(torch.view_as_real(got), torch.view_as_real(ref))
    plan.set_kernel(1, 0)
    assert plan.info()["kernel"] == 1 and plan.info()["n_b"] <= 32
    got = plan.execute(t["sub"], t["g_uv"], t["g_w"], t["uvw"])
    assert torch.equal(torch.view_as_real(got), torch.view_as_real(ref))
