"""A sort that finds no memory for the adjoint's order or workspace keeps the
work order, and the adjoint scatters; a later sort has both again."""

import pytest
import torch

import oracle
from paper_2102_12739_amd import workload as wl
from tests.gpu_common import REL_L2_FP32, announce, device, plan_for, rel_l2, upload

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n_w", [4, 9])
@pytest.mark.parametrize("fault", ["gridding", "gridding workspace"])
def test_sorting_without_memory_for_gridding(monkeypatch, fault, n_w):
    announce(f"sort without memory for {fault} {n_w}")
    p = wl.make_problem("mem", [2500, 0, 700], seed=6, kind="mixed", n_v=40, n_u=45, n_w=n_w)
    t = upload(p)
    plan = plan_for(p)
    plain = plan.execute(t["sub"], t["g_uv"], t["g_w"], t["uvw"])
    v = torch.from_numpy(wl.complex_noise(3, p.n_vis, 1.0)).to(device())
    ref, oob = oracle.grid(v.cpu().numpy(), p.g_uv, p.g_w, p.uvw, p.offsets, plan.shape)
    for inject in (fault, None, fault, None):
        if inject:
            monkeypatch.setenv("DG_FAULT_INJECT", inject)
        plan.sort(t["uvw"])
        monkeypatch.delenv("DG_FAULT_INJECT", raising=False)
        assert plan.info()["sorted"] == 1
        got = plan.execute(t["sub"], t["g_uv"], t["g_w"], t["uvw"])
        assert torch.equal(torch.view_as_real(got), torch.view_as_real(plain))
        g = plan.adjoint(v, t["g_uv"], t["g_w"], t["uvw"])
        assert rel_l2(g.cpu().numpy(), ref) <= REL_L2_FP32
        assert plan.oob_count() == oob
    again = plan.adjoint(v, t["g_uv"], t["g_w"], t["uvw"])
    assert torch.equal(torch.view_as_real(again), torch.view_as_real(g))
