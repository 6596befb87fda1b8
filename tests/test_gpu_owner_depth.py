"""Gridding of sorted plans around the deepest stack that the owner-computes
adjoint takes; deeper ones scatter."""

import pytest
import torch

import oracle
from paper_2102_12739_amd import workload as wl
from tests.gpu_common import REL_L2_FP32, announce, device, plan_for, rel_l2, upload

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n_w", [300, 3071, 3072, 3073])
def test_deepest_stacks(n_w):
    announce(f"depth {n_w}")
    p = wl.make_problem("depth", [900, 0, 700], seed=n_w, kind="uniform", n_v=17, n_u=20, n_w=n_w)
    t = upload(p)
    plan = plan_for(p)
    v = wl.complex_noise(3, p.n_vis, 1.0)
    ref, oob = oracle.grid(v, p.g_uv, p.g_w, p.uvw, p.offsets, plan.shape)
    base = torch.from_numpy(wl.perturbation(9, plan.shape, 1.0)).to(device())
    for sort in (plan.sort_forward, plan.sort):
        sort(t["uvw"])
        g = plan.adjoint(torch.from_numpy(v).to(device()), t["g_uv"], t["g_w"], t["uvw"])
        assert rel_l2(g.cpu().numpy(), ref) <= REL_L2_FP32
        assert plan.oob_count() == oob
        acc = plan.adjoint(torch.from_numpy(v).to(device()), t["g_uv"], t["g_w"], t["uvw"], out=base.clone(), accumulate=True)
        assert rel_l2(acc.cpu().numpy(), ref + base.cpu().numpy()) <= REL_L2_FP32
