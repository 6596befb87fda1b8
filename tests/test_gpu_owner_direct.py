"""The owner-computes adjoint on both sides of the number of visibilities (3 * 2^16)
up to which it reads the visibilities themselves instead of records of them:
every table type and path, deep stacks, moved and out-of-range coordinates,
accumulation and values that are not finite, against the FP64 oracle."""

import numpy as np
import pytest
import torch

import oracle
from paper_2102_12739_amd import workload as wl
from tests.gpu_common import REL_L2_FP32, announce, device, plan_for, rel_l2, stored_reference_inputs, upload

pytestmark = pytest.mark.gpu

DIRECT = 3 << 16


@pytest.mark.parametrize("n", [DIRECT, DIRECT + 1])
@pytest.mark.parametrize("n_v,n_u,n_w,os_uv,gcf", [
    (97, 113, 4, 16, "f32"), (64, 240, 4, 8, "f16"), (65, 63, 4, 64, "bf16"), (33, 40, 7, 8, "f32"), (40, 41, 9, 64, "f16"),
])
def test_records_and_direct_reads(n, n_v, n_u, n_w, os_uv, gcf):
    announce(f"owner direct {n} {n_v}x{n_u}x{n_w} {gcf} {os_uv}")
    p = wl.make_problem("direct", [n - 900, 0, 1, 899], seed=n_u, kind="mixed", n_v=n_v, n_u=n_u, n_w=n_w, os_uv=os_uv)
    p.uvw[[5, n - 3]] = np.nan
    p.uvw[6:4000:97, 0] = 2.0
    t = upload(p, "c64", gcf)
    plan = plan_for(p, gcf_dtype=gcf).sort(t["uvw"])
    v = wl.complex_noise(3, p.n_vis, 1.0)
    vt = torch.from_numpy(v).to(device())
    _, g_uv, g_w = stored_reference_inputs(p, "c64", gcf)
    ref, oob = oracle.grid(v, g_uv, g_w, p.uvw, p.offsets, plan.shape)
    out = torch.full(plan.shape, float("nan"), dtype=torch.complex64, device=device())
    for _ in range(2):
        g = plan.adjoint(vt, t["g_uv"], t["g_w"], t["uvw"], out=out)
        assert rel_l2(g.cpu().numpy(), ref) <= REL_L2_FP32
        assert plan.oob_count() == oob
    again = plan.adjoint(vt, t["g_uv"], t["g_w"], t["uvw"])
    assert torch.equal(torch.view_as_real(again), torch.view_as_real(g))
    for share in (1.0, 0.001):      # moved since the sort, into range and out of it too
        moved = p.uvw.copy()
        pick = np.random.default_rng(1).random(n) < share
        moved[pick] = np.roll(p.uvw, 7, axis=0)[pick]
        ref_m, oob_m = oracle.grid(v, g_uv, g_w, moved, p.offsets, plan.shape)
        base = torch.from_numpy(wl.perturbation(9, plan.shape, 1.0)).to(device())
        mt = torch.from_numpy(moved).to(device())
        g = plan.adjoint(vt, t["g_uv"], t["g_w"], mt)
        assert rel_l2(g.cpu().numpy(), ref_m) <= REL_L2_FP32
        assert plan.oob_count() == oob_m
        g = plan.adjoint(vt, t["g_uv"], t["g_w"], mt, out=base.clone(), accumulate=True)
        assert rel_l2(g.cpu().numpy(), ref_m + base.cpu().numpy()) <= REL_L2_FP32
    g = plan.adjoint(vt, t["g_uv"], t["g_w"], t["uvw"])     # and back
    assert torch.equal(torch.view_as_real(again), torch.view_as_real(g))


@pytest.mark.parametrize("n", [DIRECT, DIRECT + 1])
@pytest.mark.parametrize("n_w", [4, 6])
def test_values_that_are_not_finite_stay_in_their_windows(n, n_w):
    announce(f"owner direct not finite {n} {n_w}")
    p = wl.make_problem("inf", [n], seed=4, kind="uniform", n_v=120, n_u=130, n_w=n_w, os_uv=8, os_w=8)
    t = upload(p)
    plan = plan_for(p).sort(t["uvw"])
    v = wl.complex_noise(6, p.n_vis, 1.0)
    bad = np.zeros(n, bool)
    bad[[10, n - 1]] = True
    v[10], v[n - 1] = complex(np.inf, 1.0), complex(0.5, np.nan)
    touched, _ = oracle.grid(bad.astype(np.complex64), np.ones_like(p.g_uv), np.ones_like(p.g_w), p.uvw, p.offsets,
                             plan.shape)
    ref, _ = oracle.grid(np.where(bad, 0, v).astype(np.complex64), p.g_uv, p.g_w, p.uvw, p.offsets, plan.shape)
    g = plan.adjoint(torch.from_numpy(v).to(device()), t["g_uv"], t["g_w"], t["uvw"]).cpu().numpy()
    free = touched == 0
    assert np.isfinite(g[free]).all() and rel_l2(g[free], ref[free]) <= REL_L2_FP32
    assert not np.isfinite(g[~free]).any()


def test_adjoints_of_small_plans_replay_from_a_graph():
    """Captured once and replayed with the program's own calls between."""
    announce("owner direct graph")
    p = wl.make_problem("graph", [3000, 200], seed=3, kind="uniform", n_v=49, n_u=50)
    t = upload(p)
    plan = plan_for(p).sort(t["uvw"])
    vt = torch.from_numpy(wl.complex_noise(3, p.n_vis, 1.0)).to(device())
    ref = plan.adjoint(vt, t["g_uv"], t["g_w"], t["uvw"])
    out = torch.zeros_like(ref)
    uvw = t["uvw"].clone()
    g = torch.cuda.CUDAGraph()
    torch.cuda.synchronize()
    with torch.cuda.graph(g):
        plan.adjoint(vt, t["g_uv"], t["g_w"], uvw, out=out)
    for k in range(3):
        out.zero_()
        g.replay()
        torch.cuda.synchronize()
        assert torch.equal(torch.view_as_real(out), torch.view_as_real(ref)), k
        assert rel_l2(plan.adjoint(vt, t["g_uv"], t["g_w"], t["uvw"].roll(1, 0)).cpu().numpy(),
                      oracle.grid(vt.cpu().numpy(), p.g_uv, p.g_w, np.roll(p.uvw, 1, 0), p.offsets, plan.shape)[0]) <= REL_L2_FP32
