"""Gridding of sorted plans whose visibilities crowd a few bands and columns, so
that the owner-computes adjoint cuts its longest runs into slices and joins
them: against the FP64 oracle, around the length of a slice, for spots at the
edges of segments and bands, one heavy subgrid among light ones, deep stacks,
every storage and table type, accumulation, moved coordinates and values that
are not finite. Every result repeats bit for bit."""

import numpy as np
import pytest
import torch

import oracle
from paper_2102_12739_amd import workload as wl
from tests.gpu_common import REL_L2_FP32, announce, device, plan_for, rel_l2, stored_reference_inputs, upload

pytestmark = pytest.mark.gpu


def crowd(p, lo, hi, share=1.0, seed=0):
    """A share of the first subgrid's first taps into [lo, hi] (columns, rows)."""
    rng = np.random.default_rng(seed)
    n = int(share * p.offsets[1])
    p.uvw[:n, 0] = rng.integers(lo[0], hi[0] + 1, n) + 3 + rng.uniform(0.01, 0.99, n)
    p.uvw[:n, 1] = rng.integers(lo[1], hi[1] + 1, n) + 3 + rng.uniform(0.01, 0.99, n)
    return p


def check(p, gcf="f32", grid="c64", kernel=None, moved=False):
    t = upload(p, grid, gcf)
    plan = plan_for(p, grid_dtype=grid, gcf_dtype=gcf).sort(t["uvw"])
    if kernel is not None:
        plan.set_kernel(kernel)
    v = wl.complex_noise(3, p.n_vis, 1.0)
    vt = torch.from_numpy(v).to(device())
    _, g_uv, g_w = stored_reference_inputs(p, grid, gcf)
    ref, oob = oracle.grid(v, g_uv, g_w, p.uvw, p.offsets, plan.shape)
    out = torch.full(plan.shape, float("nan"), dtype=torch.complex64, device=device())
    g = plan.adjoint(vt, t["g_uv"], t["g_w"], t["uvw"], out=out)
    assert rel_l2(g.cpu().numpy(), ref) <= REL_L2_FP32
    assert plan.oob_count() == oob
    again = plan.adjoint(vt, t["g_uv"], t["g_w"], t["uvw"])
    assert torch.equal(torch.view_as_real(again), torch.view_as_real(g))
    base = torch.from_numpy(wl.perturbation(9, plan.shape, 1.0)).to(device())
    acc = plan.adjoint(vt, t["g_uv"], t["g_w"], t["uvw"], out=base.clone(), accumulate=True)
    assert rel_l2(acc.cpu().numpy(), ref + base.cpu().numpy()) <= REL_L2_FP32
    if moved:
        u = p.uvw.copy()
        u[::3, 0] = 3.5 + (u[::3, 0] + 1.0) % (p.n_u - 7.5)
        ref_m, oob_m = oracle.grid(v, g_uv, g_w, u, p.offsets, plan.shape)
        g = plan.adjoint(vt, t["g_uv"], t["g_w"], torch.from_numpy(u).to(device()))
        assert rel_l2(g.cpu().numpy(), ref_m) <= REL_L2_FP32
        assert plan.oob_count() == oob_m


# one column and one row of first taps: the run of one band holds every visibility
@pytest.mark.parametrize("n", [255, 256, 257, 270, 271, 272, 273, 320, 511, 512, 513, 530, 529, 4000])
def test_runs_around_the_length_of_a_slice(n):
    announce(f"slice length {n}")
    check(crowd(wl.make_problem("len", [n, 40], seed=n, kind="uniform", n_v=41, n_u=47), (20, 10), (20, 10)))


@pytest.mark.parametrize("n_v,n_u,lo,hi", [
    (33, 35, (15, 15), (16, 16)),      # across segments and bands
    (16, 16, (0, 0), (8, 8)),          # one segment, every window position
    (8, 8, (0, 0), (0, 0)),
    (50, 61, (0, 42), (3, 42)),        # first columns, last band
    (49, 50, (40, 41), (42, 41)),      # last columns, a band of one row
    (64, 240, (5, 3), (230, 30)),      # wide: slices of many columns
])
@pytest.mark.parametrize("gcf,os_uv", [("f32", 8), ("bf16", 64), ("f16", 16)])
def test_crowds_at_the_edges(n_v, n_u, lo, hi, gcf, os_uv):
    announce(f"slices {n_v}x{n_u} {lo} {hi} {gcf} {os_uv}")
    p = crowd(wl.make_problem("edge", [3000, 0, 200], seed=n_u, kind="mixed", n_v=n_v, n_u=n_u, os_uv=os_uv), lo, hi, 0.9)
    p.uvw[7] = np.nan
    check(p, gcf, moved=True)


@pytest.mark.parametrize("n_w", [5, 8, 11])
def test_crowds_in_deep_stacks(n_w):
    announce(f"deep slices {n_w}")
    check(crowd(wl.make_problem("deep", [4000, 100], seed=n_w, kind="uniform", n_v=33, n_u=40, n_w=n_w), (14, 12), (17, 20)),
          moved=True)


@pytest.mark.parametrize("grid,gcf,kernel", [("c64", "f32", None), ("c64", "f32", 0), ("c64", "f32", 6), ("cf16", "f16", None),
                                             ("cbf16", "bf16", None), ("cbf16", "f32", 4)])
@pytest.mark.parametrize("counts,n_v,n_u", [([30000] + [50] * 20, 99, 60), ([12000, 11000], 48, 40), ([9000, 9000], 33, 31)])
def test_heavy_and_light_subgrids(grid, gcf, kernel, counts, n_v, n_u):
    """Whatever the plan's gather kernel: it has no say in how a sorted plan grids."""
    announce(f"heavy {counts[:2]} {n_v}x{n_u} {grid} {kernel}")
    check(wl.make_problem("heavy", counts, seed=n_v, kind="uniform", n_v=n_v, n_u=n_u), gcf, grid, kernel)


def test_more_tasks_are_split_than_a_workgroup_has_threads():
    announce("many split tasks")
    # 24 subgrids of 5 bands x 4 segments, every run longer than a slice
    check(wl.make_problem("tasks", [16000] * 24, seed=2, kind="uniform", n_v=72, n_u=56))


def test_values_that_are_not_finite_stay_in_their_windows():
    announce("slices not finite")
    p = crowd(wl.make_problem("inf", [2000], seed=4, kind="uniform", n_v=50, n_u=60), (20, 20), (30, 24), 0.95)
    t = upload(p)
    plan = plan_for(p).sort(t["uvw"])
    v = wl.complex_noise(6, p.n_vis, 1.0)
    bad = np.zeros(p.n_vis, bool)
    bad[[10, 1990]] = True
    v[10], v[1990] = complex(np.inf, 1.0), complex(0.5, np.nan)
    touched, _ = oracle.grid(bad.astype(np.complex64), np.ones_like(p.g_uv), np.ones_like(p.g_w), p.uvw, p.offsets,
                             plan.shape)
    ref, _ = oracle.grid(np.where(bad, 0, v).astype(np.complex64), p.g_uv, p.g_w, p.uvw, p.offsets, plan.shape)
    g = plan.adjoint(torch.from_numpy(v).to(device()), t["g_uv"], t["g_w"], t["uvw"]).cpu().numpy()
    free = touched == 0
    assert np.isfinite(g[free]).all() and rel_l2(g[free], ref[free]) <= REL_L2_FP32
    assert not np.isfinite(g[~free]).any()
