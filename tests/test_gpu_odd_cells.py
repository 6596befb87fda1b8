"""The scatter adjoint on outputs of an odd number of cells (an odd number of
8-byte values to clear first): odd sides, odd depths, odd numbers of subgrids."""

import pytest
import torch

import oracle
from paper_2102_12739_amd import workload as wl
from tests.gpu_common import REL_L2_FP32, announce, device, plan_for, rel_l2, upload

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("counts,n_v,n_u,n_w", [([5], 9, 9, 5), ([300, 0, 70], 17, 33, 7), ([200], 9, 11, 3073), ([40, 3], 9, 9, 5)])
@pytest.mark.parametrize("how", ["none", "sort_forward", "sort"])
def test_odd_numbers_of_cells(counts, n_v, n_u, n_w, how):
    announce(f"odd cells {counts} {n_v}x{n_u}x{n_w} {how}")
    p = wl.make_problem("odd", counts, seed=n_w, kind="uniform", n_v=n_v, n_u=n_u, n_w=n_w)
    t = upload(p)
    plan = plan_for(p)
    if how != "none":
        getattr(plan, how)(t["uvw"])
    v = wl.complex_noise(3, p.n_vis, 1.0)
    ref, oob = oracle.grid(v, p.g_uv, p.g_w, p.uvw, p.offsets, plan.shape)
    cells = ref.size
    buf = torch.full((cells + 1,), complex("nan+nanj"), dtype=torch.complex64, device=device())
    out = buf[:cells].view(plan.shape)
    plan.adjoint(torch.from_numpy(v).to(device()), t["g_uv"], t["g_w"], t["uvw"], out=out)
    assert rel_l2(out.cpu().numpy(), ref) <= REL_L2_FP32
    assert plan.oob_count() == oob
    assert torch.isnan(torch.view_as_real(buf[cells])).all()      # nothing past the end
