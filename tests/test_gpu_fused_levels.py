"""Which node-block levels finish their interface groups in the stencil kernel: those whose couplings come from
the class tables, 2D levels, and small ones that stream.  A product then takes one launch instead of
two.  Either way V-cycle and product equal those of one launch per region (batched = 0) bit for bit, and
since the sums of CG are grouped alike, so do the solve's iterates.
"""
import numpy as np
import pytest

import synth
from tests import harness

pytestmark = pytest.mark.gpu

# (ndof, regions a side, extent, problem, options, launches of a product)
CASES = [
    (1, 3, 13, "laplace", dict(), 1),
    (1, 3, 13, "laplace", dict(region_table=0), 2),
    (1, 3, 13, "laplace", dict(symmetric=0), 2),
    (1, 3, 13, "diffusion", dict(), 2),
    (1, 2, 17, "diffusion", dict(), 1),
    (3, 2, 10, "elasticity", dict(region_table=0), 1),
    (3, 3, 10, "elasticity", dict(region_table=0), 2),
    (3, 3, 10, "elasticity", dict(), 1),
    (1, 3, 13, "laplace", dict(precision=1), 1),  # (launches of the FP64 product)
    (1, 2, 20, "laplace", dict(precision=2), 1),
]


@pytest.mark.parametrize("case", range(len(CASES)))
def test_fused_where_it_pays(hip_device, case):
    import torch

    from paper_2103_11962_amd import regmg

    ndof, r, ex, pde, opts, launches = CASES[case]
    print(f"[fused] {CASES[case]}", flush=True)
    o, e = synth.tensor_layout([[ex] * r] * 3)
    w = synth.Workload("fused", 3, ndof, o, e, 63, 2, 3, pde, h=0.1, seed=case)
    b = harness.to_dev(synth.rhs(w))
    got = []
    for batched in (1, 0):
        h = harness.gpu_problem(w, batched=batched, stencil_kernel=1, **opts)
        n = h.level_info(0)["n_regional"]
        v = torch.from_numpy(np.random.RandomState(1).uniform(-1, 1, n)).to("cuda:0")
        y = torch.empty_like(v)
        before = regmg.kernel_launches()
        h.regional_matvec(0, v, y)
        if batched:
            assert regmg.kernel_launches() - before == launches
        z = torch.empty_like(b)
        h.apply_vcycle(b, z)
        x = torch.zeros_like(b)
        out = h.solve(b, x, rtol=1e-8, maxit=60)
        got.append((z, y, x, out))
        h.close()
    for k in range(3):
        assert torch.equal(got[0][k], got[1][k]), k
    assert got[0][3]["history"] == got[1][3]["history"]


@pytest.mark.parametrize("ext,launches", [([[120, 90], [100, 100]], 1), ([[9] * 9] * 3, 2)])
def test_fused_by_copies(hip_device, ext, launches):
    """2D levels stream five couplings and are fused; 3D ones with more copies than the line are not."""
    import torch

    from paper_2103_11962_amd import regmg

    o, e = synth.tensor_layout(ext)
    dim = len(ext)
    w = synth.Workload("copies", dim, 1, o, e, (1 << 2 * dim) - 1, 3, 2, "fd5" if dim == 2 else "laplace", h=0.1)
    h = harness.gpu_problem(w, stencil_kernel=1)
    n = h.level_info(0)["n_regional"]
    v = torch.zeros(n, dtype=torch.float64, device="cuda:0")
    y = torch.empty_like(v)
    before = regmg.kernel_launches()
    h.regional_matvec(0, v, y)
    assert regmg.kernel_launches() - before == launches
    h.close()
