"""Small levels in few launches: the stencil operations and the restriction finish the interface groups
in their own launch, and the coarse solve gathers, multiplies and scatters in one.  V-cycle and product
must equal those of one launch per region with interface kernels after them (batched = 0) bit for bit;
the sums of CG are grouped by other blocks, so its solution agrees to rounding.
"""
import numpy as np
import pytest

import synth
from tests import harness

pytestmark = pytest.mark.gpu

# (dim, ndof, extents, levels, problem): one copy block and several, groups of 2 to 8, one region
CASES = [
    (2, 1, [[4, 4], [4]], 2, "fd5"),
    (2, 1, [[31, 28, 10], [25, 31, 4]], 3, "fd5"),
    (2, 1, [[82], [55]], 3, "fd5"),
    (3, 1, [[4, 7], [4, 4], [4, 7]], 2, "laplace"),
    (3, 1, [[10, 19], [10, 28], [19, 10]], 3, "laplace"),
    (3, 3, [[10, 10], [10, 7], [4, 10]], 2, "elasticity"),
]


def faces(dim):
    return 15 if dim == 2 else 63


@pytest.mark.parametrize("case", range(len(CASES)))
@pytest.mark.parametrize("opts", [
    dict(),
    dict(smoother=1, cheb_degree=1),
    dict(precision=1),
    dict(precision=2, symmetric=0),
    dict(block_diag=1, use_graph=1),
    dict(region_table=0, use_graph=1),
])
def test_small_levels_equal_separate_launches(hip_device, case, opts):
    import torch

    dim, ndof, ext, nl, prob = CASES[case]
    if (opts.get("precision") and dim == 2) or (opts.get("block_diag") and ndof == 1):
        pytest.skip("27-point or 3-dof option")
    print(f"[small] {CASES[case]} {opts}", flush=True)
    o, e = synth.tensor_layout(ext)
    w = synth.Workload("small", dim, ndof, o, e, faces(dim), nl, 3, prob, h=0.1, seed=case)
    b = harness.to_dev(synth.rhs(w))
    got = []
    for batched in (1, 0):
        h = harness.gpu_problem(w, batched=batched, **opts)
        z = torch.empty_like(b)
        h.apply_vcycle(b, z)
        n = h.level_info(0)["n_regional"]
        v = torch.from_numpy(np.random.RandomState(1).uniform(-1, 1, n)).to("cuda:0")
        y = torch.empty_like(v)
        h.regional_matvec(0, v, y)
        x = torch.zeros_like(b)
        out = h.solve(b, x, rtol=1e-8, maxit=200)
        x2 = torch.zeros_like(b)
        h.solve(b, x2, rtol=1e-8, maxit=200)
        assert torch.equal(x, x2)
        got.append((z, y, x, out))
        h.close()
    assert torch.equal(got[0][0], got[1][0])
    assert torch.equal(got[0][1], got[1][1])
    assert got[0][3]["converged"] and got[0][3]["iterations"] == got[1][3]["iterations"]
    harness.assert_close(got[0][2].cpu().numpy(), got[1][2].cpu().numpy(), 1e-7 if opts.get("precision") else 1e-10)


@pytest.mark.parametrize("ext,nc", [([[97, 94], [97, 97]], 64 * 65), ([[97, 97], [94, 94]], 65 * 63)])
def test_coarse_solve_launch_rule(hip_device, ext, nc):
    """A coarse problem above and one below the one-launch solve's size, against the oracle."""
    import torch

    from oracle import regional

    o, e = synth.tensor_layout(ext)
    w = synth.Workload("coarse", 2, 1, o, e, 15, 2, 3, "fd5", seed=3)
    lay, levels, opt = harness.oracle_problem(w)
    b = synth.rhs(w)
    ref = regional.pcg(levels, lay.to_regional(b), opt, rtol=1e-8, maxit=100)
    h = harness.gpu_problem(w)
    assert h.level_info(1)["n_composite"] == nc
    x = torch.zeros(lay.n_composite, dtype=torch.float64, device="cuda:0")
    out = h.solve(harness.to_dev(b), x, rtol=1e-8, maxit=100)
    assert out["iterations"] == ref.iterations
    harness.assert_close(x.cpu().numpy(), lay.to_composite_owner(ref.x).reshape(-1), 1e-10)
    h.close()
