"""Element tiles: on a finest level assembled from element-wise coefficients the FP64 stencil
operations assemble their couplings on the fly.  The V-cycle must equal the streamed one
(region_table = 0) bit for bit and PCG to the rounding of its inner products, on regions at the edges of
the tiles (one region, rows that fill the block, extents of two, mixed with regions of constant
coefficient that class tables serve), with and without Dirichlet faces, also with non-zero values on the
Dirichlet rows.
"""
import numpy as np
import pytest

import synth
from tests import harness

pytestmark = pytest.mark.gpu

LAYOUTS = [
    ([[41]], [[40]], [[63]]),
    ([[2, 9]], [[3, 8]], [[5, 2]]),
    ([[33, 17]], [[29, 6]], [[12, 30]]),
    ([[130]], [[9, 12]], [[7]]),
    ([[512]], [[5]], [[4]]),
]


@pytest.mark.parametrize("mask", [63, 0b010110, 1])
@pytest.mark.parametrize("layout", range(len(LAYOUTS)))
@pytest.mark.parametrize("constant", [False, True])
def test_elem_tiles_equal_streaming(hip_device, layout, mask, constant):
    import torch

    from paper_2103_11962_amd import regmg

    print(f"[elem tiles] {layout} mask {mask} constant {constant}", flush=True)
    o, e = synth.tensor_layout([s[0] for s in LAYOUTS[layout]])
    w = synth.Workload("elem", 3, 1, o, e, mask, 2, 3, "diffusion", h=0.1, seed=layout)
    c = synth.jump_coefficients(w)
    if constant:  # the first region's interior elements alike: its classes may serve it
        c[tuple(slice(int(a), int(a + b - 1)) for a, b in zip(o[0][::-1], e[0][::-1]))] = 2.5
    ec = torch.from_numpy(np.ascontiguousarray(c)).to("cuda:0").reshape(-1)
    rng = np.random.Generator(np.random.PCG64(5))
    b = harness.to_dev(rng.uniform(-1, 1, w.composite_shape))  # Dirichlet rows included
    got = []
    for table in (1, 0):
        h = regmg.Handle(0)
        h.build_regions(3, 1, e, o, mask)
        h.assemble_q1(regmg.PDE_DIFFUSION, w.h, elem_coef=ec)
        h.setup_hierarchy(nlevels=2, cheb_degree=3, stencil_kernel=2, region_table=table)
        z = torch.empty_like(b)
        h.apply_vcycle(b, z)
        n = h.level_info(0)["n_regional"]
        v = torch.from_numpy(np.random.RandomState(1).uniform(-1, 1, n)).to("cuda:0")
        y = torch.empty_like(v)
        h.regional_matvec(0, v, y)
        x = torch.zeros_like(b)
        out = h.solve(b, x, rtol=1e-8, maxit=60, raise_on_fail=False)
        got.append((z, y, x, out))
        h.close()
    assert torch.equal(got[0][0], got[1][0])
    assert torch.equal(got[0][1], got[1][1])
    assert got[0][3]["iterations"] == got[1][3]["iterations"]
    # inner products summed in another order: rounding, grown by the iterations as in the solve's history
    harness.assert_close(got[0][2].cpu().numpy(), got[1][2].cpu().numpy(), 1e-9)
