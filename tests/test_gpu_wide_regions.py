"""Class tables on regions of long rows: a table tile holds rows of at most 339 nodes.  Longer served
regions stream their couplings on 2.5D tiles, beside the table tiles of the shorter ones, and setup
accepts them in every precision; the V-cycle equals the streamed one (region_table = 0) bit for bit.
"""
import pytest

import synth
from tests import harness

pytestmark = pytest.mark.gpu

# (extents, regions that table tiles run)
LAYOUTS = [
    ([[339], [5], [6]], 1),
    ([[340], [5], [6]], 0),
    ([[400], [6], [5]], 0),
    ([[400, 20], [9, 7], [11]], 2),
]


@pytest.mark.parametrize("layout", range(len(LAYOUTS)))
@pytest.mark.parametrize("precision", [0, 1, 2])
def test_wide_regions(hip_device, layout, precision):
    import torch

    ext, tabled = LAYOUTS[layout]
    print(f"[wide] {ext} precision {precision}", flush=True)
    o, e = synth.tensor_layout(ext)
    w = synth.Workload("wide", 3, 1, o, e, 63, 2, 3, "laplace", h=0.1, seed=layout)
    b = harness.to_dev(synth.rhs(w))
    got = []
    for table in (1, 0):
        h = harness.gpu_problem(w, stencil_kernel=2, region_table=table, precision=precision)
        if precision == 0:
            assert h.level_table_regions(0) == (tabled if table else 0)
        z = torch.empty_like(b)
        h.apply_vcycle(b, z)
        x = torch.zeros_like(b)
        out = h.solve(b, x, rtol=1e-8, maxit=100)
        got.append((z, out))
        h.close()
    assert torch.equal(got[0][0], got[1][0])
    assert got[0][1]["converged"] and got[0][1]["iterations"] == got[1][1]["iterations"]
