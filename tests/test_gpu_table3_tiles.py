"""Table tiles of 3-dof levels: on elasticity levels whose regions the class tables all serve, the stencil
operations run whole-row and x-face tiles.  V-cycle and product must equal those of streaming every
coupling (region_table = 0) bit for bit: FP64, FP32 and BF16 couplings, point and nodal-block D~, on
regions at the edges of the tiles (five nodes a side, more than 64 rows, single rows a tile, ragged).
"""
import numpy as np
import pytest

import synth
from tests import harness

pytestmark = pytest.mark.gpu

LAYOUTS = [
    [[10, 7], [9], [12, 8]],
    [[5], [5, 6], [5]],
    [[6, 5], [66], [7]],
    [[200], [6], [5]],
    [[19], [70, 20], [9, 19]],
]


@pytest.mark.parametrize("layout", range(len(LAYOUTS)))
@pytest.mark.parametrize("precision,block", [(0, 0), (0, 1), (1, 0), (1, 1), (2, 0)])
def test_table3_tiles_equal_streaming(hip_device, layout, precision, block):
    import torch

    print(f"[table3] {layout} precision {precision} block {block}", flush=True)
    o, e = synth.tensor_layout(LAYOUTS[layout])
    w = synth.Workload("table3", 3, 3, o, e, 63, 2, 3, "elasticity", h=0.1, seed=layout)
    b = harness.to_dev(synth.rhs(w))
    got = []
    for table in (1, 0):
        # tile_planes forces the tiles on levels of any size
        h = harness.gpu_problem(w, tile_planes=21, region_table=table, precision=precision, block_diag=block)
        if precision == 0:
            assert h.level_table_regions(0) == (len(e) if table else 0)
        z = torch.empty_like(b)
        h.apply_vcycle(b, z)
        n = h.level_info(0)["n_regional"]
        v = torch.from_numpy(np.random.RandomState(1).uniform(-1, 1, n)).to("cuda:0")
        y = torch.empty_like(v)
        h.regional_matvec(0, v, y)
        x = torch.zeros_like(b)
        out = h.solve(b, x, rtol=1e-8, maxit=60)
        got.append((z, y, x, out))
        h.close()
    assert torch.equal(got[0][0], got[1][0])
    assert torch.equal(got[0][1], got[1][1])
    assert got[0][3]["iterations"] == got[1][3]["iterations"]
    harness.assert_close(got[0][2].cpu().numpy(), got[1][2].cpu().numpy(), 1e-12 if precision == 0 else 1e-7)
