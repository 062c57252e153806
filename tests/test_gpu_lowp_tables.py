"""FP32 V-cycle on levels too small for 2.5D tiles by default: where table tiles run such a level, the
cycle must equal the streamed one (region_table = 0, node blocks) bit for bit.
"""
import pytest

import synth
from tests import harness

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("ext", [[[110], [104], [103]], [[62, 55], [60, 57], [60, 62]]])
@pytest.mark.parametrize("degree", [1, 3])
def test_fp32_table_tiles_equal_node_blocks(hip_device, ext, degree):
    import torch

    print(f"[lowp tables] {ext} degree {degree}", flush=True)
    o, e = synth.tensor_layout(ext)
    w = synth.Workload("lowptab", 3, 1, o, e, 63, 4, degree, "laplace", h=0.1, seed=3)
    b = harness.to_dev(synth.rhs(w))
    got = []
    for table in (1, 0):
        h = harness.gpu_problem(w, precision=1, region_table=table)
        s = h.level_split(0)
        assert h.level_tiles(0)["ntiles"] == 0 and (s["table_tiles"] > 0) == (table == 1), s
        z = torch.empty_like(b)
        h.apply_vcycle(b, z)
        got.append(z)
        h.close()
    assert torch.equal(got[0], got[1])
