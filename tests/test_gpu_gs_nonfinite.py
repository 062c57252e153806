"""Gauss-Seidel sweeps of 2D levels with one infinite right-hand side entry: the forward sweep carries it to the
nodes that the lower triangle reaches from there and to no other (rmg_smooth from a zero guess, one
region): five-point stencils reach x' >= x, y' >= y, nine-point ones one node further left a row.
"""
import numpy as np
import pytest

import synth
from tests import harness

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("ext", [(150, 140), (61, 300)])
@pytest.mark.parametrize("level", [0, 1])
@pytest.mark.parametrize("where", [(1.0, 0.5), (0.5, 0.5), (0.0, 0.4), (1.0, 0.9), (0.9, 0.0)])
def test_infinite_entry_stays_downstream(hip_device, ext, level, where):
    import torch

    print(f"[gs inf] {ext} level {level} at {where}", flush=True)
    o, e = synth.tensor_layout([[ext[0]], [ext[1]]])
    w = synth.Workload("gsinf", 2, 1, o, e, 15, 3, 1, "fd5", seed=3)
    h = harness.gpu_problem(w, smoother=2, jacobi_omega=1.0)
    nx, ny = ext
    for _ in range(level):
        nx, ny = (nx + 1) // 3 + 1, (ny + 1) // 3 + 1
    b = np.random.default_rng(5).uniform(-1, 1, (ny, nx))
    x, y = int(round(where[0] * (nx - 1))), int(round(where[1] * (ny - 1)))
    b[y, x] = np.inf
    u = torch.zeros(nx * ny, dtype=torch.float64, device="cuda:0")
    h.smooth(level, harness.to_dev(b), u)
    yy, xx = np.meshgrid(np.arange(ny), np.arange(nx), indexing="ij")
    left = x if level == 0 else x - (yy - y)
    reached = np.where(yy == y, xx >= x, (yy > y) & (xx >= left))
    got = ~np.isfinite(u.cpu().numpy().reshape(ny, nx))
    assert not (got & ~reached).any(), np.argwhere(got & ~reached)[:5]
    assert got[y, x]
    h.close()
