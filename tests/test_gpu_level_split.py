"""The path that a level's stencil operations take, as rmg_level_split reports it, where the results of the
paths are compared: element tiles up to rows of 339 nodes and streaming above, and the class tables
of a low-precision V-cycle in whole-row tiles (3 dofs, FP32 2.5D tiles) and node blocks.
"""
import numpy as np
import pytest

import synth
from tests import harness

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("ex", [300, 339, 340])
@pytest.mark.parametrize("mask", [63, 0b010110])
def test_elem_tiles_run(hip_device, ex, mask):
    import torch

    from paper_2103_11962_amd import regmg

    print(f"[split] element rows of {ex}, mask {mask}", flush=True)
    o, e = synth.tensor_layout([[ex], [5, 4], [4]])
    w = synth.Workload("elemrow", 3, 1, o, e, mask, 2, 3, "diffusion", h=0.1, seed=1)
    ec = torch.from_numpy(np.ascontiguousarray(synth.jump_coefficients(w))).to("cuda:0").reshape(-1)
    b = harness.to_dev(synth.rhs(w))
    got = []
    for table in (1, 0):
        h = regmg.Handle(0)
        h.build_regions(3, 1, e, o, mask)
        h.assemble_q1(regmg.PDE_DIFFUSION, w.h, elem_coef=ec)
        h.setup_hierarchy(nlevels=2, cheb_degree=3, stencil_kernel=2, region_table=table)
        s = h.level_split(0)
        assert (s["elem_tiles"] > 0) == (table == 1 and ex < 340) and s["table_tiles"] == 0 and s["regions_lo"] == 0
        z = torch.empty_like(b)
        h.apply_vcycle(b, z)
        got.append(z)
        h.close()
    assert torch.equal(got[0], got[1])


@pytest.mark.parametrize("ndof,precision,opts,tiles", [
    (3, 0, dict(tile_planes=21), True),
    (3, 1, dict(tile_planes=21), True),
    (3, 2, dict(tile_planes=21), True),
    (3, 1, dict(), False),
    (1, 1, dict(stencil_kernel=2), True),
    (1, 1, dict(), False),
    (1, 2, dict(), False),
])
def test_table_path(hip_device, ndof, precision, opts, tiles):
    o, e = synth.tensor_layout([[10, 7], [9], [12, 8]])
    pde = "elasticity" if ndof == 3 else "laplace"
    w = synth.Workload("tabpath", 3, ndof, o, e, 63, 2, 3, pde, h=0.1, seed=1)
    for table in (1, 0):
        h = harness.gpu_problem(w, precision=precision, region_table=table, **opts)
        s = h.level_split(0)
        assert (s["table_tiles"] > 0) == (tiles and table == 1) and s["elem_tiles"] == 0
        assert s["regions_lo"] == (len(e) if table and precision else 0)
        assert h.level_table_regions(0) == (len(e) if table and not precision else 0)
        h.close()
