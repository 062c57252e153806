"""From which sizes, and how full, levels without 2.5D tiles run table and element tiles (rmg_level_split), in FP64
and around an FP32 cycle, and that either side of each line computes the same V-cycle.
"""
import numpy as np
import pytest

import synth
from tests import harness

pytestmark = pytest.mark.gpu

# (regions a side, extent, problem, options, table tiles, element tiles, regions on low-precision tables)
CASES = [
    (2, 28, "laplace", dict(), False, False, 0),
    (2, 36, "laplace", dict(), False, False, 0),  # 373,000 nodes
    (3, 25, "laplace", dict(), True, False, 0),  # 422,000
    (10, 8, "laplace", dict(), False, False, 0),  # planes of 64 nodes
    (1, 66, "laplace", dict(), False, False, 0),  # 287,000
    (1, 70, "laplace", dict(), True, False, 0),  # 343,000, long rows
    (2, 37, "laplace", dict(precision=1), False, False, 8),
    (3, 30, "laplace", dict(precision=1), False, False, 0),  # 729,000: streams
    (3, 31, "laplace", dict(precision=1), True, False, 27),  # 804,000
    (1, 100, "laplace", dict(precision=1), False, False, 1),  # 1.0M: class rows on node blocks
    (3, 46, "laplace", dict(precision=1), True, False, 27),
    (8, 12, "laplace", dict(precision=1), False, False, 0),
    (3, 25, "diffusion", dict(), False, False, 0),
    (2, 34, "diffusion", dict(), False, False, 0),  # 314,000
    (2, 35, "diffusion", dict(), False, True, 0),  # 343,000, edge 35
    (3, 31, "diffusion", dict(), False, True, 0),
    (3, 31, "diffusion", dict(precision=1), False, True, 0),
]


@pytest.mark.parametrize("case", range(len(CASES)))
def test_table_rules(hip_device, case):
    import torch

    from paper_2103_11962_amd import regmg

    r, ex, pde, opts, table, elem, lo = CASES[case]
    print(f"[rules] {CASES[case]}", flush=True)
    o, e = synth.tensor_layout([[ex] * r] * 3)
    w = synth.Workload("rules", 3, 1, o, e, 63, 3, 2, pde, h=0.1, seed=case)
    ec = None
    if pde == "diffusion":
        g = torch.Generator(device="cuda:0")
        g.manual_seed(case)
        ec = torch.empty([n - 1 for n in w.composite_shape], dtype=torch.float64, device="cuda:0").normal_(generator=g).exp_()
    b = harness.to_dev(np.random.RandomState(1).uniform(-1, 1, w.composite_shape))
    got = []
    for on in (1, 0):
        h = regmg.Handle(0)
        h.build_regions(3, 1, e, o, 63)
        h.assemble_q1(regmg.PDE_DIFFUSION if ec is not None else regmg.PDE_LAPLACE, w.h,
                      elem_coef=None if ec is None else ec.reshape(-1))
        h.setup_hierarchy(nlevels=3, cheb_degree=2, region_table=on, **opts)
        if on:
            s = h.level_split(0)
            assert h.level_tiles(0)["ntiles"] == 0
            assert (s["table_tiles"] > 0, s["elem_tiles"] > 0, s["regions_lo"]) == (table, elem, lo), s
        z = torch.empty_like(b)
        h.apply_vcycle(b, z)
        got.append(z)
        h.close()
    assert torch.equal(got[0], got[1])


def test_fp32_small_planes_stream_on_tiles(hip_device):
    """2197 regions of 8^3 run 2.5D tiles by default: FP32 operations stream them, a forced tile kernel
    takes table tiles."""
    import torch

    o, e = synth.tensor_layout([[8] * 13] * 3)
    w = synth.Workload("planes", 3, 1, o, e, 63, 3, 2, "laplace", h=0.1)
    b = harness.to_dev(np.random.RandomState(1).uniform(-1, 1, w.composite_shape))
    got = []
    for opts, lo in ((dict(), 0), (dict(stencil_kernel=2), 2197), (dict(region_table=0), 0)):
        h = harness.gpu_problem(w, precision=1, **opts)
        assert h.level_tiles(0)["ntiles"] > 0 and h.level_split(0)["regions_lo"] == lo
        z = torch.empty_like(b)
        h.apply_vcycle(b, z)
        got.append(z)
        h.close()
    assert torch.equal(got[0], got[2])


# (extents, options, table tiles): 3-dof levels by size and by the shorter edge of their planes
CASES3 = [
    ([[28] * 3] * 3, dict(), False),  # 593,000 nodes, edge 28
    ([[40] * 3] * 3, dict(), False),  # 1.7M, edge 40
    ([[50] * 2] * 3, dict(), False),  # 1.0M, edge 50
    ([[46] * 2] * 3, dict(precision=1), True),  # 779,000, edge 46, FP32
    ([[44] * 2] * 3, dict(precision=1), False),  # 681,000
    ([[58] * 2] * 3, dict(), True),  # 1.6M, edge 58
    ([[97], [97], [97]], dict(), True),  # 913,000, edge 97
    ([[97], [97], [97]], dict(precision=1), True),
    ([[25, 30], [61, 61], [120, 120]], dict(), False),  # 1.6M, short rows
    ([[61, 61], [25, 30], [120, 120]], dict(), False),  # 1.6M, short planes
    ([[10, 7], [9], [12]], dict(tile_planes=21), True),  # asked for
]


@pytest.mark.parametrize("case", range(len(CASES3)))
def test_table3_rules(hip_device, case):
    ext, opts, table = CASES3[case]
    print(f"[rules3] {CASES3[case]}", flush=True)
    o, e = synth.tensor_layout(ext)
    w = synth.Workload("rules3", 3, 3, o, e, 63, 4 if len(e) > 2 or ext[0][0] > 50 else 2, 2, "elasticity", h=0.1, seed=case)
    h = harness.gpu_problem(w, **opts)
    assert (h.level_split(0)["table_tiles"] > 0) == table
    assert len(e) == (h.level_split(0)["regions_lo"] if opts.get("precision") else h.level_table_regions(0))
    h.close()
