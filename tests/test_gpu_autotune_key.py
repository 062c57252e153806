"""Autotuner choices belong to the kernels they were timed on: a choice written without class tables is not read for
a level that they serve, nor one of other regions; levels that table tiles cover have no choice of depth
or grid; a choice of shallower tiles than the default has room for its partial sums.
"""
import re

import numpy as np
import pytest

import synth
from tests import harness

pytestmark = pytest.mark.gpu


def test_choice_is_not_shared(hip_device, tmp_path):
    cache = str(tmp_path / "tune.txt")
    o, e = synth.tensor_layout([[28, 31], [28], [28, 25]])
    w = synth.Workload("key", 3, 1, o, e, 63, 2, 2, "laplace", h=0.1)
    runs = [dict(region_table=0), dict(region_table=1), dict(region_table=0), dict(region_table=1)]
    for k, opts in enumerate(runs):
        h = harness.gpu_problem(w, autotune=1, autotune_cache=cache, **opts)
        assert h.tune_report().count("cached") == (1 if k >= 2 else 0), (k, h.tune_report())
        h.close()
    # as many nodes and regions, the first four extents alike, the others not
    for last in ([20, 20, 29], [20, 29, 20]):
        o, e = synth.tensor_layout([[20], [20], [20, 20] + last])
        h = harness.gpu_problem(synth.Workload("key", 3, 1, o, e, 63, 2, 2, "laplace", h=0.1), autotune=1,
                                autotune_cache=cache)
        assert "cached" not in h.tune_report(), (last, h.tune_report())
        h.close()


@pytest.mark.parametrize("precision", [0, 1])
def test_covered_levels_have_two_candidates(hip_device, tmp_path, precision):
    o, e = synth.tensor_layout([[40, 31], [28], [28, 25]])
    w = synth.Workload("covered", 3, 1, o, e, 63, 2, 2, "laplace", h=0.1)
    for _ in range(3):
        h = harness.gpu_problem(w, stencil_kernel=2, tile_planes=41, precision=precision, autotune=1)
        assert re.search(r"mode [01] depth 41 grid 0 ", h.tune_report()), h.tune_report()
        h.close()


def test_shallow_tiles_have_room(hip_device, tmp_path):
    """256 columns of 2 x 2 x 12 nodes: one node block a region, two tiles of eleven planes at most."""
    import torch

    cache = tmp_path / "tune.txt"
    print("[autotune] shallow tiles", flush=True)
    o, e = synth.tensor_layout([[2] * 16, [2] * 16, [12]])
    w = synth.Workload("shallow", 3, 1, o, e, 48, 2, 2, "laplace", h=0.1)
    b = harness.to_dev(synth.rhs(w))
    got = []
    for opts in (dict(autotune=1, autotune_cache=str(cache)), dict(autotune=1, autotune_cache=str(cache)), dict()):
        h = harness.gpu_problem(w, **opts)
        if got:
            assert ("cached mode 1 depth 11" in h.tune_report()) == bool(opts)
        x = torch.zeros_like(b)
        out = h.solve(b, x, rtol=1e-8, maxit=300)
        got.append((x.cpu().numpy(), out["iterations"]))
        h.close()
        if len(got) == 1:  # the same level, told to take eleven planes a tile
            cache.write_text(re.sub(r" \d+ \d+ \d+$", " 1 11 0", cache.read_text(), flags=re.M))
    for x, it in got[:2]:
        assert it == got[2][1]
        harness.assert_close(x, got[2][0], 1e-10)
