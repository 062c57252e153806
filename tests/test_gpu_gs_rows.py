"""Gauss-Seidel sweeps of 2D levels at the edges of the row-wavefront kernel's ranges.

A wavefront owns 64 rows of a region and chunks are 16, 8 or 4 steps long with up to 4, 8 or 16
wavefronts; regions of more than 1024 rows take the hyperplane kernel.  One V-cycle with forward
sweeps before and backward sweeps after the coarse correction (five-point finest level, nine-point
level below) against the oracle, at the FP64 tolerance of the other cycle tests.
"""
import numpy as np
import pytest

import synth
from tests import harness

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("rows", [2, 63, 64, 65, 129, 256, 257, 513, 771, 1030])
@pytest.mark.parametrize("cols", [(5, 18), (2, 70)])
def test_gs_rows_vcycle(hip_device, rows, cols):
    import torch

    from oracle import regional

    print(f"[gs rows] {rows} x {cols}", flush=True)
    o, e = synth.tensor_layout([list(cols), [rows, 20]])
    w = synth.Workload("gs_rows", 2, 1, o, e, 15, 3, 1, "fd5", seed=3)
    lay, levels, opt = harness.oracle_problem(w, smoother="sgs", jacobi_omega=0.9)
    b = synth.rhs(w)
    h = harness.gpu_problem(w, smoother=3, jacobi_omega=0.9)
    z = torch.empty(lay.n_composite, dtype=torch.float64, device="cuda:0")
    h.apply_vcycle(harness.to_dev(b), z)
    ref = lay.to_composite_owner(regional.vcycle(levels, lay.to_regional(b), opt)).reshape(-1)
    harness.assert_close(z.cpu().numpy(), ref, 1e-12)
    h.close()
