"""Device memory across operator changes and repeated setups, counted by a memory provider: staging buffers of the
calls that hand an operator over go back with the call, a setup with other options never holds the old
hierarchy beside the new one, a repeated one asks for no large buffer again, and everything is
returned when the handle closes.
"""
import numpy as np
import pytest

import synth
from tests import harness

pytestmark = pytest.mark.gpu
LARGE = 1 << 20


class Counter:
    def __init__(self):
        import torch

        from paper_2103_11962_amd import regmg

        self.size, self.live, self.peak, self.large = {}, 0, 0, 0

        def alloc(nbytes, ctx):
            p = torch.cuda.caching_allocator_alloc(int(nbytes), device=0, stream=torch.cuda.current_stream(0))
            self.size[p] = int(nbytes)
            self.live += int(nbytes)
            self.peak = max(self.peak, self.live)
            self.large += nbytes >= LARGE
            return p

        def free(ptr, ctx):
            self.live -= self.size.pop(ptr)
            torch.cuda.caching_allocator_delete(ptr)

        self.provider = regmg.Allocator(regmg.ALLOC_FN(alloc), regmg.FREE_FN(free), None)


def layout():
    # ragged regions: every staging buffer has a size of its own
    return synth.tensor_layout([[22, 25], [24, 31], [20]])


def test_region_stencils_leave_no_staging(hip_device):
    from paper_2103_11962_amd import regmg

    o, e = layout()
    c = Counter()
    h = regmg.Handle(0, allocator=c.provider)
    h.build_regions(3, 1, e, o, 63)
    w = synth.Workload("x", 3, 1, o, e, 63, 2, 2, "laplace", h=0.1)
    src = harness.gpu_problem(w, setup=False)
    held = []
    for _ in range(2):
        for k, n in enumerate(np.prod(e, axis=1)):
            h.set_region_stencil(k, 27, src.level_stencil(0, k, 27, int(n)))
            held.append(c.live)
    assert held == [held[0]] * len(held)
    src.close()
    h.close()
    assert c.live == 0


@pytest.mark.parametrize("form", ["stencil", "csr"])
def test_composite_operator_leaves_no_staging(hip_device, form):
    import scipy.sparse as sp

    from paper_2103_11962_amd import regmg

    o, e = synth.tensor_layout([[150, 130], [160, 141]])
    w = synth.Workload("x", 2, 1, o, e, 15, 2, 2, "fd5")
    st = synth.fd5_composite_stencil(w)
    c = Counter()
    h = regmg.Handle(0, allocator=c.provider)
    h.build_regions(2, 1, e, o, 15)
    h.set_composite_stencil(5, st)
    held = c.live
    if form == "csr":
        ny, nx = w.composite_shape
        st = np.asarray(st).reshape(5, ny, nx)
        offs = [(0, -1), (-1, 0), (0, 0), (1, 0), (0, 1)]
        jj, ii = np.meshgrid(np.arange(ny), np.arange(nx), indexing="ij")
        rows, cols, vals = [], [], []
        for s, (dx, dy) in enumerate(offs):
            ok = (ii + dx >= 0) & (ii + dx < nx) & (jj + dy >= 0) & (jj + dy < ny)
            rows.append((jj * nx + ii)[ok])
            cols.append(((jj + dy) * nx + ii + dx)[ok])
            vals.append(st[s][ok])
        A = sp.csr_matrix((np.concatenate(vals), (np.concatenate(rows), np.concatenate(cols))), shape=(nx * ny,) * 2)
    for _ in range(2):
        if form == "csr":
            h.set_composite_csr(5, A)
        else:
            h.set_composite_stencil(5, st)
        assert c.live == held
    h.close()
    assert c.live == 0


def test_setups_of_other_and_of_same_options(hip_device):
    from paper_2103_11962_amd import regmg

    o, e = synth.tensor_layout([[46, 43], [40, 37], [43]])

    def handle():
        c = Counter()
        h = regmg.Handle(0, allocator=c.provider)
        h.build_regions(3, 1, e, o, 63)
        h.assemble_q1(regmg.PDE_LAPLACE, 0.1)
        return c, h

    c0, h0 = handle()  # a first FP64 setup
    h0.setup_hierarchy(nlevels=3, cheb_degree=2)
    above = c0.peak - c0.live  # beyond what the setup keeps
    h0.close()
    c, h = handle()
    h.setup_hierarchy(nlevels=3, cheb_degree=2, precision=1)
    before, c.peak = c.live, 0
    h.setup_hierarchy(nlevels=3, cheb_degree=2)
    # at most what it starts from, or what it keeps and a first setup's intermediates
    assert c.peak <= max(before, c.live + above), (c.peak, before, c.live, above)
    h.assemble_q1(regmg.PDE_LAPLACE, 0.1)
    h.setup_hierarchy(nlevels=3, cheb_degree=2)
    c.large = 0
    for _ in range(2):
        h.assemble_q1(regmg.PDE_LAPLACE, 0.1)
        h.setup_hierarchy(nlevels=3, cheb_degree=2)
    # a repeat asks only for the Galerkin product's intermediates (held for one setup only)
    assert c.large <= 2 * 4, c.large
    h.close()
    assert c.live == c0.live == 0


@pytest.mark.parametrize("opts", [dict(region_table=0), dict(symmetric=0), dict(batched=0)])
def test_element_coefficients_only_where_used(hip_device, opts):
    """A setup that always streams gives the kept element coefficients back: beside the Laplacian's, the
    diffusion operator's handle then holds the network's FP32 features only."""
    import torch

    from paper_2103_11962_amd import regmg

    o, e = synth.tensor_layout([[46, 43], [40], [43]])
    cells = [int(v) for v in (o + e).max(axis=0) - 1]
    elements = int(np.prod(cells))
    ec = torch.ones(elements, dtype=torch.float64, device="cuda:0")
    held = []
    for pde, coef in ((regmg.PDE_LAPLACE, None), (regmg.PDE_DIFFUSION, ec)):
        c = Counter()
        h = regmg.Handle(0, allocator=c.provider)
        h.build_regions(3, 1, e, o, 63)
        h.assemble_q1(pde, 0.1, elem_coef=coef)
        h.setup_hierarchy(nlevels=3, cheb_degree=2, **opts)
        held.append(c.live)
        h.close()
        assert c.live == 0
    assert held[1] - held[0] == 4 * elements
