"""The restriction's kernels against one another, bit for bit, on coarse levels small enough for any of them: by
rows and planes (batched = 0, transfer_rows = 1), one thread per coarse node with the interface sum after
it (transfer_rows = 0) and both in one launch (the default there, one launch less).
"""
import numpy as np
import pytest

import synth
from tests import harness

pytestmark = pytest.mark.gpu

NAMES = ["c2_small", "c2_mid", "uneven3d_small", "uneven3e_small", "uneven_tiny3d", "c1_small", "uneven2d_small", "c3_small"]


@pytest.mark.parametrize("name", NAMES)
def test_restriction_paths_agree(hip_device, name):
    import torch

    from paper_2103_11962_amd import regmg

    print(f"[restriction] {name}", flush=True)
    w = synth.workload(name)
    rng = np.random.default_rng(7)
    hs = [harness.gpu_problem(w, **kw) for kw in (dict(), dict(transfer_rows=0), dict(batched=0), dict(batched=0, transfer_rows=0))]
    try:
        for l in range(w.nlevels - 1):
            nf, nc = hs[0].level_info(l)["n_regional"], hs[0].level_info(l + 1)["n_regional"]
            r = torch.from_numpy(rng.uniform(-1, 1, nf)).to("cuda:0")
            out, launches = [], []
            for h in hs:
                wc = torch.full((nc,), np.nan, dtype=torch.float64, device="cuda:0")
                before = regmg.kernel_launches()
                h.restrict(l, r, wc)
                launches.append(regmg.kernel_launches() - before)
                out.append(wc)
            for k in range(1, 4):
                assert torch.equal(out[0], out[k]), (l, k)
            # the same launches but for the interface sum (every layout here has shared nodes)
            assert launches[1] == launches[0] + 1, (l, launches)
            assert hs[2].level_transfer_tiles(l)["restriction"] > 0 and hs[3].level_transfer_tiles(l)["restriction"] == 0
    finally:
        for h in hs:
            h.close()


def counts_split(h, nf):
    """Launches of a restriction without its interface sum: fill, scaling product, one."""
    import torch

    from paper_2103_11962_amd import regmg

    v = torch.zeros(nf, dtype=torch.float64, device="cuda:0")
    before = regmg.kernel_launches()
    h.regional_matvec(0, v, torch.empty_like(v))
    return 2 + regmg.kernel_launches() - before


def test_restriction_line(hip_device):
    """Into a coarse level above either line the interface sum is a launch of its own."""
    import torch

    from paper_2103_11962_amd import regmg

    # (dofs, regions a side, extent, one launch): few copies, too many nodes, many copies (a line on 3 dofs)
    for ndof, r, ex, fused in ((1, 3, 46, True), (1, 4, 46, False), (1, 8, 15, True), (3, 6, 15, True), (3, 8, 15, False)):
        o, e = synth.tensor_layout([[ex] * r] * 3)
        w = synth.Workload("line", 3, ndof, o, e, 63, 3, 1, "elasticity" if ndof == 3 else "laplace", h=0.1)
        h = harness.gpu_problem(w)
        nf, nc = h.level_info(0)["n_regional"], h.level_info(1)["n_regional"]
        x = torch.zeros(nf, dtype=torch.float64, device="cuda:0")
        y = torch.empty(nc, dtype=torch.float64, device="cuda:0")
        counts = []
        for _ in range(2):
            before = regmg.kernel_launches()
            h.restrict(0, x, y)
            counts.append(regmg.kernel_launches() - before)
        assert counts[0] == counts[1]
        assert counts[0] - counts_split(h, nf) == (0 if fused else 1), (ndof, r, ex, counts)
        h.close()
