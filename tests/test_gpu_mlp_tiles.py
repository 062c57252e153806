"""Loss and gradient of the interpolation network at sample counts around the matrix-core kernels'
tiles (32 samples a wavefront, 256 a block, slices of a multiple of 16 samples): against the FP64 oracle,
to the FP32 bounds of the other training tests, and the first gradient repeated bit for bit."""
import numpy as np
import pytest

import synth
from tests import harness

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("loss", ["l2", "energy"])
@pytest.mark.parametrize("n", [1, 2, 15, 31, 32, 33, 63, 65, 255, 257, 1040, 8209])
def test_loss_and_gradient_at_tile_edges(hip_device, n, loss):
    from oracle import learned
    from paper_2103_11962_amd import regmg

    print(f"[mlp tiles] {n} {loss}", flush=True)
    rng = np.random.Generator(np.random.PCG64(n))
    X = rng.standard_normal((n, 27)).astype(np.float32)
    E = rng.standard_normal((n, 64)).astype(np.float32)
    if n > 2:
        E[1] = 0.0  # a cell without error: norm taken as 1
    theta = synth.mlp_params(3, out_scale=0.5)
    m = regmg.Mlp(0)
    m.set_loss(regmg.MLP_LOSS_ENERGY if loss == "energy" else regmg.MLP_LOSS_L2)
    m.set_params(theta)
    m.add_data(X, E)
    got, g = m.loss_grad()
    again, g2 = m.loss_grad()
    ref, gr = learned.loss_and_grad(theta, X.astype(np.float64), E.astype(np.float64).reshape(n, 4, 4, 4), kind=loss)
    assert again == got and np.array_equal(g, g2)
    assert abs(got - ref) <= 1e-5 * abs(ref)
    harness.assert_close(g, gr, 1e-4, floor=1.0, what="gradient")
    m.close()
