"""Thick steps beside a much stronger source on the shell: the upwind weight of a step
D is about 1/D, the small rest of e0 - beta - gamma, so an error of the weights that
is small beside beta = 1 - 1/D may still be the whole of it."""
import numpy as np
import pytest

from tests.gpu_helpers import to_dev, torch_cuda

pytestmark = pytest.mark.gpu

HOT = 1e8


# Beside the hot layer J is a sum of weights of at most 2/D times HOT.  Single
# precision rounds each weight, the geometry (path lengths, averaging weights) and
# every step of the recurrence by 6e-8 of itself, about ten roundings in all: 1e-6 of
# the largest term, and ten in hand.
@pytest.mark.parametrize("lam", [1, 16])
def test_thick_steps_beside_a_hot_layer(lam):
    import paper_2102_01734_amd as rt
    torch = torch_cuda()
    nr, nt, npp = 9, 8, 10
    shape = (lam, npp, nt, nr)
    rng = np.random.default_rng(7)
    chi = (10.0 ** rng.uniform(7.5, 8.5, shape)).astype(np.float32)
    S = rng.uniform(0.5, 1.5, shape).astype(np.float32)
    S[..., 4] *= HOT
    J = {}
    for prec in ("f64", "f32"):
        g = rt.SphereGrid(nr, nt, npp, 1.0, 2.0, 4, 8, prec, lam)
        J[prec] = g.formal_solution(to_dev(chi, prec), to_dev(S, prec))[0].double()
        torch.cuda.synchronize()
        g.close()
    a, b = J["f32"].cpu().numpy(), J["f64"].cpu().numpy()
    beside = np.zeros(shape, bool)
    beside[..., [3, 5]] = True
    thin = float(b[beside].max())  # the largest terms there
    print("lam", lam, "beside the hot layer: J", b[beside].min(), thin, "error", np.abs(a - b)[beside].max(), flush=True)
    assert b[beside].max() > 5.0  # the hot layer is what they see
    np.testing.assert_allclose(a[beside], b[beside], rtol=1e-5, atol=1e-5 * thin)
    np.testing.assert_allclose(a[..., 4], b[..., 4], rtol=1e-5)
