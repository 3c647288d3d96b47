"""A small batch runs the launch shape of a single wavelength as long as that shape's
workgroups of a ray bundle are at least its wavelengths times directions: every direction
has a partial sum of its own and the batch gives each wavelength's results bit for bit.
Beyond that, directions share partial sums in another order."""
import numpy as np
import pytest

import synthetic as sy
from tests.gpu_helpers import make_grid, to_dev, torch_cuda

pytestmark = pytest.mark.gpu

# 128 positive terms in the field precision, in two orders: 128 roundings of the sum
ROUNDINGS = {"f64": 128 * 1.2e-16, "f32": 128 * 6e-8}


@pytest.mark.parametrize("prec", ["f64", "f32"])
@pytest.mark.parametrize("nx,n_mu,n_phi,lam,own", [(13, 4, 8, 3, True), (24, 8, 16, 2, None), (46, 8, 16, 3, None),
                                                   (46, 8, 13, 4, False)])
def test_batch_against_its_wavelengths(nx, n_mu, n_phi, lam, own, prec):
    torch = torch_cuda()
    case = sy.random_box(nx, 45, 5, n_mu, n_phi, seed=nx, dtype=prec, n_lambda=lam)
    S = to_dev(sy.random_source(case.chi.shape, seed=3, dtype=prec), prec)
    chi, bc = to_dev(case.chi, prec), to_dev(case.I_bc, prec)
    single = make_grid(case, n_lambda_max=1)
    per_bundle = single.info()["n_workgroups"] // single.launch_shape()["bundles"]
    single.close()
    g = make_grid(case)
    fits = lam * n_mu * n_phi <= per_bundle
    print(nx, n_mu * n_phi, lam, prec, g.launch_shape(), "workgroups a bundle", per_bundle, fits, flush=True)
    assert own is None or fits == own
    J = g.formal_solution(chi, S, bc)[0].cpu().numpy()
    for l in range(lam):
        one = g.formal_solution(chi[l:l + 1].contiguous(), S[l:l + 1].contiguous(), bc[l:l + 1].contiguous())[0]
        one = one.cpu().numpy()[0]
        if fits:
            assert (one == J[l]).all()
        else:
            np.testing.assert_allclose(one, J[l], rtol=ROUNDINGS[prec])
    torch.cuda.synchronize()
    g.close()
