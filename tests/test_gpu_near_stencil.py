"""The voxel-wise kernel of the linear nearest-neighbour Lambda* against one thread
per characteristic: contributions are the same numbers and the sums are integers, so
the stencils are equal bit for bit.  Grids of one and two voxels a side (a voxel is
its own neighbour across the period), layers of one wavefront and just more, one
layer, few and many directions (octants without any, split over blocks), vacuum,
opaque and NaN voxels, several wavelengths."""
import numpy as np
import pytest

import synthetic as sy
from tests.gpu_helpers import make_grid, to_dev, torch_cuda

pytestmark = pytest.mark.gpu


def _stencil(case):
    torch = torch_cuda()
    g = make_grid(case)
    out = g.lstar_stencil(to_dev(case.chi, case.dtype))
    torch.cuda.synchronize()
    res = out.cpu().numpy()
    g.close()
    return res


@pytest.mark.parametrize("prec", ["f64", "f32"])
@pytest.mark.parametrize("dims", [(1, 1, 1, 2, 1, 1), (1, 2, 3, 2, 3, 1), (2, 3, 2, 4, 8, 2), (8, 8, 4, 2, 4, 1),
                                  (13, 5, 6, 8, 16, 3), (3, 4, 9, 16, 1, 1), (33, 31, 5, 4, 6, 1)])
def test_voxelwise_equals_per_characteristic(dims, prec, monkeypatch):
    Nx, Ny, Nz, n_mu, n_phi, n_lambda = dims
    print(dims, prec, flush=True)
    case = sy.random_box(Nx, Ny, Nz, n_mu, n_phi, seed=Nx + Nz, dtype=prec, n_lambda=n_lambda)
    a = _stencil(case)
    monkeypatch.setenv("RT3D_STENCIL_PER_CHARACTERISTIC", "1")
    np.testing.assert_array_equal(a, _stencil(case))


@pytest.mark.parametrize("prec", ["f64", "f32"])
def test_special_opacities(prec, monkeypatch):
    case = sy.random_box(12, 9, 8, 4, 8, seed=5, dtype=prec, n_lambda=2)
    case.chi[0].flat[::7] = 0.0
    case.chi[0].flat[3::11] = 1e8
    case.chi[1].flat[100] = np.nan
    case.chi[1].flat[500] = np.inf
    case.chi[1].flat[700] = -1.0
    a = _stencil(case)
    monkeypatch.setenv("RT3D_STENCIL_PER_CHARACTERISTIC", "1")
    np.testing.assert_array_equal(a, _stencil(case))
