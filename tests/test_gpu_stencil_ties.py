"""The linear nearest-neighbour Lambda* on quadratures whose templates cross two faces at
once (45 degrees; path ratios of three), which goes by windows of rows from 400000
characteristics on (the last four of these): bit for bit the stencil of one thread per characteristic, as the sums are integers and both spell out
their rounding.  Few rows and rays, one and two rays a thread, several wavelengths,
vacuum, opaque and non-finite opacities."""
import numpy as np
import pytest

import synthetic as sy
from tests.test_gpu_near_stencil import _stencil

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("prec", ["f64", "f32"])
@pytest.mark.parametrize("dims", [(1, 1, 2, 4, 4, 1), (2, 3, 4, 2, 3, 1), (9, 8, 6, 4, 12, 2), (33, 31, 5, 36, 12, 1),
                                  (230, 220, 3, 2, 4, 1), (9, 8, 4, 40, 36, 4), (66, 65, 5, 8, 12, 1)])
def test_rows_equal_per_characteristic(dims, prec, monkeypatch):
    Nx, Ny, Nz, n_mu, n_phi, n_lambda = dims
    print(dims, prec, flush=True)
    case = sy.random_box(Nx, Ny, Nz, n_mu, n_phi, seed=Nx + Nz, dtype=prec, n_lambda=n_lambda)
    if Nx == 9:
        case.chi[0].flat[::7] = 0.0
        case.chi[0].flat[3::11] = 1e8
        case.chi[1].flat[100] = np.nan
        case.chi[1].flat[200] = np.inf
    a = _stencil(case)
    monkeypatch.setenv("RT3D_STENCIL_PER_CHARACTERISTIC", "1")
    np.testing.assert_array_equal(a, _stencil(case))
