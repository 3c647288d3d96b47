"""The spherical gather and input layout over batch sizes and grid sizes: the sums
of a voxel's visits are cut by the number of voxels alone, so a batch entry is
bitwise the single-wavelength result on either side of every size at which runs
get threads of their own, blocks hold one voxel or less, or the input's tiles of
64 voxels and 16 wavelengths end; the oracle agrees as for the other formal
solutions of the sphere (rounding only, 1e-12, in double)."""
import dataclasses

import numpy as np
import pytest

import synthetic as sy
from tests.gpu_helpers import gpu_fs, make_grid

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("prec", ["f64", "f32"])
@pytest.mark.parametrize("dims,n_lambda", [((7, 6, 8, 4, 4), 16), ((7, 6, 8, 4, 4), 33), ((5, 4, 3, 2, 4), 257),
                                           ((1, 1, 1, 2, 2), 3), ((41, 40, 40, 2, 2), 3), ((41, 40, 40, 2, 2), 65),
                                           ((82, 80, 80, 2, 2), 2)])
def test_batch_entries_equal_single_wavelengths(orc, dims, n_lambda, prec):
    Nr, Nt, Np, n_mu, n_phi = dims
    case = sy.random_sphere(Nr, Nt, Np, n_mu, n_phi, seed=Nr + n_lambda, dtype=prec, n_lambda=n_lambda)
    S = sy.random_source(case.chi.shape, seed=5, dtype=prec)
    print(dims, n_lambda, prec, flush=True)
    g = make_grid(case)
    J, L = gpu_fs(case, S, grid=g)
    g.close()
    for l in sorted({0, n_lambda // 2, n_lambda - 1}):
        one = dataclasses.replace(case, chi=case.chi[l:l + 1], eps=case.eps[l:l + 1], B=case.B[l:l + 1],
                                  I_bc=case.I_bc[l:l + 1])
        g = make_grid(one, n_lambda_max=1)
        J1, L1 = gpu_fs(one, S[l:l + 1], grid=g)
        g.close()
        np.testing.assert_array_equal(J1[0], J[l])
        np.testing.assert_array_equal(L1[0], L[l])
    if prec == "f64" and case.n_vox < 100000:
        gs = orc.SphereGrid(Nr, Nt, Np, case.r_core, case.r_out)
        l = n_lambda - 1
        I_out, I_core, J_sub = case.I_bc[l]
        Jr, Lr = orc.fs_sphere(gs, n_mu, n_phi, case.chi[l], S[l], np.full(case.n_vox, I_core), I_out=I_out,
                               dsrc=case.source_distance, B_sub=J_sub, kind="linear")
        np.testing.assert_allclose(J[l].ravel(), Jr.ravel(), rtol=1e-12, atol=1e-14)
        np.testing.assert_allclose(L[l].ravel(), Lr.ravel(), rtol=1e-12, atol=1e-14)


@pytest.mark.parametrize("value", [np.nan, 0.0])
def test_special_opacities_stay_on_their_characteristics(value):
    """A voxel of NaN or zero opacity: single precision treats it as the
    double-precision sweep does (NaN where and only where that has NaN)."""
    case = sy.random_sphere(8, 6, 9, 2, 4, seed=3, dtype="f64", n_lambda=1)
    case.chi[0].flat[0] = value
    case.chi[0].flat[case.n_vox // 2] = value
    S = sy.random_source(case.chi.shape, seed=6)
    J64, L64 = gpu_fs(case, S)
    J32, L32 = gpu_fs(dataclasses.replace(case, dtype="f32"), S, prec="f32")
    np.testing.assert_array_equal(np.isnan(J32), np.isnan(J64))
    ok = ~np.isnan(J64)
    np.testing.assert_allclose(J32[ok], J64[ok], rtol=2e-5, atol=1e-6 * np.abs(J64[ok]).max())
