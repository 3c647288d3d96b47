"""Launch shapes of the box sweep by their estimated time: the shape of a call is
chosen from its wavelengths and directions, with as many ray bundles as keep the
chip busy.  At the edges of that choice (one ray column, layers just below and
above the size from which band tiles compete, items below and above the number of
compute units, the first and later items of a slot) results match the oracle with
the tolerances of the other formal-solution tests."""
import dataclasses

import numpy as np
import pytest

import synthetic as sy
from tests.gpu_helpers import gpu_fs, make_grid, to_dev, torch_cuda

pytestmark = pytest.mark.gpu


def _check(J, L, Jo, Lo, prec):
    tol = dict(rtol=1e-12, atol=1e-14) if prec == "f64" else dict(rtol=5e-6, atol=1e-7 * np.abs(Jo).max())
    np.testing.assert_allclose(J, Jo, **tol)
    np.testing.assert_allclose(L, Lo, rtol=1e-12 if prec == "f64" else 5e-6, atol=1e-14 if prec == "f64" else 1e-8)


@pytest.mark.parametrize("prec", ["f64", "f32"])
@pytest.mark.parametrize("dims", [(1, 1, 3, 2, 1, 1), (45, 45, 5, 4, 8, 1), (46, 45, 5, 4, 8, 1), (46, 45, 5, 4, 8, 9),
                                  (46, 45, 4, 8, 33, 2), (130, 20, 6, 4, 8, 1)])
def test_default_shapes_match_the_oracle(orc, dims, prec):
    Nx, Ny, Nz, n_mu, n_phi, n_lambda = dims
    case = sy.random_box(Nx, Ny, Nz, n_mu, n_phi, seed=Nx + Nz, dtype=prec, n_lambda=n_lambda)
    S = sy.random_source(case.chi.shape, seed=3, dtype=prec)
    g = make_grid(case, lstar="parabolic")
    print(dims, prec, g.launch_shape(), g.info()["n_workgroups"], flush=True)
    J, L = gpu_fs(case, S, grid=g)
    J1, _ = gpu_fs(case, S, grid=g, want_lstar=False)
    for l in {0, n_lambda - 1}:
        Jo, Lo = orc.fs_box(case.chi[l], S[l], case.I_bc[l, 0], case.I_bc[l, 1], n_mu, n_phi, kind="parabolic")
        _check(J[l], L[l], Jo, Lo, prec)
        _check(J1[l], L[l], Jo, Lo, prec)
    # a smaller call on the same grid, and a share of its directions, run shapes of their own
    if n_lambda > 1:
        one = dataclasses.replace(case, chi=case.chi[:1], eps=case.eps[:1], B=case.B[:1], I_bc=case.I_bc[:1])
        Ja, _ = gpu_fs(one, S[:1], grid=g, want_lstar=False)
        np.testing.assert_allclose(Ja[0], J1[0], rtol=1e-13 if prec == "f64" else 2e-6, atol=1e-7 * np.abs(J1).max())
    torch = torch_cuda()
    chi, St, Ib = to_dev(case.chi, prec), to_dev(S, prec), to_dev(case.I_bc, prec)
    total = sum(g.formal_solution_dirs(chi, St, g.shard_directions(2, k), Ib)[0].double() for k in range(2))
    torch.cuda.synchronize()
    np.testing.assert_allclose(total.cpu().numpy(), J1, rtol=1e-13 if prec == "f64" else 2e-6, atol=1e-7 * np.abs(J1).max())
    g.close()


@pytest.mark.parametrize("band", [False, True])
def test_default_shape_can_be_set_again(band):
    """Setting the shape a fresh grid reports reproduces its results bit for bit."""
    case = sy.random_box(33, 31, 6, 4, 8, seed=5, dtype="f32")
    S = sy.random_source(case.chi.shape, seed=6, dtype="f32")
    g = make_grid(case, band_tiles=band)
    J0, _ = gpu_fs(case, S, grid=g, want_lstar=False)
    ls = g.launch_shape()
    g.set_launch_shape(ls["threads"], ls["rays"], band=ls["band"])
    assert g.launch_shape() == ls
    J1, _ = gpu_fs(case, S, grid=g, want_lstar=False)
    g.close()
    assert np.array_equal(J0, J1)


def test_slot_sums_over_every_group_count(orc):
    """Partial slots are summed by 16, 4 or 1 wavefronts below 65536, below 262144
    and from 262144 voxels on."""
    for Nz in (15, 16, 63, 64):
        case = sy.random_box(64, 64, Nz, 2, 4, seed=Nz, dtype="f64")
        S = sy.random_source(case.chi.shape, seed=9)
        J, L = gpu_fs(case, S)
        Jo, Lo = orc.fs_box(case.chi[0], S[0], case.I_bc[0, 0], case.I_bc[0, 1], 2, 4)
        _check(J[0], L[0], Jo, Lo, "f64")
