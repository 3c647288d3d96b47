"""The launch shape that a fresh grid reports, set again through either entry point,
reproduces its results bit for bit, band tiles on a grid whose layers would fit the
LDS whole among them; calls of other sizes and shares agree to the rounding of their
sums in double precision."""
import dataclasses

import numpy as np
import pytest

import synthetic as sy
from tests.gpu_helpers import gpu_fs, make_grid, to_dev, torch_cuda

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("named", [False, True])
@pytest.mark.parametrize("nx,prec", [(46, "f32"), (46, "f64"), (33, "f32")])
def test_reported_shape_set_again(nx, prec, named):
    case = sy.random_box(nx, 45, 5, 4, 8, seed=nx, dtype=prec)
    S = sy.random_source(case.chi.shape, seed=6, dtype=prec)
    g = make_grid(case)
    J0, _ = gpu_fs(case, S, grid=g, want_lstar=False)
    ls = g.launch_shape()
    print(nx, prec, ls, flush=True)
    if named:
        g.set_launch_shape(ls["threads"], ls["rays"], band=ls["band"])
    else:
        g.set_launch_shape(ls["threads"], ls["rays"])
    assert g.launch_shape() == ls
    J1, _ = gpu_fs(case, S, grid=g, want_lstar=False)
    g.close()
    assert np.array_equal(J0, J1)


# J is a sum of 32 directions' terms, all positive, in double: two orders of summation
# differ by at most 32 roundings of 1.1e-16 of the sum, 4e-15, and J is at most the
# largest source or boundary intensity here.
def test_shares_and_single_calls_agree_in_double():
    case = sy.random_box(46, 45, 5, 4, 8, seed=51, dtype="f64", n_lambda=9)
    S = sy.random_source(case.chi.shape, seed=3)
    g = make_grid(case)
    J, _ = gpu_fs(case, S, grid=g, want_lstar=False)
    tol = dict(rtol=4e-15, atol=1e-14 * np.abs(J).max())
    one = dataclasses.replace(case, chi=case.chi[4:5], eps=case.eps[4:5], B=case.B[4:5], I_bc=case.I_bc[4:5])
    np.testing.assert_allclose(gpu_fs(one, S[4:5], grid=g, want_lstar=False)[0][0], J[4], **tol)
    torch = torch_cuda()
    chi, St, Ib = (to_dev(x, "f64") for x in (case.chi, S, case.I_bc))
    total = sum(g.formal_solution_dirs(chi, St, g.shard_directions(2, k), Ib)[0] for k in range(2))
    torch.cuda.synchronize()
    np.testing.assert_allclose(total.cpu().numpy(), J, **tol)
    g.close()
