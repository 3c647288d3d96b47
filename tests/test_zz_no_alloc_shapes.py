"""rt_formal_solution_noalloc runs the launch shape of rt_formal_solution wherever its
partial sums fit the fixed array: the same bits.  Where they do not, the default shape
with fewer workgroups, in another order of summation."""
import numpy as np
import pytest

import synthetic as sy
from tests.gpu_helpers import make_grid
from tests.test_zz_no_alloc import _both, _check

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("want_lstar", [False, True])
@pytest.mark.parametrize("prec,band,n_lambda", [("f64", False, 1), ("f64", False, 3), ("f32", False, 2), ("f32", True, 1)])
def test_same_bits_where_the_shape_fits(prec, band, n_lambda, want_lstar):
    case = sy.random_box(24, 20, 10, 4, 8, seed=71, dtype=prec, n_lambda=n_lambda)
    g = make_grid(case, band_tiles=band)
    print(prec, band, n_lambda, want_lstar, g.launch_shape(), g.info()["n_workgroups"], flush=True)
    (J0, L0), (J1, L1) = _both(g, case, prec, n_lambda, want_lstar)
    g.close()
    assert np.array_equal(J0, J1)
    assert not want_lstar or np.array_equal(L0, L1)


def test_other_shape_where_it_does_not_fit():
    case = sy.random_box(46, 45, 40, 4, 8, seed=72, dtype="f64")
    g = make_grid(case)
    print(g.launch_shape(), g.info()["n_workgroups"], flush=True)
    for want_lstar in (False, True):
        _check(_both(g, case, "f64", 1, want_lstar), "f64")
    g.close()
