"""The launch shape that a batch gets by its estimated time against shapes that used to be
the default for its layer: never much slower.  (Batches of a few hundred items had been
estimated as a single wavelength, and workgroups of nine waves as if four SIMDs shared
them evenly: up to 1.7 times slower.)"""
import time

import pytest

import synthetic as sy
from tests.gpu_helpers import make_grid, to_dev, torch_cuda

pytestmark = pytest.mark.gpu


def _ms(torch, g, chi, S):
    best = 1e9
    for _ in range(8):
        torch.cuda.synchronize()
        t0 = time.perf_counter()
        g.formal_solution(chi, S)
        torch.cuda.synchronize()
        best = min(best, time.perf_counter() - t0)
    return 1e3 * best


@pytest.mark.parametrize("nx,ny,nz,n_mu,n_phi,lam,fixed", [
    (63, 110, 15, 14, 13, 5, (1024, 8)), (130, 33, 22, 24, 42, 3, (768, 6)), (90, 50, 28, 24, 8, 6, (768, 6)),
    (34, 52, 114, 12, 37, 2, (1024, 2))])
def test_chosen_shape_is_not_much_slower(nx, ny, nz, n_mu, n_phi, lam, fixed):
    torch = torch_cuda()
    case = sy.random_box(nx, ny, nz, n_mu, n_phi, seed=nx, dtype="f32", n_lambda=lam)
    chi, S = to_dev(case.chi, "f32"), to_dev(sy.random_source(case.chi.shape, seed=1, dtype="f32"), "f32")
    g = make_grid(case)
    chosen, shape = _ms(torch, g, chi, S), g.launch_shape()
    g.set_launch_shape(*fixed, band=False)
    widest = _ms(torch, g, chi, S)
    g.close()
    print(nx, ny, nz, shape, "%.3f ms" % chosen, fixed, "%.3f ms" % widest, flush=True)
    assert chosen < 1.25 * widest
