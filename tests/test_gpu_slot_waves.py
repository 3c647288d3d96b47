"""Partial slots of batches: one, four or sixteen wavefronts a voxel by the batch's voxels,
with the order of summation kept by the grid's, so that every wavelength of a batch comes
out as it does alone, bit for bit, wherever both run the same launch shape.  Grids of the
sixteen-run and the four-run order (below and from 65536 voxels), batches below and from
65536 and 262144 voxels in all; every direction has a slot of its own."""
import pytest

import synthetic as sy
from tests.gpu_helpers import make_grid, to_dev, torch_cuda

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("prec", ["f64", "f32"])
@pytest.mark.parametrize("dims,lam", [((9, 8, 7), 3), ((32, 32, 20), 4), ((32, 32, 20), 14), ((64, 64, 17), 5),
                                      ((33, 33, 31), 9)])
def test_batch_sums_as_its_wavelengths(dims, lam, prec):
    torch = torch_cuda()
    case = sy.random_box(*dims, 2, 3, seed=dims[0], dtype=prec, n_lambda=lam)
    S = to_dev(sy.random_source(case.chi.shape, seed=3, dtype=prec), prec)
    chi, bc = to_dev(case.chi, prec), to_dev(case.I_bc, prec)
    single = make_grid(case, n_lambda_max=1)
    assert lam * 6 <= single.info()["n_workgroups"] // single.launch_shape()["bundles"]
    single.close()
    g = make_grid(case)
    print(dims, lam, prec, g.launch_shape(), flush=True)
    J, L = g.formal_solution(chi, S, bc, want_lstar=True)
    for l in range(lam):
        one = [x[l:l + 1].contiguous() for x in (chi, S, bc)]
        Jl, Ll = g.formal_solution(*one, want_lstar=True)
        assert torch.equal(Jl[0], J[l]) and torch.equal(Ll[0], L[l])
        # J alone may run another shape than J and Lambda* together
        Ja = g.formal_solution(*one)[0]
        assert torch.equal(Ja[0], g.formal_solution(chi, S, bc)[0][l])
    # one step of the batch against one-wavelength steps
    eps, B = to_dev(case.eps, prec), to_dev(case.B, prec)
    opts = g.opts(tol=1e-30, max_iter=1, ng_every=0)
    st = g.new_state(chi, eps, B, bc)
    for _ in range(2):
        g.ali_step(st, opts)
    whole = g.state_tensors(st)["J"].clone()
    for l in {0, lam - 1}:
        part = g.new_state(*[x[l:l + 1].contiguous() for x in (chi, eps, B, bc)])
        for _ in range(2):
            g.ali_step(part, opts)
        assert torch.equal(g.state_tensors(part)["J"][0], whole[l])
    g.close()
