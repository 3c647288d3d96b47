"""Solves whose wavelengths converge at different steps: every step has a batch of
its own, and one grid goes through more of them than it keeps schedules for (64).
Each wavelength must come out as it does alone on a fresh grid."""
import dataclasses

import numpy as np
import pytest

import synthetic as sy
from tests.gpu_helpers import gpu_solve, make_grid, to_dev, torch_cuda

pytestmark = pytest.mark.gpu


# Two solves to a relative change of tol differ by about 2 tol / (1 - rho) of the
# iteration's contraction rho, at most 0.98 here: a hundred times tol, and ten in hand.
@pytest.mark.parametrize("prec,tol,rtol", [("f64", 1e-9, 1e-6), ("f32", 1e-8, 1e-5)])
def test_shrinking_batches_match_single_solves(prec, tol, rtol):
    torch = torch_cuda()
    n = 24
    case = sy.random_box(11, 9, 7, 4, 4, seed=3, dtype=prec, n_lambda=n)
    eps = np.logspace(0.0, -3.0, n)[:, None, None, None] * np.ones_like(case.eps)
    case = dataclasses.replace(case, eps=eps.astype(np.float32).astype(np.float64))
    pick = lambda c, idx: dataclasses.replace(c, chi=c.chi[idx], eps=c.eps[idx], B=c.B[idx], I_bc=c.I_bc[idx])
    alone, steps = [], []
    for l in range(n):
        r = gpu_solve(pick(case, [l]), tol=tol, max_iter=400)
        assert r["status"] == 0
        alone.append(r["J"][0])
        steps.append(r["report"].iters)
    alone = np.stack(alone)
    turns = 8
    print(prec, "steps of single solves:", steps, flush=True)
    assert turns * len(set(steps)) > 64
    g = make_grid(case)
    rng = np.random.default_rng(1)
    for turn in range(turns):
        idx = rng.permutation(n)
        c = pick(case, idx)
        st = g.new_state(to_dev(c.chi, prec), to_dev(c.eps, prec), to_dev(c.B, prec), to_dev(c.I_bc, prec))
        stream = torch.cuda.Stream()
        stream.wait_stream(torch.cuda.current_stream())
        with torch.cuda.stream(stream):
            status, rep = g.solve(st, g.opts(tol=tol, max_iter=400, ng_every=4, ng_start=4, use_graph=bool(turn % 2)),
                                  stream=stream)
        torch.cuda.synchronize()
        assert status == 0
        J = g.state_tensors(st)["J"].cpu().numpy()
        np.testing.assert_allclose(J, alone[idx], rtol=rtol, err_msg=f"turn {turn}")
    g.close()
