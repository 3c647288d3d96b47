"""The tiled convolutions of the correction network at the edges of their tiles: rows
of one block and just more (44, 33 and 22 voxels for 16, 32 and 64 input channels; with stride 2
22, 11 and 11),
layers and rows that fill a tile or leave one over, volumes smaller than a tile, every
pair of channel numbers.  Reference and tolerance as for the other forward tests."""
import numpy as np
import pytest

import synthetic as sy
from paper_2102_01734_amd import precond
from tests.gpu_helpers import make_grid, torch_cuda
from tests.test_gpu_precond import reference_forward

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("shape,C", [((44, 4, 4), (16,)), ((45, 5, 3), (16, 16)), ((2, 2, 1), (16, 32)),
                                     ((89, 3, 5), (16, 64)), ((33, 4, 4), (32, 32)), ((67, 9, 5), (32, 64)),
                                     ((34, 5, 9), (32, 16)), ((22, 4, 2), (64, 16)), ((45, 5, 3), (64, 32)),
                                     ((3, 17, 6), (64, 64)), ((130, 6, 7), (16, 32, 16)),
                                     ((88, 8, 4), (16, 32)), ((45, 17, 5), (32, 64)), ((46, 9, 9), (64, 32)),
                                     ((23, 5, 3), (64, 64, 64)), ((1, 1, 2), (32, 64, 16))])
def test_forward_at_tile_edges(shape, C):
    torch = torch_cuda()
    Nx, Ny, Nz = shape
    print(f"net forward {shape} {C}", flush=True)
    g = make_grid(sy.random_box(Nx, Ny, Nz, 2, 4, seed=3, dtype="f32"))
    blob = precond.random_blob(C, seed=Nx)
    g.set_preconditioner(blob)
    f = np.random.default_rng(Nx).uniform(-1, 1, size=(Nz, Ny, Nx, 3)).astype(np.float32)
    out = g.precond_forward(torch.tensor(f, device="cuda"))
    torch.cuda.synchronize()
    ref = reference_forward(blob, f)
    np.testing.assert_allclose(out.cpu().numpy(), ref, rtol=2e-2, atol=2e-2 * np.abs(ref).max())
    g.close()
