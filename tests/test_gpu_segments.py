"""Boxes at the edges of the launch tilings: sides around the segment lengths
and wavefronts of the marching kernels, sides of one to three cells, and rows
around the block widths and in pieces.  FP64 against the oracle at the bound of
tolerance.py, after two steps at the oracle's CFL step."""
import pytest

import oracle
from paper_1608_08748_amd import binding, inputs

from test_gpu_parity import TOL64, assert_fields_close

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", autouse=True)
def _need_gpu():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("needs a GPU")
    torch.cuda.set_device(0)


# (nz, ny, nx)
SHAPES = [(1, 1, 200), (2, 3, 5), (1, 33, 64), (33, 1, 63), (31, 65, 17), (65, 32, 33), (97, 5, 130), (7, 67, 65),
          (3, 40, 257),
          # rows in pieces with halos: two and more per row, even and ragged,
          # several pieces and parts of rows in a block
          (2, 3, 252), (3, 2, 301), (2, 5, 515), (5, 1, 767), (2, 2, 1031)]


@pytest.mark.parametrize("shape", SHAPES)
def test_tiling_edges(shape):
    print("segments", shape, flush=True)
    W = inputs.white_noise(shape, seed=sum(shape), sigma=0.3, B=(0.2, -0.3, 0.1))
    box = binding.Box(shape)
    box.init_state(W)
    P = oracle.make_params(shape)
    U = oracle.prim_to_cons(P, W)
    for _ in range(2):
        dt = oracle.cfl_dt(P, U)
        box.step(dt)
        oracle.step(P, U, dt)
    assert_fields_close(box.get_state(), U, TOL64, "tiling %s" % (shape,))
