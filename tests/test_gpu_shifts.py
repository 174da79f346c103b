"""A periodic box shifted by whole cells gives the shifted result, bit for bit:
no cell depends on where the tiles, segments, row pieces and loop trips of the
launches end.  Both precisions, with and without the ionisation network (each
has march code of its own: window lengths, faces per trip, field groups), over
rows in whole blocks, in pieces and with both sides of the FP32 choice between
them (367: pieces, 500: whole rows)."""
import numpy as np
import pytest

from paper_1608_08748_amd import binding, inputs

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", autouse=True)
def _need_gpu():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("needs a GPU")
    torch.cuda.set_device(0)


# (nz, ny, nx)
SHAPES = [(1, 1, 9), (2, 3, 5), (1, 33, 64), (33, 1, 63), (31, 65, 17), (65, 32, 33), (97, 5, 130), (7, 67, 65),
          (3, 40, 257), (4, 5, 367), (5, 4, 500), (2, 3, 1031), (72, 70, 100)]


@pytest.mark.parametrize("precision", [binding.FP64, binding.FP32_MIXED])
@pytest.mark.parametrize("network", [False, True])
@pytest.mark.parametrize("shape", SHAPES)
def test_shifted_box(shape, network, precision):
    print("shift", shape, network, precision, flush=True)
    W = inputs.white_noise(shape, seed=sum(shape), sigma=0.3, B=(0.2, -0.3, 0.1))
    W = np.concatenate([W, np.zeros((binding.NPRIM - W.shape[0],) + shape)])
    W[8] = 0.01
    W[9] = 0.02 if network else 0.0
    by = tuple(max(1, int(0.4 * n)) for n in shape)
    out = []
    for shift in ((0, 0, 0), by):
        box = binding.Box(shape, precision=precision, ionisation=network)
        box.init_state(np.roll(W, shift, axis=(1, 2, 3)))
        dts = []
        for _ in range(3):
            dts.append(box.cfl_dt())
            box.step_cfl()
        out.append((dts, np.roll(box.get_state(), tuple(-s for s in shift), axis=(1, 2, 3))))
    assert out[0][0] == out[1][0]
    np.testing.assert_array_equal(out[1][1], out[0][1])
