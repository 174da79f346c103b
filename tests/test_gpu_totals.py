"""The totals' reduction at the edges of its chunks (4096 cells, 512 chunks):
every field against the exact sum.  Each value passes through fewer than 64
additions (16 in a running sum, then trees over the thread's sums, the wave, the
block and the chunks), so the error is below 64 rounding units of the sum of the
magnitudes."""
import math

import numpy as np
import pytest

from paper_1608_08748_amd import binding

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", autouse=True)
def _need_gpu():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("needs a GPU")
    torch.cuda.set_device(0)


@pytest.mark.parametrize("precision", [binding.FP64, binding.FP32_MIXED])
@pytest.mark.parametrize("shape", [(1, 1, 1), (1, 5, 51), (1, 64, 64), (17, 1, 241), (3, 64, 65), (128, 128, 128),
                                   (1, 3, 699051)])
def test_totals_at_chunk_edges(shape, precision):
    import torch
    rng = np.random.default_rng(sum(shape))
    n = int(np.prod(shape))
    U = rng.normal(size=(binding.NFIELDS, n)) * 10.0 ** rng.uniform(-6, 6, size=(binding.NFIELDS, 1))
    dt = torch.float64 if precision == binding.FP64 else torch.float32
    dev = torch.from_numpy(U).to(device="cuda", dtype=dt).reshape((binding.NFIELDS,) + shape).contiguous()
    stored = dev.cpu().double().numpy().reshape(binding.NFIELDS, n)
    out = torch.full((binding.NFIELDS,), float("nan"), dtype=torch.float64, device="cuda")
    print("totals", shape, precision, flush=True)
    assert binding.conserved_totals_noalloc(dev, precision, out) == binding.MHD_OK
    got = out.cpu().numpy()
    for f in range(binding.NFIELDS):
        assert abs(got[f] - math.fsum(stored[f])) <= 64 * 2.0 ** -53 * math.fsum(np.abs(stored[f])), f
