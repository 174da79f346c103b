"""mhd_get_state and the kinds of memory a caller may hand it: the copy to pinned
host memory and to device memory is the runtime's, whatever the size, and holds
the bits of the copy to pageable memory."""
import ctypes

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


@pytest.mark.parametrize("precision", [binding.FP64, binding.FP32_MIXED])
@pytest.mark.parametrize("shape", [(5, 6, 7), (61, 59, 67)])
def test_state_to_device_and_pinned_memory(shape, precision):
    import torch
    box = binding.Box(shape, precision=precision)
    box.init_state(inputs.white_noise(shape, seed=4, sigma=0.3, B=(0.2, -0.3, 0.1)))
    box.step_cfl()
    want = box.get_state()
    for dst in (torch.zeros(want.shape, dtype=torch.float64, device="cuda"),
                torch.zeros(want.shape, dtype=torch.float64).pin_memory()):
        torch.cuda.synchronize()
        st = binding.lib().mhd_get_state(box.h, ctypes.cast(dst.data_ptr(), ctypes.POINTER(ctypes.c_double)))
        assert st == binding.MHD_OK
        np.testing.assert_array_equal(dst.cpu().numpy(), want)
