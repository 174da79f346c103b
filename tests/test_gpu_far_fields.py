"""A box whose fields pass 4 GiB, where the kernels take 64-bit offsets: eight
copies of a small box along z give eight copies of its result, bit for bit.
Needs 233 GB of device memory and about 60 GB of host memory."""
import gc
import os

import numpy as np
import pytest

from paper_1608_08748_amd import binding, inputs

pytestmark = pytest.mark.gpu

COPIES, SMALL = 8, (257, 512, 512)


def test_copies_of_a_small_box():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("needs a GPU")
    torch.cuda.set_device(0)
    shape = (COPIES * SMALL[0],) + SMALL[1:]
    assert np.prod(shape) * 8 > 1 << 32
    gc.collect()
    torch.cuda.empty_cache()
    host = os.sysconf("SC_AVPHYS_PAGES") * os.sysconf("SC_PAGE_SIZE")
    if torch.cuda.mem_get_info()[0] < 240e9 or host < 100e9:
        pytest.skip("needs 240 GB of device memory and 100 GB of host memory")
    W = inputs.white_noise(SMALL, seed=3, sigma=0.3, B=(0.2, -0.3, 0.1))
    W[0] += 0.1 * np.sin(np.arange(SMALL[2]) * 0.05)[None, None, :]
    small = binding.Box(SMALL)
    small.init_state(W)
    dts = []
    for _ in range(2):
        dts.append(small.cfl_dt())
        small.step_cfl()
    want = small.get_state()
    small.close()
    del small
    torch.cuda.empty_cache()
    V = np.empty((W.shape[0],) + shape)
    for r in range(COPIES):
        V[:, r * SMALL[0]:(r + 1) * SMALL[0]] = W
    print("far fields: state of", V.nbytes, flush=True)
    box = binding.Box(shape)
    box.init_state(V)
    del V
    for dt in dts:
        assert box.cfl_dt() == dt
        box.step_cfl()
    got = box.get_state()
    box.close()
    del box
    torch.cuda.empty_cache()
    for f in range(binding.NFIELDS):
        for r in range(COPIES):
            assert np.array_equal(got[f, r * SMALL[0]:(r + 1) * SMALL[0]], want[f]), (binding.FIELDS[f], r)
