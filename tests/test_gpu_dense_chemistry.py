"""H2 formation at densities whose product has no FP64 value (an infinite rate):
the update ends at its clamp, all hydrogen molecular, as the oracle's does."""
import numpy as np
import pytest

import oracle
from paper_1608_08748_amd import binding

from test_gpu_parity import TOL64, assert_fields_close
from test_oracle_full_cells import full_state, molecular

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", autouse=True)
def _need_gpu():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("needs a GPU")
    torch.cuda.set_device(0)


@pytest.mark.parametrize("network", [False, True])
def test_infinite_formation_rate(network):
    shape, n = (4, 8, 8), 256
    kw = dict(units=(1e160,) + tuple(binding.DEFAULT_UNITS[1:]), ionisation=network)
    P = oracle.make_params(shape, **kw)
    U = full_state(P, molecular(n)).reshape((binding.NFIELDS,) + shape).copy()
    V = U.copy()
    oracle.clamp_h2(P, V)
    oracle.chemistry(P, V, 1e-3)
    oracle.regularise(P, V)
    assert np.isfinite(V).all() and np.allclose(V[9], V[0], rtol=1e-15)
    box = binding.Box(shape, **kw)
    box.set_state(U)
    box.debug_stage(binding.STAGE_TAIL, 1e-3)
    assert_fields_close(box.get_state(), V, TOL64, "infinite rate, network %s" % network)
