"""Cells that one chemistry update leaves without atomic hydrogen (all ionised,
all molecular, some with rho_H2 + rho_H+ a unit in the last place above rho):
the tail with heating and cooling against the oracle, and once more from there."""
import numpy as np
import pytest

import oracle
from paper_1608_08748_amd import binding

from test_gpu_parity import TOL64, assert_fields_close
from test_oracle_full_cells import CASES, full_state

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", autouse=True)
def _need_gpu():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("needs a GPU")
    torch.cuda.set_device(0)


@pytest.mark.parametrize("precision", [binding.FP64, binding.FP32_MIXED])
@pytest.mark.parametrize("network, cells, n_u, dt", CASES)
def test_full_cells(network, cells, n_u, dt, precision):
    shape, n = (5, 20, 20), 2000
    kw = dict(units=(n_u,) + tuple(binding.DEFAULT_UNITS[1:]), cooling=True, ionisation=network)
    P = oracle.make_params(shape, **kw)
    U = full_state(P, cells(n)).reshape((binding.NFIELDS,) + shape).copy()
    box = binding.Box(shape, precision=precision, **kw)
    box.set_state(U)
    box.debug_stage(binding.STAGE_TAIL, dt)
    G = box.get_state()
    if precision == binding.FP64:
        V = U.copy()
        oracle.clamp_h2(P, V)
        oracle.chemistry(P, V, dt)
        oracle.cooling(P, V, dt)
        oracle.regularise(P, V)
        assert_fields_close(G, V, TOL64, "full cells, network %s" % network)
    rest = G[0] - G[9] - G[10]
    assert np.abs(rest).max() <= (4e-16 if precision == binding.FP64 else 4e-7) * G[0].max()
    box.debug_stage(binding.STAGE_TAIL, dt)
    assert np.isfinite(box.get_state()).all()
