"""The scheme does not depend on the units of density and pressure: a state with
jumps, scaled by an even power of two (the fields by its root), gives the same
bits after both stages.  The scales are those where the square of a jump's
difference leaves the range of the stored type, in the weight of the parabola's
discontinuity step, but nothing else does."""
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


def _state(shape, axis):
    """Jumps from 1 to 2 of density and pressure across the axis, in a shear flow with a field."""
    rng = np.random.default_rng(5 + axis)
    U = np.zeros((binding.NFIELDS,) + shape)
    n = shape[2 - axis]
    x = np.arange(n).reshape([n if d == 2 - axis else 1 for d in range(3)])
    step = np.broadcast_to(1.0 + ((x > n // 4) & (x <= 3 * n // 4)), shape)
    U[0] = step + 0.01 * rng.uniform(size=shape)
    U[1:4] = U[0] * (0.2 + 0.05 * rng.normal(size=(3,) + shape))
    e = 1.5 * (step + 0.01 * rng.uniform(size=shape))
    U[4], U[5] = e + 0.5 * (U[1:4] ** 2).sum(0) / U[0], e
    U[6:9] = np.array([0.1, 0.2, 0.3])[:, None, None, None]
    U[9] = 1e-3 * U[0]
    return U.astype(np.float32).astype(np.float64)


@pytest.mark.parametrize("axis", [0, 1, 2])
@pytest.mark.parametrize("stage", [binding.STAGE_NONADV, binding.STAGE_ADV])
@pytest.mark.parametrize("precision, power", [(binding.FP64, 510), (binding.FP32_MIXED, 62)])
def test_scaled_jumps(precision, power, stage, axis):
    shape = (12, 14, 16)
    U = _state(shape, axis)
    scale = np.ones((binding.NFIELDS, 1, 1, 1))
    scale[[0, 1, 2, 3, 4, 5, 9]] = 2.0 ** power
    scale[6:9] = 2.0 ** (power // 2)
    got = []
    for s in (1.0, scale):
        box = binding.Box(shape, precision=precision)
        box.set_state(U * s)
        box.debug_stage(stage, 0.01)
        got.append(box.get_state() / s)
    assert np.isfinite(got[0]).all() and np.abs(got[0] - U).max() > 1e-3
    np.testing.assert_array_equal(got[1], got[0])
