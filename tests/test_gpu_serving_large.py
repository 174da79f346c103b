"""A served batch whose launches stream their outputs past the caches (fields of
more than 12 MB over all boxes) while each box alone does not: the bits of every
box alone, with one workgroup per tile and with a resident grid.  The kept
states grow from box to box, so the server's pinned slots are replaced by larger
ones on the way."""
import numpy as np
import pytest

from paper_1608_08748_amd import binding, inputs, serving

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", autouse=True)
def _need_gpu():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("needs a GPU")
    torch.cuda.set_device(0)


@pytest.mark.parametrize("precision, sides", [(binding.FP64, (48, 112)), (binding.FP32_MIXED, (48, 96, 130))])
def test_streamed_batch_equals_single_boxes(precision, sides):
    size = 8 if precision == binding.FP64 else 4
    assert sum(n ** 3 for n in sides) * size > 12e6 > max(sides) ** 3 * size
    states = [inputs.white_noise((n, n, n), seed=n, sigma=0.3, B=(0.2, -0.3, 0.1)) for n in sides]
    alone = []
    for W in states:
        box = binding.Box(W.shape[1:], precision=precision)
        box.init_state(W)
        for _ in range(3):
            box.step_cfl()
        alone.append((box.get_state(), box.totals()))
        box.close()
    p = binding.server_params(precision=precision)
    room = sum(binding.server_box_bytes(p, W.shape[1:]) for W in states)
    for persistent in (False, True):
        print("streamed batch", precision, persistent, flush=True)
        sv = binding.Server(room, max_slots=8, precision=precision, persistent=persistent)
        out = serving.run(sv, states, 3, keep_state=True)
        assert out["max_active"] == len(sides) and out["statuses"] == [0]
        for (U, tot), r in zip(alone, out["records"]):
            np.testing.assert_array_equal(sv.result(r["id"]), U)
            np.testing.assert_array_equal(r["totals"], tot)
        sv.close()
