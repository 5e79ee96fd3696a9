"""What a workgroup of the batched pass finds in LDS before it has staged anything there must not reach an output."""
import numpy as np
import pytest

from paper_1102_0183_amd import binding
from tests.parity_helpers import to_dev

pytestmark = pytest.mark.gpu


def _run(net, imgs):
    import torch
    n = len(imgs)
    probs = torch.full((n * net.num_classes,), -1.0, dtype=torch.float32, device="cuda:0")
    scratch = torch.empty(net.forward_batch_scratch_bytes(n), dtype=torch.uint8, device="cuda:0")
    net.forward_batch(to_dev(imgs), n, probs, scratch, n)
    net.synchronize()
    return probs.cpu().numpy().reshape(n, -1)


@pytest.mark.parametrize("inputs", [150, 130, 33])
def test_ragged_chunk_behind_images_of_no_numbers(inputs):
    """A fully connected layer whose last chunk of inputs is no multiple of what the matrix instructions take, behind a pass
    that staged images of NaN in every compute unit's LDS."""
    rng = np.random.default_rng(1)
    bad = binding.Cnn("1x30x30-300N-10N")
    bad.set_weights(rng.uniform(-0.05, 0.05, bad.num_weights).astype(np.float32))
    good = binding.Cnn("1x%dx1-40N-10N" % inputs)
    good.set_weights(rng.uniform(-0.05, 0.05, good.num_weights).astype(np.float32))
    imgs = rng.uniform(-1, 1, (2000, inputs)).astype(np.float32)
    want = _run(good, imgs)
    assert np.all(np.isnan(_run(bad, np.full((20000, 900), np.nan, dtype=np.float32))))
    got = _run(good, imgs)
    assert np.isfinite(want).all() and np.array_equal(want, got)
    bad.close()
    good.close()
