"""Small calls in resident mode: a wait that gave up in one of several calls in a row is not forgotten; forward calls of a few
images, which run as launches of their stages, between training calls, which do not."""
import numpy as np
import pytest

from paper_1102_0183_amd import binding, synth
from tests.parity_helpers import build_pair, compare_forward_state, to_dev

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("name", ["cfg1", "cfg3"])
def test_a_wait_that_gave_up_is_reported_after_later_calls(name):
    wl = synth.WORKLOADS[name]
    print("case", name, flush=True)
    imgs, labs = synth.images(wl, 3), synth.labels(wl, 3)
    d_imgs, d_labs = to_dev(imgs), to_dev(labs)
    g, _ = build_pair(wl)
    g.set_mode(binding.MODE_RESIDENT)
    w0 = g.get_weights()
    g.train_many(d_imgs, d_labs, 0.001)
    g.synchronize()
    want = g.get_weights()
    g.set_spin_limit(0)       # some wait of this call always gives up
    g.train_many(d_imgs, d_labs, 0.001)
    g.set_spin_limit(1 << 22)
    g.train_many(d_imgs, d_labs, 0.001)   # (on undefined weights: what counts is that it ends, and what the next line says)
    with pytest.raises(binding.CnnError) as e:
        g.synchronize()
    assert e.value.code == binding.E_HIP
    g.synchronize()           # (told once)
    g.set_weights(w0)
    for t in range(3):        # one image a call, nothing asked for in between
        g.train_step(d_imgs[t].contiguous().view(-1), int(labs[t]), 0.001)
    np.testing.assert_array_equal(g.get_weights(), want)
    g.close()


@pytest.mark.parametrize("arch", ["1x29x29-20C4-MP2-40C5-MP3-150N-10N", "3x32x32-70C5-MP2-66C5-MP2-64C4-MP2-30N-10N",
                                  "1x12x12-6C3-MP2-9C2-7N-4N"])
def test_forward_calls_of_any_size_between_training_calls(arch):
    """One image to five a call (on both sides of where the launches of stages stop): outputs and parity taps of the last
    image are the oracle's, on the weights the training calls before have left."""
    import torch
    print("case", arch, flush=True)
    g, o = build_pair(arch=arch, seed=5)
    g.set_mode(binding.MODE_RESIDENT)
    info = o.layer_info(0)
    rng = np.random.default_rng(6)
    imgs = (rng.random((5, info["maps"], info["h"], info["w"]), dtype=np.float32) * 2 - 1).astype(np.float32)
    d_imgs = to_dev(imgs)
    for n in range(1, 6):
        g.train_step(d_imgs[n - 1].contiguous().view(-1), n % g.num_classes, 0.01)
        o.train_step(imgs[n - 1], n % g.num_classes, 0.01)
        probs = torch.empty(n * g.num_classes, dtype=torch.float32, device="cuda:0")
        g.forward_many(d_imgs, n, probs)
        g.synchronize()
        want = o.forward_many(imgs[:n], n)
        # (the weights after up to five steps agree to 1e-5 of their largest, activations and outputs to the usual bar)
        assert np.abs(probs.cpu().numpy().reshape(n, -1) - want).max() <= 1e-5, n
        o.forward(imgs[n - 1])
        compare_forward_state(g, o)
    g.close()
