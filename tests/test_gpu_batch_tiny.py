"""Activations far below those that two halves hold to 23 bits, in the batched pass's products of halves: every tile that writes or
reads them, against the oracle (64 bits), to the parity bar of the image's own layer."""
import numpy as np
import pytest

from paper_1102_0183_amd import binding
from tests.parity_helpers import build_pair, to_dev
from tests.test_gpu_batch import _scratch, _trainable
from tests.test_gpu_batch_halves import FIRST, TILES
from tests.test_gpu_batch_tail import TILES as HIDDEN

pytestmark = pytest.mark.gpu


def _parameters(net, w):
    """Views of each trainable layer's biases and connections in the canonical weights."""
    out, at = [], 0
    for l in range(1, net.num_layers):
        a = net.layer_info(l)
        if a["kind"] == 2:
            continue
        below = net.layer_info(l - 1)
        n = a["maps"] * below["maps"] * (a["K"] ** 2 if a["kind"] == 1 else below["h"] * below["w"])
        out.append((w[at:at + a["maps"]], w[at + a["maps"]:at + a["maps"] + n]))
        at += a["maps"] + n
    assert at == len(w)
    return out


def _no_biases(g, o, scales=()):
    w = g.get_weights()
    for k, (bias, connections) in enumerate(_parameters(g, w)):
        bias[:] = 0
        if k < len(scales):
            connections *= np.float32(scales[k])
    g.set_weights(w)
    o.set_weights(w.astype(np.float64))


def _check(g, o, imgs, batch, layers, sample):
    scratch = _scratch(g, batch)
    d = to_dev(imgs)
    got = [g.debug_forward_batch_layer(d, batch, k, scratch).astype(np.float64) for k in range(layers)]
    for i in sample:
        o.forward(imgs[i])
        for k in range(layers):
            l = _trainable(o)[k]
            pooled = l + 1 < o.num_layers and o.layer_info(l + 1)["kind"] == 2
            want = np.asarray(o.activation(l + 1 if pooled else l), dtype=np.float64).ravel()
            assert np.abs(want).max() > 0
            assert np.abs(got[k][i] - want).max() <= 1e-5 * np.abs(want).max(), (i, k, np.abs(want).max())


CASES = sorted({(t[0], t[1], 2) for t in TILES} | {(t[0], t[1], 2) for t in FIRST} | {(t[0], t[1], 3) for t in HIDDEN})


@pytest.mark.parametrize("arch,batch,layers", CASES)
def test_tiny_images_beside_others(arch, batch, layers):
    """No biases, and some images a millionth to a 10^-20th of the others: each to the bar of its own activations."""
    print("case", arch, batch, flush=True)
    assert binding.batch_plan(arch, batch)[0][layers - 1]["split"]
    g, o = build_pair(arch=arch, wscale=0.1)
    _no_biases(g, o)
    imgs = (np.random.default_rng(31).random((batch, g.image_size)) * 2 - 1).astype(np.float32)
    scales = {1: 1e-6, 2: 1e-8, batch // 2: 1e-12, batch - 1: 1e-20}
    for i, s in scales.items():
        imgs[i] *= np.float32(s)
    _check(g, o, imgs, batch, layers, sorted(set(scales) | {0, 3}))
    g.close()


@pytest.mark.parametrize("scale", [1e-4, 1e-6, 1e-8, 1e-12, 1e-20, 1e-30])
@pytest.mark.parametrize("layer", [0, 1, 2])
def test_a_layer_of_small_weights_below_one_of_large_ones(layer, scale):
    """The layer's activations shrink by `scale`, the next one's weights bring them back up."""
    arch, batch = "3x40x40-33C3-MP2-40C3-MP1-48C4-MP2-64N-33N-4N", 130
    plan = binding.batch_plan(arch, batch)[0]
    assert [p["first"] or p["split"] for p in plan[:4]] == [1, 1, 1, 1]
    g, o = build_pair(arch=arch, wscale=0.1)
    scales = [1.0] * 4
    scales[layer] *= scale
    scales[layer + 1] /= scale
    _no_biases(g, o, scales)
    imgs = (np.random.default_rng(32).random((batch, g.image_size)) * 2 - 1).astype(np.float32)
    _check(g, o, imgs, batch, 4, [0, 64, batch - 1])
    g.close()


@pytest.mark.parametrize("arch,batch,T,share", [("3x16x16-37C3-MP1-33C3-MP2-4N", 33, 1, 0), ("4x14x14-70C5-MP2-33C2-MP2-4N", 7, 1, 1),
                                                ("1x15x15-197C2-MP1-80C3-MP2-4N", 130, 2, 0), ("3x17x17-200C5-MP1-48C4-MP2-4N", 300, 2, 0),
                                                ("1x28x28-69C5-MP2-33C1-MP2-4N", 130, 2, 1), ("4x15x15-326C2-MP2-80C4-MP1-4N", 300, 5, 0)])
def test_groups_of_maps_that_begin_eight_earlier(arch, batch, T, share):
    """The first layer's workgroups where the last one takes eight maps from the one in front of it, some images tiny."""
    print("case", arch, batch, flush=True)
    p = binding.batch_plan(arch, batch)[0]
    assert p[1]["split"] and (p[0]["first_T"], p[0]["first_share"], p[0]["first_shift"]) == (T, share, 8), p[0]
    g, o = build_pair(arch=arch, wscale=0.1)
    _no_biases(g, o)
    imgs = (np.random.default_rng(33).random((batch, g.image_size)) * 2 - 1).astype(np.float32)
    imgs[1] *= np.float32(1e-6)
    imgs[2] *= np.float32(1e-12)
    _check(g, o, imgs, batch, 2, [0, 1, 2, 3, batch - 1])
    g.close()
