"""The fully connected layers of a batch: products of halves at the edges of their tiles, chunks and slices, and the last two
layers in one launch over hidden neurons, outputs and images, against the oracle."""
import numpy as np
import pytest

from paper_1102_0183_amd import binding
from tests.parity_helpers import build_pair, to_dev
from tests.test_gpu_batch import _check_layers, _scratch

pytestmark = pytest.mark.gpu

# (arch, batch, tiles of the first hidden layer: RT, CT, TR, its k range in slices)
TILES = [
    ("2x10x10-50C3-MP2-17C3-MP2-150N-10N", 7, 1, 1, 32, False),
    ("1x12x12-50C3-MP2-80C3-MP1-20N-4N", 7, 1, 1, 32, True),
    ("1x10x10-20C3-MP2-112C3-MP2-16N-4N", 7, 1, 2, 16, False),
    ("2x17x17-8C3-MP1-100C4-MP4-16N-4N", 7, 1, 2, 16, True),
    ("1x20x20-33C3-MP2-80C3-MP1-500N-5N", 130, 1, 2, 32, True),
    ("2x24x24-8C3-MP2-17C3-MP3-300N-5N", 2000, 1, 4, 16, False),
    ("1x17x17-20C3-MP1-48C3-MP1-112N-9N", 130, 1, 4, 16, True),
    ("1x12x12-33C3-MP2-17C4-MP2-100N-64N-10N", 33, 2, 1, 32, False),
    ("1x14x14-33C3-MP1-40C3-MP2-100N-64N-10N", 7, 2, 1, 32, True),
    ("1x29x29-50C3-MP1-17C3-MP1-500N-5N", 2000, 2, 2, 32, True),
    ("2x12x12-33C3-MP2-40C3-MP3-33N-10N", 7, 3, 2, 16, False),
    ("2x16x16-8C3-MP2-100C4-MP2-33N-10N", 33, 3, 2, 16, True),
    ("1x17x17-50C3-MP1-112C2-MP1-33N-10N", 2000, 3, 4, 16, True),
    ("1x10x10-50C3-MP2-80C2-MP3-65N-33N-3N", 130, 5, 2, 16, False),
    ("2x16x16-33C3-MP2-112C2-MP3-65N-33N-3N", 7, 5, 2, 16, True),
    ("2x12x12-50C3-MP1-112C4-MP1-112N-9N", 300, 7, 2, 16, True),
]


def _outputs(g, d_imgs, n, batch):
    import torch
    probs = torch.full((n * g.num_classes,), -1.0, dtype=torch.float32, device="cuda:0")
    g.forward_batch(d_imgs, n, probs, _scratch(g, batch), batch)
    g.synchronize()
    return probs.cpu().numpy().reshape(n, -1)


@pytest.mark.parametrize("arch,batch,RT,CT,TR,slices", TILES)
def test_every_tile_of_a_hidden_layer(arch, batch, RT, CT, TR, slices):
    """The hidden layers of a batch, as planned, against the oracle, the outputs with a ragged second batch against the one-image
    path."""
    import torch
    print("case", arch, batch, flush=True)
    layers, whole = binding.batch_plan(arch, batch)
    h = layers[2]
    assert h["split_fc"] and (h["split_RT"], h["split_CT"], h["split_TR"], h["split_slices"] > 1) == (RT, CT, TR, slices), h
    assert whole["tail"]
    n = batch + batch // 2 + 1
    g, o = build_pair(arch=arch, wscale=0.03)
    imgs = (np.random.default_rng(8).random((n, g.image_size)) * 2 - 1).astype(np.float32)
    d_imgs = to_dev(imgs)
    _check_layers(g, o, d_imgs, imgs, batch, sorted({0, 1, batch // 2, batch - 1}), list(range(2, len(layers) - 1)))
    one = torch.empty(n * g.num_classes, dtype=torch.float32, device="cuda:0")
    g.forward_many(d_imgs, n, one)
    g.synchronize()
    assert np.abs(_outputs(g, d_imgs, n, batch) - one.cpu().numpy().reshape(n, -1)).max() <= 1e-5
    g.close()


@pytest.mark.parametrize("hidden,classes,batch", [
    (1, 2, 1), (63, 8, 3), (64, 9, 5), (65, 7, 4), (128, 16, 33), (129, 17, 33), (192, 64, 9), (193, 33, 9), (320, 38, 5), (321, 32, 5),
    (512, 24, 130), (513, 5, 130), (1024, 12, 9), (1000, 2, 300), (100, 10, 4099)])
@pytest.mark.parametrize("units", [binding.OUTPUT_SOFTMAX_XENT, binding.OUTPUT_TANH_SQERR])
def test_the_last_two_layers_in_one_launch(hidden, classes, batch, units):
    arch = "1x9x9-4C2-MP2-%dN-%dN" % (hidden, classes)
    print("case", arch, batch, units, flush=True)
    assert binding.batch_plan(arch, batch)[1]["tail"]
    g, o = build_pair(arch=arch, wscale=0.2)
    g.set_output_units(units)
    o.set_output_units(int(units == binding.OUTPUT_TANH_SQERR))
    imgs = (np.random.default_rng(9).random((batch, g.image_size)) * 2 - 1).astype(np.float32)
    got = _outputs(g, to_dev(imgs), batch, batch).astype(np.float64)
    for i in sorted({0, batch // 2, batch - 1}):
        want = np.asarray(o.forward(imgs[i]), dtype=np.float64).ravel()
        assert np.abs(got[i] - want).max() <= 1e-5 * max(np.abs(want).max(), 1.0), i
    g.close()


@pytest.mark.parametrize("value", [np.inf, -np.inf, np.nan, 1e30, 1e-30, 0.0])
def test_weights_of_hidden_layers_that_do_not_split(value):
    """One weight, and a whole row, of each of two hidden layers in products of halves: the layers' outputs as 64-bit sums of the
    layer's inputs have them (where the 32-bit product has its k range in planes, a sum that is no number counts as -inf)."""
    arch, n, pix, maps, h1, h2 = "1x10x10-50C3-MP2-80C2-MP3-65N-33N-3N", 130, 1, 80, 65, 33
    layers = binding.batch_plan(arch, n)[0]
    assert layers[2]["split_fc"] and layers[3]["split_fc"]
    g = binding.Cnn(arch)
    w = ((np.random.default_rng(4).random(g.num_weights) - 0.5) * 0.2).astype(np.float32)
    at = 50 + 50 * 9 + 80 + 80 * 50 * 4
    b1, w1 = w[at:at + h1], w[at + h1:at + h1 + h1 * maps * pix].reshape(h1, maps * pix)
    at += h1 + h1 * maps * pix
    b2, w2 = w[at:at + h2], w[at + h2:at + h2 + h2 * h1].reshape(h2, h1)
    for m in (w1, w2):
        m[3, 7] = value
        m[len(m) - 1, m.shape[1] - 1] = value
        if not np.isinf(value):
            m[9] = value
    g.set_weights(w)
    d = to_dev((np.random.default_rng(14).random((n, g.image_size)) * 2 - 1).astype(np.float32))
    scratch = _scratch(g, n)
    x = [g.debug_forward_batch_layer(d, n, k, scratch).reshape(n, -1).astype(np.float64) for k in (1, 2, 3)]
    for l, m, b in ((1, w1, b1), (2, w2, b2)):
        with np.errstate(all="ignore"):
            y = x[l - 1] @ m.astype(np.float64).T
            if layers[l + 1]["gemm_KS"] > 1:
                y = np.where(np.isnan(y), -np.inf, y)
            y = 1.7159 * np.tanh(0.6666 * (y + b))
        assert np.array_equal(np.isnan(x[l]), np.isnan(y)), l
        if np.isnan(y).all():
            continue
        assert np.nanmax(np.abs(x[l] - y)) <= 1e-5 * 1.7159, l
    g.close()


def test_a_handle_plans_again_when_its_batch_table_or_filters_change():
    """A handle keeps the plan of its last batched call: after every change its outputs are those of a handle that never had
    another one."""
    from paper_1102_0183_amd import synth
    arch, table = "2x20x20-17C3-MP2-40C4-MP2-33N-4N", synth.random_table(40, 17, 5, 7)
    filters = (np.random.default_rng(1).random((2, 5, 5)) - 0.5).astype(np.float32)

    def run(g, batch, n=40):
        w = ((np.random.default_rng(5).random(g.num_weights) - 0.5) * 0.2).astype(np.float32)
        g.set_weights(w)
        imgs = (np.random.default_rng(6).random((n, g.image_size)) * 2 - 1).astype(np.float32)
        return _outputs(g, to_dev(imgs), n, batch)

    steps = [("batch", 33), ("batch", 7), ("batch", 33), ("table", 33), ("units", 33), ("front", 33), ("batch", 1)]
    kept = binding.Cnn(arch)
    done = set()
    for what, batch in steps:
        done.add(what)
        fresh = binding.Cnn(arch)
        for g in (kept, fresh):
            if "table" in done and (g is fresh or what == "table"):
                g.set_connection_table(1, table)
            if "units" in done and (g is fresh or what == "units"):
                g.set_output_units(binding.OUTPUT_TANH_SQERR)
            if "front" in done and (g is fresh or what == "front"):
                g.set_fixed_frontend(filters, np.zeros(2, dtype=np.int32), 1)
        got, want = run(kept, batch), run(fresh, batch)
        assert np.array_equal(got, want), (what, batch)
        fresh.close()
    kept.close()


@pytest.mark.parametrize("arch,most,batches", [("1x29x29-20C4-MP2-40C5-MP3-150N-10N", 100, (88, 60, 1)),
                                               ("2x48x48-50C5-MP2-128C3-MP4-100N-5N", 33, (7, 1))])
def test_scratch_memory_for_a_batch_is_enough_for_what_remains_of_a_set(arch, most, batches):
    """Fewer images may run in 32-bit products, which take more memory, where more run in halves."""
    import torch
    g, _ = build_pair(arch=arch)
    scratch = _scratch(g, most)
    d_imgs = to_dev((np.random.default_rng(3).random((most, g.image_size)) * 2 - 1).astype(np.float32))
    assert any(not binding.batch_plan(arch, b)[0][1]["split"] for b in batches) and binding.batch_plan(arch, most)[0][1]["split"]
    one = torch.empty(most * g.num_classes, dtype=torch.float32, device="cuda:0")
    g.forward_many(d_imgs, most, one)
    for batch in batches:
        probs = torch.empty(batch * g.num_classes, dtype=torch.float32, device="cuda:0")
        g.forward_batch(d_imgs[:batch], batch, probs, scratch, batch)
        g.synchronize()
        assert (probs - one[:len(probs)]).abs().max().item() <= 1e-5
    g.close()


def test_a_handle_that_goes_back_and_forth_between_batches_keeps_their_plans():
    """Asking for the memory of two batches in turn takes about what asking for one's again and again does: a plan made anew is 16 us
    or more for this network, the call 0.6."""
    import time
    g = binding.Cnn("3x40x40-240C3-MP2-240C3-MP1-240C3-MP1-240C3-300N-100N-4N")

    def us(batches):
        for b in batches:
            g.forward_batch_scratch_bytes(b)
        times = []
        for _ in range(100):
            start = time.perf_counter()
            for b in batches:
                g.forward_batch_scratch_bytes(b)
            times.append((time.perf_counter() - start) / len(batches) * 1e6)
        return sorted(times)[50]

    one, two, four = us([512] * 4), us([512, 65] * 2), us([512, 65, 7, 300])
    print("us a call", one, two, four, flush=True)
    assert max(two, four) <= 3 * one + 5, (one, two, four)
    g.close()
