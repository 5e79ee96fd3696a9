"""Stage kernels of a wide first layer (many output maps on few input maps, one image at a time) at the edges of their
tiles -- 32 output maps, 16 pixels, four taps, bands of rows -- against the oracle."""
import numpy as np
import pytest

from paper_1102_0183_amd import binding
from tests.parity_helpers import (TOL_ACT, build_pair, compare_backward_state, compare_forward_state, layer_bounds,
                                  rel_err, to_dev)

pytestmark = pytest.mark.gpu

# architecture, whether the forward product and the gradients over the whole input in LDS take the layer
CASES = [
    ("1x9x9-64C2-MP4-10N-3N", 1, 0, "four taps, one window row a band"),
    ("2x22x30-65C5-MP2-10N-3N", 1, 0, "a tile of one map, taps not a multiple of four, 13 windows a row"),
    ("3x17x17-100C3S1-MP2-10N-3N", 1, 0, "skipping factor 1, input rows left over at the right and bottom"),
    ("3x13x13-96C3-10N-3N", 1, 0, "no pooling: eleven pixels a row"),
    ("3x20x20-70C9-MP3-10N-3N", 0, 0, "243 taps, twelve items: the vector kernels"),
    ("2x40x40-257C6S1-MP3-12N-3N", 1, 1, "nine tiles of maps, the last of one"),
    ("1x33x7-64C4-MP2-10N-3N", 1, 0, "bands of four pixels a row"),
    ("1x30x30-640C3-MP2-6N-3N", 1, 1, "more items than one round in the smallest bands, three maps an item"),
    ("1x9x9-770C2-MP4-10N-3N", 1, 1, "four taps, four maps an item"),
    ("2x22x30-321C5-MP2-10N-3N", 1, 1, "50 taps, an item of one map, rows of 30"),
    ("3x17x17-300C3S1-MP2-10N-3N", 1, 1, "skipping factor 1, input rows left over"),
    ("3x13x13-258C3-10N-3N", 1, 1, "no pooling"),
    ("3x20x20-262C9-MP3-10N-3N", 1, 1, "243 taps: three groups of 64 and 51"),
    ("1x33x7-513C4-MP2-10N-3N", 1, 1, "rows of seven, three maps an item"),
]


@pytest.mark.parametrize("arch,product,gradients,what", CASES)
def test_first_layer_kernels_match_the_oracle(arch, product, gradients, what):
    print("case", arch, what, flush=True)
    g, o = build_pair(arch=arch, seed=len(arch))
    g.set_mode(binding.MODE_STAGES)
    assert ("conv_fwd_mx" in g.plan_text(), "conv_wgrad_first" in g.plan_text()) == (bool(product), bool(gradients))
    info = o.layer_info(0)
    rng = np.random.default_rng(len(arch))
    img = (rng.random((info["maps"], info["h"], info["w"]), dtype=np.float32) * 2 - 1).astype(np.float32)
    d_img = to_dev(img)
    grad = g.debug_gradients(d_img, 1)
    grad_o, _ = o.gradients(img, 1)
    compare_forward_state(g, o)
    compare_backward_state(g, o)
    for a, b in layer_bounds(o):
        assert rel_err(grad[a:b], grad_o[a:b]) <= TOL_ACT, (a, b)
    o.train_step(img, 2, 0.1)
    g.train_step(d_img, 2, 0.1)
    assert rel_err(g.get_weights(), o.get_weights()) <= TOL_ACT
    g.close()
