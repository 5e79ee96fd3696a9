"""The matrix product of a wide layer with one buffer in LDS -- maps of more than 512 pixels, maps and kernels of which half of the
LDS holds none, the persistent kernel -- at the edges of its tiles, against the oracle."""
import re

import numpy as np
import pytest

from paper_1102_0183_amd import binding
from tests.parity_helpers import (TOL_ACT, build_pair, compare_backward_state, compare_forward_state, layer_bounds,
                                  rel_err, to_dev)

pytestmark = pytest.mark.gpu

S, P = binding.MODE_STAGES, binding.MODE_PERSISTENT

# architecture, stage, its layer, buffers, mode
CASES = [
    ("1x32x32-30C3-65C3-MP4-10N-3N", "conv_mfma", 1, 1, S, "784 pixels, a row tile of one map, taps that are no whole eights"),
    ("1x32x32-30C3-65C3-MP4-10N-3N", "conv_mfma", 1, 1, P, "the same in the persistent kernel"),
    ("2x20x24-33C3-65C3-MP2-10N-3N", "conv_mfma", 1, 2, S, "320 pixels: two buffers"),
    ("2x20x24-33C3-65C3-MP2-10N-3N", "conv_mfma", 1, 1, P, "a wavefront's one tile in one buffer"),
    ("5x30x32-66C25-MP2-9N-3N", "conv_mfma", 0, 1, S, "a kernel of which half of LDS holds no 32 rows"),
    ("70x130x130-64C3S2-9N-3N", "conv_mfma", 0, 1, S, "maps that half of LDS does not hold, 1849 pixels, two chunks a slice"),
    ("70x130x130-64C3S2-9N-3N", "conv_mfma", 0, 1, P, "the same in the persistent kernel"),
    ("40x126x135-64C12S7-9N-3N", "conv_mfma", 0, 1, S, "such a map under 240 pixels: the wavefronts share a tile"),
    ("1x40x50-64C24-9N-3N", "conv_fwd ", 0, 0, S, "so few items that the vector kernel takes the layer"),
    ("2x25x25-40C3-140C23-9N-3N", "conv_bwd_mfma", 1, 1, S, "a pull of which half of LDS holds no 32 rows, three chunks a slice"),
    ("1x28x30-33C3-66C4-MP1-9N-3N", "conv_bwd_mfma", 1, 1, S, "a pull into 728 pixels"),
]


@pytest.mark.parametrize("arch,stage,layer,buffers,mode,what", CASES)
def test_products_match_the_oracle(arch, stage, layer, buffers, mode, what):
    print("case", arch, mode, what, flush=True)
    g, o = build_pair(arch=arch, seed=len(arch), wscale=0.02)
    g.set_mode(mode)
    lines = [l for l in g.plan_text().splitlines() if re.match(r" *\d+ " + stage, l) and "layer=%d " % layer in l]
    assert len(lines) == 1 and (buffers == 0 or "rows=%d " % buffers in lines[0]), g.plan_text()
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
