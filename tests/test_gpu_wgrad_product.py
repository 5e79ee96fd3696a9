"""Weight gradients of wide layers as a matrix product, and the adjustment that follows them, at the edges of their tiles
-- 32 output maps, column tiles of 32 weights one to a wavefront, shared by several, and several to one -- against the
oracle."""
import numpy as np
import pytest

from paper_1102_0183_amd import binding
from tests.parity_helpers import TOL_ACT, build_pair, layer_bounds, rel_err, to_dev

pytestmark = pytest.mark.gpu

CASES = [
    ("1x10x10-97C3-390C3-MP3-9N-3N", "a row tile of 30 maps; columns shared by wavefronts"),
    ("1x12x12-130C3-257C3-MP4-9N-3N", "one map over; a column tile not filled"),
    ("1x9x9-300C3-300C4-MP2-9N-3N", "four winners a map"),
    ("2x9x9-700C4-1900C2-MP5-8N-3N", "several column tiles a wavefront"),
    ("1x24x24-518C1-MP2-518C5-MP4-10N-3N", "41 column tiles"),
]


@pytest.mark.parametrize("arch,what", CASES)
def test_gradient_products_match_the_oracle(arch, what):
    print("case", arch, what, flush=True)
    g, o = build_pair(arch=arch, seed=len(arch))
    g.set_mode(binding.MODE_STAGES)
    assert "conv_wgrad_mfma" in g.plan_text()
    info = o.layer_info(0)
    rng = np.random.default_rng(len(arch))
    img = (rng.random((info["maps"], info["h"], info["w"]), dtype=np.float32) * 2 - 1).astype(np.float32)
    d_img = to_dev(img)
    grad = g.debug_gradients(d_img, 1)
    grad_o, _ = o.gradients(img, 1)
    for a, b in layer_bounds(o):
        assert rel_err(grad[a:b], grad_o[a:b]) <= TOL_ACT, (a, b)
    o.train_step(img, 2, 0.1)
    g.train_step(d_img, 2, 0.1)
    assert rel_err(g.get_weights(), o.get_weights()) <= TOL_ACT
    g.close()
