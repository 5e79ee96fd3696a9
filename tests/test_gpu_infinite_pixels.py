"""An infinite pixel reaches what its sums reach and nothing else: the operands with which a kernel fills its last group of taps
are no product of zero and a pixel."""
import numpy as np
import pytest

from paper_1102_0183_amd import binding
from tests.parity_helpers import TOL_ACT, build_pair, rel_err, to_dev

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("arch,stage", [("3x17x17-100C3S1-MP2-10N-3N", "conv_fwd_mx"),     # 27 taps
                                        ("2x22x30-65C5-MP2-10N-3N", "conv_fwd_mx"),        # 50
                                        ("1x30x30-64C3-10N-3N", "conv_fwd_mx")])           # 9, no pooling
@pytest.mark.parametrize("sign", [1, -1])
def test_an_infinite_pixel_saturates_the_units_above_it(arch, stage, sign):
    print("case", arch, sign, flush=True)
    g, o = build_pair(arch=arch, seed=len(arch))
    g.set_mode(binding.MODE_STAGES)
    assert stage in g.plan_text()
    info = o.layer_info(0)
    rng = np.random.default_rng(2)
    img = (rng.random((info["maps"], info["h"], info["w"]), dtype=np.float32) * 2 - 1).astype(np.float32)
    img[0, 6, 8] = sign * np.inf
    probs = to_dev(np.zeros(g.num_classes, dtype=np.float32))
    g.forward(to_dev(img).view(-1), probs)
    want = o.forward(img)
    for l in range(1, o.num_layers):
        assert np.isfinite(o.activation(l)).all() and rel_err(g.activation(l), o.activation(l)) <= TOL_ACT, l
    assert np.abs(probs.cpu().numpy() - np.asarray(want).ravel()).max() <= TOL_ACT
    g.close()
