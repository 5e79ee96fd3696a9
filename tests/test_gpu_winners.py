"""Stage kernels that visit the pooling winners only (a lane per input map): the delta pull and the weight gradients of
wide layers, at the edges of their tiles -- 64 input maps, groups of pooling windows, 16 output maps a work item, slices
of the output maps -- against the oracle."""
import numpy as np
import pytest

from paper_1102_0183_amd import binding
from tests.parity_helpers import (TOL_ACT, build_pair, compare_backward_state, compare_forward_state, layer_bounds,
                                  rel_err, to_dev)

pytestmark = pytest.mark.gpu

# input maps, pixels, output maps, kernel, pooling: what lies on the edge
CASES = [
    (64, 19, 150, 4, 4, "one full group of lanes, a group of windows and one more"),
    (65, 17, 121, 3, 3, "one map in the last group of lanes, five windows of six"),
    (130, 8, 110, 3, 2, "two maps in the last group of lanes, slices of unequal length"),
    (64, 21, 33, 4, 2, "eight windows and one more, one slice"),
    (127, 22, 40, 3, 4, "one idle lane, four windows and one more"),
    (70, 20, 90, 5, 4, "the largest kernel and window, two windows a group"),
    (64, 14, 215, 5, 2, "five windows of a group of six"),
    (100, 13, 64, 5, 3, "a group of windows not filled, filters of 25"),
    (33, 13, 70, 2, 2, "gradients only: 33 input maps, filters of four"),
    (64, 23, 17, 4, 4, "one output map over the wavefronts of an item"),
]


@pytest.mark.parametrize("Mi,H,Mo,K,Kp,what", CASES)
def test_winner_kernels_match_the_oracle(Mi, H, Mo, K, Kp, what):
    arch = "1x%dx%d-%dC3-%dC%d-MP%d-20N-4N" % (H + 2, H + 2, Mi, Mo, K, Kp)
    print("case", arch, what, flush=True)
    g, o = build_pair(arch=arch, seed=Mi + Mo)
    g.set_mode(binding.MODE_STAGES)
    plan = g.plan_text()
    HW = ((H - K + 1) // Kp) ** 2
    assert "conv_wgrad_win" in plan
    assert ("conv_bwd_win" in plan) == (Mi >= 64 and Mi * Mo * HW * K * K >= (1 << 23 if (K, Kp) == (5, 2) else 1 << 20))
    rng = np.random.default_rng(Mi)
    imgs = (rng.random((3, 1, H + 2, H + 2), dtype=np.float32) * 2 - 1).astype(np.float32)
    d_img = to_dev(imgs[0])
    grad = g.debug_gradients(d_img, 1)
    grad_o, _ = o.gradients(imgs[0], 1)
    compare_forward_state(g, o)
    compare_backward_state(g, o)
    for a, b in layer_bounds(o):
        assert rel_err(grad[a:b], grad_o[a:b]) <= TOL_ACT, (a, b)
    # the adjustment, with a rate that shows whether the pull has read the old weights; three calls as one
    w0 = g.get_weights()
    for t in range(3):
        g.train_step(to_dev(imgs[t]), t, 0.1)
    o.set_weights(w0.astype(np.float64))
    o.train_step(imgs[0], 0, 0.1)
    many = g.get_weights()
    g.set_weights(w0)
    g.train_step(d_img, 0, 0.1)
    assert rel_err(g.get_weights(), o.get_weights()) <= TOL_ACT
    g.set_weights(w0)
    g.train_many(to_dev(imgs), to_dev(np.arange(3, dtype=np.int32)), 0.1)
    np.testing.assert_array_equal(g.get_weights(), many)
    g.close()
