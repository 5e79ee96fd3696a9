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


# architecture, pixels of a work item of the pull's sums: what lies on the edge
UNEVEN = [
    ("1x25x21-193C3-60C4-MP4-9N-3N", 27, "rows longer than columns, one map in the last group of lanes, three windows and one more"),
    ("1x24x26-129C3-70C5-MP2-9N-3N", 24, "seven windows and three more, up to three regions above each other, 25 taps"),
    ("1x22x28-130C3-66C3-MP3-9N-3N", 24, "six windows and two more, a short last block of pixels"),
    ("1x23x15-64C3-150C4-MP2-9N-3N", 16, "a pixel a wavefront, five windows of eight"),
    ("1x16x24-33C3-130C3S1-MP2-9N-3N", 0, "gradients only: skipping factor 1, an input row and column left over"),
]


@pytest.mark.parametrize("arch,pixels,what", UNEVEN)
def test_winner_kernels_on_maps_that_are_not_square(arch, pixels, what):
    """Also the sums of the pull with more than 16 pixels an item: their terms in flight together."""
    print("case", arch, what, flush=True)
    g, o = build_pair(arch=arch, seed=len(arch))
    g.set_mode(binding.MODE_STAGES)
    plan = g.plan_text()
    assert "conv_wgrad_win" in plan
    sums = [line for line in plan.splitlines() if "conv_bwd_wepi" in line]
    assert (len(sums) == 1 and "chunk=%d " % pixels in sums[0]) if pixels else not sums
    _gradients_and_a_step(g, o)


# the two stages of one launch
PAIRS = [
    ("1x16x24-33C3-130C3S1-MP2-9N-3N", "conv_wgrad_win", "conv_wgrad"),
    ("40x14x16-130C3-MP2-20C3S1-9N-3N", "conv_wgrad", "conv_wgrad_win"),
    ("40x22x18-130C3-MP2-20C3-MP2-9N-3N", "conv_wgrad_win", "conv_wgrad_win"),
    ("1x22x18-260C3-MP2-20C3-MP2-9N-3N", "conv_wgrad_win", "conv_wgrad_first"),
    ("1x28x24-12C3-40C3-MP2-20C3-MP2-9N-3N", "conv_wgrad_win", "conv_bwd"),
    ("1x20x24-5C3-6C3-260C3-MP2-9N-3N", "conv_wgrad_first", "conv_bwd"),
    ("1x20x24-6C3-260C3-MP2-9N-3N", "conv_wgrad_first", "conv_wgrad"),
    ("1x20x22-260C3-20C3S1-9N-3N", "conv_wgrad", "conv_wgrad_first"),
]


@pytest.mark.parametrize("arch,one,other", PAIRS)
def test_stages_that_share_a_launch_match_the_oracle(arch, one, other):
    print("case", arch, one, other, flush=True)
    g, o = build_pair(arch=arch, seed=len(arch))
    g.set_mode(binding.MODE_STAGES)
    plan = [(line.split()[1], "barrier=1" in line) for line in g.plan_text().splitlines()]
    assert any(a == (one, False) and b[0] == other for a, b in zip(plan, plan[1:])), plan
    _gradients_and_a_step(g, o)


def _gradients_and_a_step(g, o):
    info = o.layer_info(0)
    rng = np.random.default_rng(7)
    img = (rng.random((info["maps"], info["h"], info["w"]), dtype=np.float32) * 2 - 1).astype(np.float32)
    d_img = to_dev(img).view(-1)
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
