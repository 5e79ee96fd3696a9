"""A handle that goes from mode to mode: each has a stage list of its own (a wide first layer's forward stage is not one the
persistent kernel holds), so every one of the six switches, and the fall-back of a team that cannot hold the network, must
leave the plan of the mode that runs.  The plan is asserted before anything is launched on it."""
import numpy as np
import pytest

from paper_1102_0183_amd import binding
from tests.parity_helpers import TOL_ACT, build_pair, compare_backward_state, compare_forward_state, rel_err, to_dev

pytestmark = pytest.mark.gpu

ARCH = "1x18x18-64C3-MP2-66C3-MP2-20N-4N"     # two ranks cannot hold it, 66 can
S, P, R = binding.MODE_STAGES, binding.MODE_PERSISTENT, binding.MODE_RESIDENT


def _check(g, o, w0, mode):
    assert g.mode == mode
    plan = g.plan_text()
    assert ("conv_fwd_mx" in plan) == (mode != P), plan
    assert ("conv_wgrad_win" in plan) == (mode == S), plan
    print("mode", mode, flush=True)
    rng = np.random.default_rng(4)
    imgs = (rng.random((5, 1, 18, 18), dtype=np.float32) * 2 - 1).astype(np.float32)
    d_imgs = to_dev(imgs)
    o.set_weights(w0.astype(np.float64))
    g.set_weights(w0)
    grad, (grad_o, _) = g.debug_gradients(d_imgs[0].contiguous().view(-1), 1), o.gradients(imgs[0], 1)
    compare_forward_state(g, o)
    compare_backward_state(g, o)
    assert rel_err(grad, grad_o) <= TOL_ACT
    want = o.forward_many(imgs, 5)
    for n in (1, 5):      # (on both sides of where a resident forward call runs as launches of its stages)
        probs = to_dev(np.zeros((n, 4), dtype=np.float32))
        g.forward_many(d_imgs[5 - n:].contiguous(), n, probs)
        g.synchronize()
        assert np.abs(probs.cpu().numpy() - want[5 - n:]).max() <= TOL_ACT, n
    g.train_step(d_imgs[1].contiguous().view(-1), 2, 0.1)
    o.train_step(imgs[1], 2, 0.1)
    assert rel_err(g.get_weights(), o.get_weights()) <= TOL_ACT


def test_every_switch_of_modes_runs_the_plan_of_the_mode_it_went_to():
    g, o = build_pair(arch=ARCH, seed=3)
    w0 = g.get_weights()
    _check(g, o, w0, S)
    for mode in (P, S, R, P, R, S):
        g.set_mode(mode)
        _check(g, o, w0, mode)
    g.close()


def test_a_team_that_cannot_hold_the_network_leaves_the_persistent_plan():
    g, o = build_pair(arch=ARCH, seed=3)
    w0 = g.get_weights()
    g.set_mode(R)
    with pytest.raises(binding.CnnError) as e:
        g.set_team(2, 1)
    assert e.value.code == binding.E_STATE and "LDS" in str(e.value)
    _check(g, o, w0, P)
    with pytest.raises(binding.CnnError):
        g.set_mode(R)
    _check(g, o, w0, P)
    g.set_team(0, 0)
    g.set_mode(R)
    _check(g, o, w0, R)
    g.close()
