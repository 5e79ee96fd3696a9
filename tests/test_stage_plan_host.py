"""Host logic of the stage planner (no GPU): networks of wide layers -- up to 600 maps, kernels up to 7 x 7 -- are all
planned, and the work items of every stage cover their layer."""
import random
import re

import pytest

from paper_1102_0183_amd import binding


def random_wide_arch(rng):
    h = rng.randint(8, 60)
    w = h if rng.random() < 0.6 else rng.randint(8, 60)
    s = "%dx%dx%d" % (rng.randint(1, 4), h, w)
    for _ in range(rng.randint(1, 4)):
        k, skip = rng.randint(1, min(7, h, w)), rng.choice([0, 0, 0, 1, 2])
        h, w = (h - k) // (skip + 1) + 1, (w - k) // (skip + 1) + 1
        s += "-%dC%d%s" % (round(2 * 300 ** rng.random()), k, "S%d" % skip if skip else "")
        if rng.random() < 0.7:
            pool = rng.choice([q for q in range(1, 8) if h % q == 0 and w % q == 0])
            s += "-MP%d" % pool
            h, w = h // pool, w // pool
        if min(h, w) < 2:
            break
    return s + "".join("-%dN" % rng.randint(2, 500) for _ in range(rng.randint(0, 2))) + "-%dN" % rng.randint(2, 10)


def stages(arch):
    out = []
    for line in binding.plan_text(arch).splitlines():
        name = line.split()[1]
        out.append((name, {k: int(v) for k, v in re.findall(r"(\w+)=(-?\d+)", line)}))
    return out


ADJUSTMENTS = ("conv_wgrad", "conv_wgrad_win", "conv_wgrad_first")


def shares_a_launch(plan, s):
    """With the sums of its layer's pull or an adjustment before it, or a vector pull or an adjustment behind it."""
    before, after = plan[s - 1] if s else None, plan[s + 1] if s + 1 < len(plan) else None
    return (before and not before[1]["barrier"] and before[0] in ADJUSTMENTS + ("conv_bwd_epi", "conv_bwd_wepi")) or \
        (after and not plan[s][1]["barrier"] and after[0] in ADJUSTMENTS + ("conv_bwd",))


def check(arch):
    layers = [i for i in binding.arch_info(arch) if i["kind"] != binding.LAYER_POOL]
    plan = stages(arch)
    for s, (name, f) in enumerate(plan):
        below, layer = layers[f["layer"]], layers[f["layer"] + 1]
        if name == "conv_wgrad_win":
            assert f["items"] == -(-below["maps"] // 64) * -(-layer["maps"] // f["chunk"]), (arch, f)
            # a work item for 64 input maps and an output map: half a round of them, or company
            assert -(-below["maps"] // 64) * layer["maps"] >= 128 or shares_a_launch(plan, s), (arch, f)
        if name == "conv_wgrad_mfma":
            assert (f["tiles"] - 1) * f["chunk"] < below["maps"] <= f["tiles"] * f["chunk"], (arch, f)
            assert f["items"] == -(-layer["maps"] // 32) * f["tiles"], (arch, f)
            # column tiles of 32 weights, four to a wavefront at most
            assert -(-min(f["chunk"], below["maps"]) * layer["K"] ** 2 // 32) <= 64, (arch, f)


@pytest.mark.parametrize("arch", ["1x28x28-431C6-274C7-500N-3N", "1x24x24-518C1-MP2-518C5-MP4-10N-3N",
                                  "1x43x43-389C6-MP2-427C6-10N-10N"])
def test_gradient_products_of_more_than_35_column_tiles_are_planned(arch):
    check(arch)
    K = binding.arch_info(arch)[3 if "MP2" in arch else 2]["K"]
    assert any(n == "conv_wgrad_mfma" and f["chunk"] * K * K > 35 * 32 for n, f in stages(arch)), arch


# few input maps: the vector kernels keep a layer whose product would be few items' long walks, and gradients of a map an item
@pytest.mark.parametrize("arch,product,gradients", [
    ("8x15x15-73C5S1-MP2-20N-5N", 0, 0), ("6x23x23-203C6-MP9-20N-5N", 0, 0), ("2x22x22-191C3-MP5-66N-8N", 0, 0),
    ("9x14x14-100C3-MP3-20N-5N", 0, 0), ("7x22x22-382C5-MP9-20N-5N", 0, 1),
    ("2x17x17-129C6-MP2-20N-5N", 1, 0), ("1x48x48-129C7-MP7-20N-5N", 1, 0), ("1x20x20-256C5-MP2-20N-5N", 1, 0),
    ("1x20x20-257C5-MP2-20N-5N", 1, 1), ("3x32x32-300C3-MP2-300C2-MP2-300C4-MP2-300N-10N", 1, 1)])
def test_which_kernels_take_a_layer_of_few_input_maps(arch, product, gradients):
    first = [name for name, f in stages(arch) if f["layer"] == 0]
    assert ("conv_fwd_mx" in first, "conv_wgrad_first" in first) == (bool(product), bool(gradients)), first


def test_adjustments_beside_a_pulls_sums_keep_short_lists_where_winners_are_many():
    """Next to the sums of its layer's pull an adjustment has fewer compute units; its lists of connections stay as long as all of
    them allow where a thread would else walk many more winners (1024 for 512 here), and get longer where it is a few."""
    def of(arch):
        return [f for name, f in stages(arch) if name == "conv_wgrad" and f["layer"] == 1][0]
    assert of("3x123x123-36C7-MP3-48C8-MP1-21N-20N-2N")["chunk"] == 8     # 36 maps in 256 // 48 lists
    assert of("1x45x41-105C2-MP1-13C5-MP2-20N-4N")["chunk"] == 8          # 105 maps in (256 - 64) // 13 lists


def test_random_wide_architectures_are_planned():
    rng = random.Random(1102)
    for _ in range(4000):
        check(random_wide_arch(rng))
