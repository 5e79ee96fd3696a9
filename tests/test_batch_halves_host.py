"""Host logic of the products of halves in the batched pass (no GPU): which layers take them, and what they take of memory,
over the benchmark networks and seeded random ones, from one image to thousands."""
import pytest

from paper_1102_0183_amd import binding, synth
from tests.test_batch_plan_host import ARCHS, BATCHES, LDS


@pytest.mark.parametrize("arch", ARCHS)
def test_products_of_halves_fit_and_take_no_more_scratch_memory(arch):
    """A caller whose scratch memory was enough for a batch with 32-bit products goes on with it; halves only behind a layer that
    writes them, and only before a layer that reads them."""
    for batch in BATCHES:
        layers, whole = binding.batch_plan(arch, batch)
        assert whole["floats"] <= whole["floats_32"], batch
        for l, p in enumerate(layers):
            where = (batch, l, p)
            if p["first"]:
                assert l == 0 and layers[1]["split"] and p["Mi"] * p["KK"] <= 16 * p["first_H"] and p["first_lds"] <= LDS, where
            if p["split"]:
                below = layers[l - 1]
                assert l > 0 and (below["split"] or below["first"]), where
                if p["split_fc"]:   # (behind a layer of p["Mi"] outputs: maps of its pixels)
                    assert not p["conv"] and l + 1 < len(layers) and p["split_slab"] == p["split_kg"] and p["split_IC"] <= p["Mi"], where
                    assert p["split_slices"] <= max(1, p["gemm_KS"]) and p["split_lds"] <= LDS, where
                    continue
                groups = -(-p["Mi"] // 8)
                step = 2 if p["split_TR"] == 32 else 4
                assert groups % p["split_IC"] == 0 and p["split_lds"] <= LDS, where
                assert p["split_kg"] == -(-p["split_IC"] * p["KK"] // step) * step and p["split_slab"] % step == 0, where
                assert 0 < p["split_slab"] <= p["split_kg"] and p["split_px"] % 64 == 0, where


@pytest.mark.parametrize("name,batch,layers", [("cfg2a", 4096, 3), ("cfg3", 33, 3), ("cfg4a", 512, 4), ("cfg4b", 512, 4)])
def test_the_benchmark_networks_take_them(name, batch, layers):
    plan, whole = binding.batch_plan(synth.WORKLOADS[name].arch, batch)
    assert whole["tail"] and plan[0]["first"] and [p["split"] for p in plan[:layers]] == [0] + [1] * (layers - 1)


def test_which_last_layers_are_one_launch():
    """Up to 1024 hidden neurons, 64 outputs and 48 KB of weights between them, behind a hidden layer."""
    for hidden, classes, one in ((1024, 12, 1), (1025, 4, 0), (192, 64, 1), (100, 65, 0), (1024, 13, 0)):
        assert binding.batch_plan("1x9x9-4C2-MP2-%dN-%dN" % (hidden, classes), 33)[1]["tail"] == one
    assert binding.batch_plan("1x9x9-4C2-MP2-10N", 33)[1]["tail"] == 0


def test_rows_of_many_inputs_keep_the_32_bit_products():
    """Each piece of a row that is turned into halves reads the row for its scale: 1.4 times as slow at 134480 inputs."""
    assert not binding.batch_plan("3x43x43-17C1-MP1-80C3-MP1-600N-12N", 33)[0][2]["split"]


def test_single_images_keep_the_32_bit_products():
    """Their layers are launches and waits, whichever the kernel; measured up to 1.2 times as slow in halves."""
    for arch in ("1x13x13-100C2-MP1-5C4S1-MP1-4N", "2x21x21-100C1-MP1-150C2S1-MP1-4N", "3x53x53-100C2-MP1-40C1S1-MP1-4N"):
        assert not any(p["split"] or p["first"] for p in binding.batch_plan(arch, 1)[0])


@pytest.mark.parametrize("arch", ARCHS)
def test_running_sums_end_after_32_groups(arch):
    """A running sum is whole slabs of weights, as many as are 32 groups of eight terms together, or one."""
    for batch in BATCHES:
        for p in binding.batch_plan(arch, batch)[0]:
            assert not p["split"] or p["split_slab"] <= 32, (batch, p)


@pytest.mark.parametrize("maps", range(33, 335, 5))
def test_no_workgroup_of_the_first_layer_has_few_maps(maps):
    """One or two maps of a pixel are all tiny by chance, which the layer behind takes for a layer of tiny activations there."""
    for arch in ("1x29x29-%dC4-MP2-40C5-MP3-150N-10N", "3x32x32-%dC3-MP2-100C2-MP2-10N", "3x32x32-%dC5-MP2-64C5-MP2-10N", "2x96x96-%dC6S1-MP2-150C4-MP4-5N"):
        for batch in (33, 300):
            p = binding.batch_plan(arch % maps, batch)[0][0]
            if not p["first"] or maps <= p["first_T"] * 32:
                continue
            rows = p["first_T"] * 32
            groups = -(-maps // rows)
            assert maps + p["first_shift"] <= groups * rows and p["first_shift"] % 8 == 0
            assert maps - ((groups - 1) * rows - p["first_shift"]) > 8, (arch % maps, batch, p)
