"""Host logic of the batched forward pass (no GPU): the plan of every layer -- kernel, tile, chunks, slices of the k
range -- against rules restated here, over the benchmark networks, the paper's and seeded random ones, from one image
to thousands."""
import numpy as np
import pytest

from paper_1102_0183_amd import binding, synth

LDS = 160 * 1024
BATCHES = (1, 2, 7, 16, 33, 64, 128, 300, 512, 1000, 4096)


def random_archs(n, seed):
    rng = np.random.default_rng(seed)
    out = []
    while len(out) < n:
        c, h = int(rng.integers(1, 5)), int(rng.integers(8, 50))
        s, layers = "%dx%dx%d" % (c, h, h), 0
        for _ in range(int(rng.integers(1, 5))):
            k, skip = int(rng.integers(1, 6)), int(rng.integers(0, 4) == 0)
            if h < k + 1:
                break
            h = (h - k) // (skip + 1) + 1
            pool = int(rng.choice([q for q in (1, 2, 3, 4, 5) if h % q == 0]))
            h //= pool
            s += "-%dC%d%s-MP%d" % (int(rng.choice([3, 16, 17, 33, 80, 100, 150, 161, 300])), k, "S1" if skip else "", pool)
            layers += 1
        if layers:
            out.append(s + "-%dN-5N" % int(rng.integers(5, 300)))
    return out


ARCHS = sorted({w.arch for w in synth.WORKLOADS.values()}) + random_archs(40, 21)


@pytest.mark.parametrize("arch", ARCHS)
def test_partial_sums_are_those_of_the_general_product(arch):
    """k_batch_conv takes a layer over from k_batch_gemm: its partial sums are those of the k slices there (rounding of
    a sum in 32 bits grows with its length), and its planes no more (the caller's scratch memory)."""
    for batch in BATCHES:
        layers, _ = binding.batch_plan(arch, batch)
        for l, p in enumerate(layers):
            where = (batch, l, p)
            assert p["run"] == p["gemm_run"], where
            assert p["n_slices"] == p["gemm_KS"], where
            assert (p["n_slices"] - 1) * p["run"] < p["Mi"] <= p["n_slices"] * p["run"], where
            assert 1 <= p["IC"] <= p["Mi"], where
            assert p["lds_bytes"] <= LDS, where


@pytest.mark.parametrize("classes", [2, 5, 10, 47, 1000])
@pytest.mark.parametrize("hidden", ["", "-300N", "-1200N"])
def test_output_units_add_planes_only_where_they_are_few(classes, hidden):
    """One thread adds an image's planes, class after class: a handful of rounds of eight loads, no more."""
    arch = "1x24x24-40C3-MP2%s-%dN" % (hidden, classes)
    for batch in BATCHES:
        layers, whole = binding.batch_plan(arch, batch)
        rounds = classes * -(-layers[-1]["n_slices"] // 8)
        assert whole["outputs_add"] == (layers[-1]["fuse"] == 0 and rounds <= 8), (batch, layers[-1], whole)


@pytest.mark.parametrize("arch,batch", [("100x4x4-100C4-10N", 5000), ("128x3x3-100C3-10N", 5000), ("64x2x2-64C2-10N", 700),
                                        ("300x1x1-300C1-10N", 5000), ("36x6x6-72C6-5N", 4837), ("1x81x81-4C6-MP2-5N", 1289),
                                        ("1x63x63-1C4-MP4-5N", 2882)])
def test_blocks_of_many_small_images_or_of_a_small_part_of_one_stay_with_the_general_product(arch, batch):
    """Measured 1.2 to 4.5 times as slow in k_batch_conv."""
    assert not binding.batch_plan(arch, batch)[0][0]["conv"]


@pytest.mark.parametrize("name,batch,layers", [("cfg2a", 4096, 2), ("cfg3", 33, 2), ("cfg4a", 512, 3), ("cfg4b", 512, 3), ("cfg5", 1024, 2)])
def test_the_benchmark_networks_convolutional_layers_run_in_the_persistent_kernel(name, batch, layers):
    plan, _ = binding.batch_plan(synth.WORKLOADS[name].arch, batch)
    assert [p["conv"] for p in plan[:layers]] == [1] * layers


def test_the_gpu_test_of_the_tiles_reaches_every_one():
    from tests.test_gpu_batch import TILES
    for arch, batch, MT, TR, members, raw, sliced, resident, several in TILES:
        p = binding.batch_plan(arch, batch)[0][0]
        assert p["conv"] and (p["MT"], p["TR"], p["members"]) == (MT, TR, members), (arch, batch, p)
        assert (p["fuse"] == 0, p["n_slices"] > 1, bool(p["resident"]), p["n_cb"] > p["gx"]) == (raw, sliced, resident, several), (arch, p)
    assert {t[2:4] for t in TILES} == {(m, 16) for m in range(1, 8)} | {(m, 32) for m in range(1, 6)}
