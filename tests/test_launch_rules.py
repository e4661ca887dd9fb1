"""The rules that size launches, on the CPU (no device): tests/launch_driver.cpp links only
paper_1005_5198_amd/csrc/rs_launch.h (pure host logic)."""
import os
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_1005_5198_amd", "csrc")


@pytest.fixture(scope="module")
def ask(tmp_path_factory):
    exe = str(tmp_path_factory.mktemp("launch") / "launch_driver")
    subprocess.run(["g++", "-std=c++17", "-O1", "-Wall", "-Werror", "-fsanitize=address,undefined",
                    "-fno-sanitize-recover=all", "-I", CSRC, "-I", os.path.join(ROOT, "include"),
                    os.path.join(ROOT, "tests", "launch_driver.cpp"), "-o", exe], check=True)

    def run(what, *args):
        return run.many([(what, *args)])

    def many(queries):
        lines = "".join(" ".join(map(str, q)) + "\n" for q in queries)
        out = subprocess.run([exe], input=lines, check=True, capture_output=True, text=True).stdout
        return [int(v) for v in out.split()]
    run.many = many
    return run


@pytest.mark.parametrize("per_block,cap", [(1, 2048), (4, 1024), (4, 512), (256, 2048)])
def test_a_queue_fills_the_chip_before_rays_wait(ask, per_block, cap):
    """Every ray of a queue has its place (a wave, a block or a thread) until the grid is full:
    none waits for another while blocks could still be added."""
    for entries in (0, 1, per_block, per_block + 1, 64, 2048, 33 * 64, per_block * cap - 1, per_block * cap,
                    per_block * cap + 1, 1 << 27):
        blocks, = ask("queue_blocks", entries, per_block, cap)
        assert 1 <= blocks <= cap
        assert blocks == cap or blocks * per_block >= entries
        assert (blocks - 1) * per_block < max(entries, 1)   # and no block without one


def _function(source, name):
    text = open(os.path.join(CSRC, source)).read()
    body = text[text.index("hipError_t " + name + "("):]
    return body[:body.index("\n}\n")]


@pytest.mark.parametrize("source,name,per_block", [("farfield.hip", "launch_recheck_far", 4),
                                                   ("recheck.hip", "launch_recheck", 1)])
def test_short_queue_forms_are_launched_by_that_rule(source, name, per_block):
    """The kernels with a wave or a block per ray get their grid from it."""
    body = _function(source, name)
    assert f"queue_blocks(max_rays, {per_block}," in body and "/ 256" not in body


@pytest.mark.parametrize("n_waves", [1, 4, 2048, 4096])
def test_a_long_queue_gives_every_wave_some_entries(ask, n_waves):
    """The runs of adjacent entries that waves take in turn cover the queue with at most a
    lane's worth each, and while waves are left without any, no run is longer than its share."""
    for entries in (1, 63, 64, 65, 32769, 65536, 64 * n_waves - 1, 64 * n_waves, 64 * n_waves + 1, 1 << 27):
        run, = ask("entry_run", entries, n_waves)
        assert 1 <= run <= 64
        assert run == 64 or run * n_waves >= entries
        assert (run - 1) * n_waves < entries


def test_one_kernel_for_the_stages_of_small_maps_only(ask):
    """Stage A shares stage F's kernel only where a call is short; what stage F leaves of a
    larger map is dealt out again by a kernel of its own."""
    assert ask("recheck_in_one", 1 << 20, 462, 0, 0) == [1]
    assert ask("recheck_in_one", 1 << 20, 462, 1, 0) == [0]
    assert ask("recheck_in_one", 1 << 19, 5000, 0, 0) == [0]
    assert ask("recheck_in_one", 19200 * 3840, 17240, 0, 0) == [0]
    assert ask("recheck_in_one", 1 << 27, 1 << 40, 0, 0) == [0]   # (no overflow)
    # crowded maps, most of whose rays come to stage A: fewer pairs
    assert ask("recheck_in_one", 256 * 256, 3000, 0, 1) == [1]
    assert ask("recheck_in_one", 512 * 512, 1500, 0, 1) == [0]
    assert ask("recheck_in_one", 512 * 512, 1500, 0, 0) == [1]


def test_crowded_maps(ask):
    """Maps whose lists cannot hold the lenses nearby, most of whose rays come to stage A; by the
    whole ray grid, not a window or launch of it."""
    assert ask("crowded", 3000, 3000, 300000) == [1]
    assert ask("crowded", 19200, 3840, 17240) == [0]
    assert ask("crowded", 55902, 55902, 10 ** 6) == [0]   # (a launch of it has 130 rays per lens)
    assert ask("crowded", 256, 1000, 1000) == [0] and ask("crowded", 255, 1000, 1000) == [1]
    assert ask("crowded", 1 << 27, 1, 1 << 62) == [1] and ask("crowded", 1 << 51, 1 << 51, 1) == [0]   # (no overflow)
    assert ask("crowded", 0, 0, 0) == [0]


def test_crowded_is_asked_of_the_whole_grid():
    assert "crowded(a.nx, a.ny, a.n_lens)" in _function("recheck.hip", "launch_recheck")


@pytest.mark.parametrize("blocks", [1, 2, 32, 768])
def test_no_block_takes_two_patches_before_every_block_has_one(ask, blocks):
    """The far-field ray kernel's blocks hold two patches at a time. Whatever the order in which
    they start, each patch is taken once, and up to two patches per block are shared evenly."""
    first = ask.many([("first_patch", b, blocks, turn) for turn in (0, 1) for b in range(blocks)])
    tickets = ask.many([("ticket_patch", t, blocks) for t in range(5)])
    assert sorted(first) + tickets == list(range(2 * blocks + 5))   # each once, tickets after them
    assert first[:blocks] == list(range(blocks))                    # the first round gives each block one


def test_the_far_field_ray_kernel_starts_by_that_rule():
    text = open(os.path.join(CSRC, "farfield.hip")).read()
    body = text[text.index("void farfield_kernel("):text.index("void recheck_far_kernel(")]
    assert "patch = first_patch(blockIdx.x, gridDim.x, 0), next = first_patch(blockIdx.x, gridDim.x, 1)" in body
    assert "ticket_patch(share++, gridDim.x)" in body


@pytest.mark.parametrize("cus", [64, 256, 304])
def test_built_in_shape(ask, cus):
    """Eight-wave blocks while there are no more patches than two per CU (FP32 mode: one), else
    shape 0; by the device's number of CUs."""
    for mixed, per_cu in ((1, 2), (0, 1)):
        wide, at, past = ask.many([("default_shape", mixed, p, cus) for p in (1, per_cu * cus, per_cu * cus + 1)])
        assert wide == at == 4 and past == 0


def test_tuner_sample(ask):
    """The work asked for and no more (but for the least of 32 rows), in bands that stay in the
    window; more rays with fewer lenses where there are lenses enough."""
    cases = [(W, H, n, rays) for W in (1, 64, 5003, 19200, 1 << 22) for H in (1, 31, 32, 3001, 3840, 1 << 52)
             for n in (0, 1, 462, 2047, 2048, 3331, 17240, 10 ** 6) for rays in (1, 1 << 20, 1 << 22, 1 << 24, (1 << 63) - 1)]
    got = ask.many([("tune_sample", *c) for c in cases])
    for (W, H, n, rays), rows, lenses in zip(cases, got[::2], got[1::2]):
        assert 1 <= rows <= H and (rows % 32 == 0 or rows == H)
        assert (n < 2048 and lenses == n) or n // 4 <= lenses <= n
        if rows > 32:
            assert rows * W * lenses <= rays * n
    # the 19200 x 3840-ray, 17240-lens map: four times the rays, a quarter of the lenses
    rows, lenses = ask("tune_sample", 19200, 3840, 17240, 1 << 22)
    assert rows == 864 and 0.95 * (1 << 22) * 17240 <= 19200 * rows * lenses <= (1 << 22) * 17240
    assert ask("tune_sample", 32768, 32768, 462, 1 << 22) == [128, 462]
    assert ask("tune_sample", 1024, 1024, 462, 1 << 22) == [1024, 462]      # the whole window
    assert ask("tune_sample", 1 << 22, 1 << 52, 17240, 1 << 22) == [32, 4310]
    assert ask("tune_sample", 1, 1 << 52, 17240, (1 << 63) - 1) == [1 << 52, 17240]   # (no overflow)


def test_the_tuner_asks_for_four_million_rays():
    import inspect

    from paper_1005_5198_amd import api
    assert inspect.signature(api.tune).parameters["sample_rays"].default == 1 << 22
    assert "if (sample_rays <= 0) sample_rays = int64_t(1) << 22;" in open(os.path.join(CSRC, "tune.cpp")).read()
