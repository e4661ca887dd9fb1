"""A forced thread shape is the one that runs, and the tuner times and reports the shapes that the
map itself would run, whatever the size of its sample."""
import os
import re
import subprocess
import sys

import numpy as np
import pytest

import oracle

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def _map(rs, nbx, nby, n=100):
    xy = np.random.default_rng(n).uniform(-15.0, 15.0, (n, 2))
    p = rs.map_params(0.3, 0.0, 0.1, (-8.0, -6.0, 16.0, 12.0, 64 * nbx, 32 * nby), (-4.0, -4.0, 8.0, 8.0, 96, 96))
    return p, xy


def test_tuner_reports_the_shapes_of_the_map():
    import paper_1005_5198_amd as rs
    cus = torch.cuda.get_device_properties(0).multi_processor_count
    for mode, per_cu in (("mixed", 2), ("fp32", 1)):
        for patches, wide in ((per_cu * cus, True), (per_cu * cus + 1, False), (8 * cus, False)):
            p, xy = _map(rs, patches, 1)
            for sample in (1 << 12, 1 << 30):
                r = rs.tune(p, xy, mode=mode, sample_rays=sample)
                got = r["shapes"][0]
                assert (got["rays_per_lane"], got["threads"]) == (((2, 2), 512) if wide else ((4, 2), 256))
                assert [s["threads"] for s in r["shapes"][1:]] == [128, 128, 64]


def test_a_forced_shape_runs():
    """The launch plan that the library prints names the shape of each launch."""
    code = """
import sys; sys.path.insert(0, %r); sys.path.insert(0, %r)
import paper_1005_5198_amd as rs, test_gpu_shapes as t
for shape in (-1, 0, 1, 2, 3):
    rs.set_shape(shape)
    for nbx, nby in ((4, 2), (64, 64)):
        rs.make_map(*t._map(rs, nbx, nby), mode="mixed")
""" % (ROOT, os.path.join(ROOT, "tests"))
    p = subprocess.run([sys.executable, "-c", code], env=dict(os.environ, RAYSHOOT_DEBUG="1"), capture_output=True,
                       text=True, timeout=100)
    assert p.returncode == 0, p.stderr[-2000:]
    shapes = [int(s) for s in re.findall(r"\[rayshoot\] map .* shape (-?\d+)", p.stderr)]
    assert shapes == [4, 0, 0, 0, 1, 1, 2, 2, 3, 3]


@pytest.mark.parametrize("nbx,nby", [(12, 7), (27, 19)])   # below and past two patches per CU
@pytest.mark.parametrize("masses", [False, True])
def test_forced_and_built_in_shapes_give_the_oracle_map(nbx, nby, masses):
    import paper_1005_5198_amd as rs
    p, xy = _map(rs, nbx, nby)
    m = np.random.default_rng(1).uniform(0.1, 3.0, len(xy)) if masses else None
    ref, _ = oracle.make_map(p, xy, m)
    fp32 = []
    try:
        for shape in (-1, 0, 1, 2, 3):
            rs.set_shape(shape)
            assert np.array_equal(rs.make_map(p, xy, m, mode="mixed").cpu().numpy(), ref), shape
            fp32.append(rs.make_map(p, xy, m, mode="fp32").view(torch.int32))
    finally:
        rs.set_shape(-1)
    assert all(torch.equal(fp32[0], f) for f in fp32[1:])


def test_default_tuning_is_the_work_of_four_million_rays():
    import paper_1005_5198_amd as rs
    from paper_1005_5198_amd import workloads as w
    s = w.config2()
    r = rs.tune(s.params, s.lens_xy)
    assert 0.9 * (1 << 22) * s.n_lens < r["sample_interactions"] <= (1 << 22) * s.n_lens


def test_a_programs_first_launches_do_not_count_against_the_first_shape():
    """Tuning as the first GPU work of a process. On this map 4 x 2 rays per lane is 2 to 3%
    ahead of the next shape and the sample's first launches take up to 8% longer than later
    ones."""
    code = """
import sys; sys.path.insert(0, %r)
import paper_1005_5198_amd as rs
from paper_1005_5198_amd import workloads as w
s = w.config2()
r = rs.tune(s.params, s.lens_xy)
print("best", r["best"], [x["ms"] for x in r["shapes"]])
""" % ROOT
    p = subprocess.run([sys.executable, "-c", code], capture_output=True, text=True, timeout=100)
    assert p.returncode == 0, p.stderr[-2000:]
    assert p.stdout.startswith("best 0"), p.stdout
