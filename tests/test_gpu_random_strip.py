"""Random rays in more bins than a block counts in LDS at once: the strip's one launch of
2^26 rays has 48000 bins, each half of it at most 24000. Counts are the definition's in both,
so the halves' maps add up to the whole's."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


def test_strip_equals_its_halves():
    import paper_1005_5198_amd as rs
    rng = np.random.default_rng(5)
    sw = 16308.0
    xy = np.stack([rng.uniform(-sw / 2, sw / 2, 40), rng.uniform(-2.0, 2.0, 40)], axis=1)
    p = rs.map_params(0.1, 0.0, 0.0, (-sw / 2, -0.5, sw, 1.0, 1 << 21, 32), (-sw / 2, -1.0, sw, 2.0, 4096, 16))
    p.update(random_rays=1, seed=9)

    def run(j0, j1):
        return rs.make_map(dict(p, j0=j0, j1=j1), *rs.lens_tensors(xy), mode="mixed").cpu().numpy().astype(np.int64)
    whole = run(0, 32)
    assert whole.sum() > 1 << 25
    assert np.array_equal(whole, run(0, 16) + run(16, 32))
