"""Far-field maps around the numbers of near lenses where the ray kernel changes its source:
none, what a record holds (24), the block's own list (512), beyond it (the patch is re-checked
whole), with and without masses, on a window that is no multiple of a patch. The map is the
definition's whatever the path, so it equals the exact re-check's."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


@pytest.mark.parametrize("cluster", [0, 1, 23, 24, 25, 511, 512, 513, 700])
@pytest.mark.parametrize("masses", [False, True])
def test_near_lenses_of_one_patch(cluster, masses):
    import paper_1005_5198_amd as rs
    rng = np.random.default_rng(cluster + masses)
    # 300 lenses over the field, and a cluster inside one patch of 0.64 x 0.32
    xy = np.concatenate([rng.uniform(-30.0, 30.0, (300, 2)), rng.uniform(0.05, 0.25, (cluster, 2))])
    m = np.concatenate([rng.uniform(0.2, 3.0, 300), np.full(cluster, 0.01)]) if masses else None
    p = rs.map_params(0.3, 0.0, 0.05, (-3.2, -1.6, 6.4, 3.2, 640, 320), (-20.0, -20.0, 40.0, 40.0, 400, 300),
                      window=(3, 637, 5, 318))
    lens = rs.lens_tensors(xy, m)
    far = rs.make_map(p, *lens, mode="farfield").view(torch.int32)
    exact = rs.make_map(p, *lens, mode="mixed", exact_recheck=True).view(torch.int32)
    assert torch.equal(far, exact)
