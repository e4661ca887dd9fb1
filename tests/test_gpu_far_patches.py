"""Far-field maps with about as many patches as the ray kernel has blocks (three per CU), twice
and three times that, and more per block and ticket: each ray counted once, and the map the
direct kernel's."""
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


@pytest.mark.parametrize("per_block,extra", [(0, 1), (0, 33), (1, -1), (1, 0), (1, 1), (2, -1), (2, 0), (2, 1), (3, 1),
                                             (16, 0), (64, 5)])
def test_patches_per_block(per_block, extra):
    import numpy as np
    import paper_1005_5198_amd as rs
    blocks = 3 * torch.cuda.get_device_properties(0).multi_processor_count
    patches = per_block * blocks + extra
    # one row of patches, or rows of 512 and a partly filled window
    nx, ny = (64 * patches, 32) if patches <= 2048 else (64 * 512, 32 * -(-patches // 512))
    xy = np.random.default_rng(patches).uniform(-30.0, 30.0, (40, 2))
    p = rs.map_params(0.1, 0.0, 0.1, (-25.0, -5.0, 50.0, 10.0, nx, ny), (-20.0, -6.0, 40.0, 12.0, 200, 60))
    far, st = rs.make_map(p, xy, mode="farfield", return_stats=True)
    assert st["rays_shot"] == nx * ny
    assert torch.equal(far.view(torch.int32), rs.make_map(p, xy, mode="mixed").view(torch.int32))
