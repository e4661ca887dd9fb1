"""Stage B of the re-check (the definition's sums, added many terms at a time) on rays whose
pixel depends on the last bit of the sum: every ray of the middle column sits on the mirror
axis of its lenses, so that its deflection is rounding noise, and the map's left edge lies
on that axis."""
import numpy as np
import pytest

import oracle

pytestmark = pytest.mark.gpu


def _mirrored(n, seed, masses):
    rng = np.random.default_rng(seed)
    r = max(3.0, 1.5 * np.sqrt(n))   # a fixed density: the rays stay in the map's rows
    half = rng.uniform(-r, r, size=((n + 1) // 2, 2))
    xy = np.concatenate([half, half * [-1.0, 1.0]])[:n]
    m = np.tile(rng.uniform(0.1, 1.9, (n + 1) // 2), 2)[:n] if masses else None
    order = rng.permutation(n)
    return xy[order], None if m is None else m[order]


# lens counts at the edges of a lane's 8 lenses, of 64 lanes' 512 and of several such chunks
@pytest.mark.parametrize("n", [2, 8, 10, 510, 512, 514, 1024, 4098])
@pytest.mark.parametrize("masses", [False, True])
@pytest.mark.parametrize("mode", ["mixed", "farfield"])
def test_rays_on_the_mirror_axis(n, masses, mode):
    import paper_1005_5198_amd as rs
    xy, m = _mirrored(n, n, masses)
    p = rs.map_params(0.4, 0.0, 0.1, (-2.0625, -2.0, 4.125, 4.0, 33, 64), (0.0, -4.0, 8.0, 8.0, 64, 64))
    pix, st = rs.ray_pixels(p, xy, m, mode=mode, return_stats=True)
    ref, _, _ = oracle.ray_pixels(p, xy, m)
    assert np.array_equal(pix.cpu().numpy(), np.asarray(ref).reshape(-1))
    assert st["rays_rechecked_direct"] >= 32   # the middle column's rays reach the stages over every lens
