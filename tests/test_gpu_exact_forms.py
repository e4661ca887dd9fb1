"""Stage B of the re-check in each of its forms (the chain of additions, the sums many terms at
a time) and places (the far-field re-check's kernel, a kernel of its own, the gathered list, the
batch), at the lens counts where one takes over from another: 2048, 8192 and 32768. Every ray of
the middle column sits on the mirror axis of its lenses, its deflection is rounding noise, and
the map's left edge lies on the axis, so that its pixel is the last bit of the sum."""
import numpy as np
import pytest

import oracle

pytestmark = pytest.mark.gpu

COUNTS = [1, 2046, 2048, 2050, 8190, 8192, 8194, 32766, 32768, 32770]


def _mirrored(n, masses):
    rng = np.random.default_rng(n)
    r = max(3.0, 1.5 * np.sqrt(n))   # a fixed density: the rays stay in the map's rows
    half = rng.uniform(-r, r, size=((n + 1) // 2, 2))
    xy = np.concatenate([half, half * [-1.0, 1.0]])[:n]
    m = np.tile(rng.uniform(0.1, 1.9, (n + 1) // 2), 2)[:n] if masses else None
    order = rng.permutation(n)
    return xy[order], None if m is None else m[order]


def _params(rs):
    return rs.map_params(0.4, 0.0, 0.1, (-2.0625, -2.0, 4.125, 4.0, 33, 64), (0.0, -4.0, 8.0, 8.0, 64, 64))


@pytest.mark.parametrize("n", COUNTS + [12290, 40002, 131070, 131074])
@pytest.mark.parametrize("masses", [False, True])
@pytest.mark.parametrize("mode", ["mixed", "farfield"])
def test_single_maps(n, masses, mode):
    import paper_1005_5198_amd as rs
    p = _params(rs)
    xy, m = _mirrored(n, masses)
    pix = rs.ray_pixels(p, xy, m, mode=mode)
    ref, _, _ = oracle.ray_pixels(p, xy, m)
    assert np.array_equal(pix.cpu().numpy(), np.asarray(ref).reshape(-1))


@pytest.mark.parametrize("top", [32768, 32770])
@pytest.mark.parametrize("masses", [False, True])
def test_batches(top, masses):
    """Batches whose longest map is and is not past the chain's limit."""
    import paper_1005_5198_amd as rs
    p = _params(rs)
    lenses = [_mirrored(n, masses and n % 4 == 2) for n in COUNTS if n <= top]
    outs = rs.make_maps([(p, xy, m) for xy, m in lenses], mode="mixed")
    for (xy, m), out in zip(lenses, outs):
        assert np.array_equal(out.cpu().numpy(), oracle.make_map(p, xy, m)[0]), len(xy)
