"""Small mixed maps, at the sizes where the launch changes, against the oracle: the wide and the
default thread shape, unit lenses and masses (which multiply the factors that four rays share),
ragged windows, the pixel table's lines and the counters."""
import numpy as np
import pytest

import oracle

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


def _case(nbx, nby, n, masses, ragged):
    import paper_1005_5198_amd as rs
    rng = np.random.default_rng(nbx * 1000 + n)
    r = np.sqrt(n / 0.4)
    xy = rng.uniform(-r, r, (n, 2))
    # (masses over six decades: large ones overflow the shared factors, small ones nearly vanish)
    m = 10.0 ** rng.uniform(-4.0, 2.0, n) if masses else None
    p = rs.map_params(0.4, 0.0, 0.1, (-8.0, -6.0, 16.0, 12.0, 64 * nbx - ragged, 32 * nby - ragged),
                      (-4.0, -4.0, 8.0, 8.0, 191, 177))
    return p, xy, m


# patches 1, 255, 256, 257 (a prime row), 512, 513
@pytest.mark.parametrize("nbx,nby", [(1, 1), (15, 17), (16, 16), (257, 1), (32, 16), (27, 19)])
@pytest.mark.parametrize("n", [1, 30, 463])
@pytest.mark.parametrize("masses", [False, True])
def test_small_maps_equal_the_oracle(nbx, nby, n, masses):
    import paper_1005_5198_amd as rs
    p, xy, m = _case(nbx, nby, n, masses, ragged=(n % 2) * 5)
    out, st = rs.make_map(p, xy, m, mode="mixed", return_stats=True)
    ref, st_o = oracle.make_map(p, xy, m)
    assert np.array_equal(out.cpu().numpy(), ref)
    for key in ("rays_in_map", "rays_out", "rays_singular"):
        assert st[key] == st_o[key], key
    assert int(ref.sum()) == st["rays_in_map"]


@pytest.mark.parametrize("nbx,nby", [(64, 64), (241, 17)])   # 4096 and 4097 patches
@pytest.mark.parametrize("n,masses", [(30, False), (463, True), (2048, False), (2049, True)])
@pytest.mark.parametrize("mode", ["mixed", "fp32", "farfield"])
def test_every_ray_is_counted(nbx, nby, n, masses, mode):
    import paper_1005_5198_amd as rs
    p, xy, m = _case(nbx, nby, n, masses, ragged=5)
    out, st = rs.make_map(p, xy, m, mode=mode, return_stats=True)
    rays = (p["i1"] - p["i0"]) * (p["j1"] - p["j0"])
    assert st["rays_shot"] == rays == st["rays_in_map"] + st["rays_out"] + st["rays_singular"]
    assert int(out.view(torch.int32).sum(dtype=torch.int64)) == st["rays_in_map"]
