"""Launch choices by map size: eight-wave blocks up to 256 patches (FP32 mode) and 512 (mixed),
records built by the clearing launch up to 4096, the exact stage in stage A's kernel up to 2048
lenses. The bars are exact: FP32 maps do not depend on the thread shape, and mixed maps equal
the definition's, which exact_recheck reaches without the far-field stage."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


def _case(nbx, nby, n, masses, ragged):
    rng = np.random.default_rng(nbx * 1000 + n)
    r = np.sqrt(n / 0.4)
    xy = rng.uniform(-r, r, (n, 2))
    m = rng.uniform(0.2, 3.0, n) if masses else None
    import paper_1005_5198_amd as rs
    p = rs.map_params(0.4, 0.0, 0.1, (-8.0, -6.0, 16.0, 12.0, 64 * nbx - ragged, 32 * nby - ragged),
                      (-4.0, -4.0, 8.0, 8.0, 192, 176))
    return p, xy, m


# patches 1, 255, 256, 257 (a prime row), 512, 513, 4096, 4097
@pytest.mark.parametrize("nbx,nby", [(1, 1), (15, 17), (16, 16), (257, 1), (32, 16), (27, 19), (64, 64), (241, 17)])
@pytest.mark.parametrize("n,masses", [(30, False), (463, True), (2048, False), (2049, True)])
def test_sizes_at_the_choices(nbx, nby, n, masses):
    import paper_1005_5198_amd as rs
    p, xy, m = _case(nbx, nby, n, masses, ragged=(n % 2) * 5)
    lens = rs.lens_tensors(xy, m)
    mixed = rs.make_map(p, *lens, mode="mixed").view(torch.int32)
    exact = rs.make_map(p, *lens, mode="mixed", exact_recheck=True).view(torch.int32)
    assert torch.equal(mixed, exact)
    fp32 = rs.make_map(p, *lens, mode="fp32").view(torch.int32)
    before = rs.set_shape(1)
    try:
        assert torch.equal(fp32, rs.make_map(p, *lens, mode="fp32").view(torch.int32))
        assert torch.equal(mixed, rs.make_map(p, *lens, mode="mixed").view(torch.int32))
    finally:
        rs.set_shape(before)
