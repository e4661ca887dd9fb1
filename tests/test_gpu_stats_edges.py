"""Map statistics at the edges of the kernels' tiles and ranges against the oracle.

Tolerances, from the FP64 arithmetic: counts exact; D to 2 ulp(1) (the same CDF values are
differenced); the RMS to n 2^-53 + 1e-13 over n terms; dm to 4 ulp (the device's and the
host's logarithm are each within one)."""
import numpy as np
import pytest

import oracle
from oracle import stats as S

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


def dev(a):
    return torch.from_numpy(np.ascontiguousarray(a)).cuda()


# largest counts at the ends of the on-chip bins and table (4096), of a scan tile (4096 bins),
# of one tile per block (1024 tiles) and several tiles per block
@pytest.mark.parametrize("top", [1, 4094, 4095, 4096, 8191, 8192, 4194303, 4194304, 9000001])
@pytest.mark.parametrize("npix", [1, 5, 1027, 4 * 1024 + 1])
def test_compare_at_the_ends_of_the_bins(npix, top):
    import paper_1005_5198_amd as rs
    rng = np.random.default_rng(top + npix)
    a = rng.integers(0, top + 1, npix).astype(np.uint32)
    b = (rng.integers(0, 2 * top + 1, npix) // 3 * 3).astype(np.uint32)
    a[0], b[-1] = top, 2 * top
    for nr_a, nr_b in ((top / 3.0, 2 * top / 3.0), (7.0, 7.0), (0.3, 11.0)):
        ref = S.compare_maps(a, b, nr_a, nr_b)
        got = rs.compare_maps(dev(a), dev(b), nr_a, nr_b, max_a=top + 5, max_b=2 * top)
        for k in ("max_a", "max_b", "n_zero_a", "n_zero_b", "n_both"):
            assert got[k] == ref[k], k
        assert got["ks_d"] == pytest.approx(ref["ks_d"], abs=4.5e-16)
        assert got["rms_dm"] == pytest.approx(ref["rms_dm"], rel=npix * 2.0 ** -53 + 1e-13, abs=1e-13, nan_ok=True)


# map sizes about the least that uses the table form, aligned and not
@pytest.mark.parametrize("npix", [6291455, 6291456, 6291459])
@pytest.mark.parametrize("skip", [0, 1])
def test_delta_m_of_large_maps(npix, skip):
    import paper_1005_5198_amd as rs
    rng = np.random.default_rng(npix)
    c = rng.integers(0, 5000, npix + skip).astype(np.uint32)
    c[:3] = 0, 4095, 4096
    got = rs.delta_m(dev(c)[skip:], 700.0).cpu().numpy()
    ref = S.delta_m(c[skip:], 700.0)
    fin = np.isfinite(ref)
    assert np.array_equal(fin, np.isfinite(got)) and np.all(got[~fin] == np.inf)
    assert np.all(np.abs(got[fin] - ref[fin]) <= 4 * np.spacing(np.abs(ref[fin])) + 1e-300)
