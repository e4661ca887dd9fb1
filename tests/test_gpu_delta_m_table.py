"""dm of large maps, where it may come from an on-chip table of the counts below 4096.

dm to 4 ulp of the oracle's (the device's and the host's logarithm are each within one)."""
import numpy as np
import pytest

import oracle  # noqa: F401
from oracle import stats as S

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

TABLE_MIN = 6291456   # pixels from which the table form runs


@pytest.mark.parametrize("npix", [TABLE_MIN, TABLE_MIN + 3, 8 * 1024 * 1024 + 1])
@pytest.mark.parametrize("low", [0.0, 0.5, 1.0])   # share of the map's pixels, in one piece, below 4096
def test_values_where_blocks_choose_differently(npix, low):
    import paper_1005_5198_amd as rs
    rng = np.random.default_rng(npix)
    c = rng.integers(4096, 1 << 32, npix, dtype=np.uint32)
    k = int(low * npix)
    c[:k] = rng.integers(0, 4097, k)
    c[-3:] = 0, 4095, 4096
    got = rs.delta_m(torch.from_numpy(c).cuda(), 5.0e4).cpu().numpy()
    ref = S.delta_m(c, 5.0e4)
    fin = np.isfinite(ref)
    assert np.array_equal(fin, np.isfinite(got)) and np.all(got[~fin] == np.inf)
    assert np.all(np.abs(got[fin] - ref[fin]) <= 4 * np.spacing(np.abs(ref[fin])) + 1e-300)


def test_no_table_is_made_for_counts_beyond_it():
    """Tables made for nothing: 39 us; the plain form: 24."""
    import paper_1005_5198_amd as rs
    c = torch.full((TABLE_MIN,), 70000, dtype=torch.int32, device="cuda").view(torch.uint32)

    def best(x):
        times = []
        for _ in range(40):
            a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
            a.record()
            for _ in range(10):
                rs.delta_m(x, 5.0e4)
            b.record()
            b.synchronize()
            times.append(a.elapsed_time(b))
        return min(times)

    best(c)
    with_choice, plain = best(c), best(c[:TABLE_MIN - 4])
    assert with_choice <= 1.2 * plain, (with_choice, plain)
