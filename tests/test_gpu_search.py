"""The binomial search steps its cdf in passes of eight terms: sizes at the
edges of a pass and of a chunk of 1000 trials, with answers at both ends of
the range, against the oracle bit for bit."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("m", [1, 7, 8, 9, 15, 16, 17, 64, 999, 1000, 1001, 1008, 2047])
@pytest.mark.parametrize("p", [2.0**-40, 0.01, 0.5, 0.97])
def test_search_pass_edges(oracle_lib, m, p):
    from paper_1610_02258_amd import rdx
    print(f"case: Bin({m}, {p})", flush=True)
    got = rdx.selftest_binom(7, m, p, 8192, stream_id=2, window=5)
    ref = oracle_lib.sample_binom(7, m, p, 8192, stream_id=2, window=5)
    np.testing.assert_array_equal(got, ref)
