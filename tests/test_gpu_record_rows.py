"""Per-region sums where a row's tets are no multiple of four (rows that start
off a 16-byte boundary, a remainder) and where a block's last loads pass the
row's end, for each number of accumulators."""
import numpy as np
import pytest

from paper_1610_02258_amd import inputs as I
from tests.randmodels import random_model

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n_regions", [1, 2, 3, 8])
@pytest.mark.parametrize("T", [1, 2, 3, 5, 1023, 1026, 4097, 16390, 33001])
def test_region_sums_of_ragged_rows(T, n_regions):
    from paper_1610_02258_amd import rdx
    n = 1
    while 6 * n ** 3 < T:
        n += 1
    mesh = I.box_mesh(n, n, n, 0.5e-6, jitter=0.1, seed=T).as_dict()
    rng = np.random.default_rng(T + n_regions)
    label = rng.integers(0, n_regions, T).astype(np.uint8)
    mesh = dict(verts=mesh["verts"], tets=np.asarray(mesh["tets"])[:T], region=label if n_regions > 1 else None)
    counts = rng.integers(0, 1 << 30, (5, T)).astype(np.int32)
    print(f"case: T={T} regions {n_regions}", flush=True)
    sim = rdx.Sim(mesh, random_model(rng, 5, 2, n_regions), 1, tau_override=1e-6)
    sim.set_counts(counts)
    want = [[int(counts[s, label == g].astype(np.int64).sum()) for s in range(5)] for g in range(n_regions)]
    np.testing.assert_array_equal(sim.region_counts(), want)
    sim.close()
