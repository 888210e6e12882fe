"""Per-region sums on both sides of the size where a lane goes from one load to
four (51 blocks of 1,024 tets at 5 species), and with remainders there."""
import numpy as np
import pytest

from paper_1610_02258_amd import inputs as I
from tests.randmodels import random_model


@pytest.mark.gpu
@pytest.mark.parametrize("n_regions", [1, 2, 3, 8])
@pytest.mark.parametrize("T", [51 * 1024 - 1, 51 * 1024, 51 * 1024 + 1, 90001])
def test_region_sums_around_the_switch(T, n_regions):
    from paper_1610_02258_amd import rdx
    mesh = I.box_mesh(25, 25, 25, 0.5e-6, jitter=0.1, seed=3).as_dict()
    rng = np.random.default_rng(T + n_regions)
    label = rng.integers(0, n_regions, T).astype(np.uint8)
    mesh = dict(verts=mesh["verts"], tets=np.asarray(mesh["tets"])[:T], region=label if n_regions > 1 else None)
    assert len(mesh["tets"]) == T
    counts = rng.integers(0, 1 << 30, (5, T)).astype(np.int32)
    print(f"case: T={T} regions {n_regions}", flush=True)
    sim = rdx.Sim(mesh, random_model(rng, 5, 2, n_regions), 1, tau_override=1e-6)
    sim.set_counts(counts)
    want = [[int(counts[s, label == g].astype(np.int64).sum()) for s in range(5)] for g in range(n_regions)]
    np.testing.assert_array_equal(sim.region_counts(), want)
    sim.close()
