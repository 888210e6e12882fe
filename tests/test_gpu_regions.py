"""Listing where a tile holds one, two and more regions, labels mixed at random
or in runs, against the oracle bit for bit, on each kernel instance."""
import numpy as np
import pytest

from paper_1610_02258_amd import inputs as I
from tests.randmodels import random_counts, random_model


@pytest.mark.gpu
@pytest.mark.parametrize("n_regions", [2, 3, 8])
@pytest.mark.parametrize("labels", ["mixed", "runs", "one odd"])
@pytest.mark.parametrize("S,R", [(4, 4), (7, 8), (10, 12), (15, 20), (16, 32)])
def test_regions_match_oracle(oracle_lib, S, R, labels, n_regions):
    from paper_1610_02258_amd import rdx
    rng = np.random.default_rng(100 * S + R + n_regions)
    mesh = I.box_mesh(4, 4, 3, 0.5e-6, jitter=0.1, seed=S).as_dict()
    T = len(mesh["tets"])
    reg = {"mixed": rng.integers(0, n_regions, T), "runs": np.arange(T) // 5 % n_regions,
           "one odd": np.where(np.arange(T) % 17 == 16, rng.integers(0, n_regions, T), n_regions - 1)}[labels]
    mesh["region"] = reg.astype(np.uint8)
    md = random_model(rng, S, R, n_regions)
    md["kcst"] *= 1e-4 / oracle_lib.Instance(mesh, md, 9).tau
    md["kcst"][:, md["lhs"].sum(1) == 0] *= 0.01
    counts = random_counts(rng, S, T, 2.0)
    print(f"case: S={S} R={R} {labels} {n_regions} regions", flush=True)
    ref = oracle_lib.Instance(mesh, md, 9)
    ref.reset(counts)
    ref.step(4)
    sim = rdx.Sim(mesh, md, 9)
    sim.set_counts(counts)
    sim.step(4)
    np.testing.assert_array_equal(sim.get_counts(), ref.counts)
    assert sim.stats().ssa_events == ref.tallies.ssa_events > 0
    sim.close()
