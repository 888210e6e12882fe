"""Every tile width (64, 32 and 16 tets) with static and with claimed tiles, on
a quarter of the resident blocks, against the oracle bit for bit.  The width
follows from the number of tiles, as stated at the rule: the test repeats it,
so that a box that no longer takes its width is seen."""
import numpy as np
import pytest

from paper_1610_02258_amd import inputs as I
from tests.randmodels import random_counts, random_model


def _width(tiles, resident, claim, S, R):
    most = resident * 5 // 4 if claim else resident // 2
    shift = 6
    while shift > 4 and tiles << (7 - shift) <= most and (R > 0 or S << (shift - 1) > 32):
        shift -= 1
    return 1 << shift


CASES = [((8, 8, 19), 3, 5, 16, 16), ((13, 13, 15), 3, 5, 32, 16), ((18, 18, 19), 3, 5, 64, 32),
         ((20, 20, 19), 3, 5, 64, 64), ((8, 8, 19), 1, 0, 64, 64), ((8, 8, 19), 2, 0, 32, 32), ((8, 8, 19), 3, 0, 16, 16)]


@pytest.mark.gpu
@pytest.mark.parametrize("claim", [0, 1])
@pytest.mark.parametrize("box,S,R,static,claimed", CASES)
def test_each_width_matches_oracle(oracle_lib, box, S, R, static, claimed, claim):
    import torch
    from paper_1610_02258_amd import rdx
    rng = np.random.default_rng(sum(box) + S)
    mesh = I.box_mesh(*box, 0.5e-6, jitter=0.1, seed=3).as_dict()
    T = len(mesh["tets"])
    resident = 16 * torch.cuda.get_device_properties(0).multi_processor_count // 4  # up to 12 species: 16 blocks a CU
    assert _width((T + 63) // 64, resident, claim, S, R) == (claimed if claim else static)
    md = random_model(rng, S, R)
    if R:
        md["kcst"] *= 3e-4 / oracle_lib.Instance(mesh, md, 5).tau
        md["kcst"][:, md["lhs"].sum(1) == 0] *= 0.01
    counts = random_counts(rng, S, T, 6.0)
    print(f"case: T={T} S={S} R={R} tile_claim {claim}", flush=True)
    ref = oracle_lib.Instance(mesh, md, 5)
    sim = rdx.Sim(mesh, md, 5)
    sim.set_exec_options(fast_grid_div=4, graph_windows=2, tile_claim=claim)
    ref.reset(counts)
    sim.set_counts(counts)
    for k in (1, 4):
        ref.step(k)
        sim.step(k)
        np.testing.assert_array_equal(sim.get_counts(), ref.counts)
    sim.close()
