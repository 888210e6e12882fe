"""Tiles whose every tet has events in most of its species: more changed items
than are held at a time, up to the items' whole space, for the largest tables
and for few species beside many reactions, against the oracle bit for bit."""
import numpy as np
import pytest

from paper_1610_02258_amd import inputs as I


@pytest.mark.gpu
@pytest.mark.parametrize("mean,events", [(2.0, 1.0), (6.0, 12.0), (30.0, 40.0)])
@pytest.mark.parametrize("S,R", [(16, 32), (16, 24), (16, 3), (13, 32), (13, 13), (6, 30), (3, 25), (1, 32), (1, 13),
                                 (12, 12), (4, 4)])
def test_changed_items_match_oracle(oracle_lib, S, R, mean, events):
    from paper_1610_02258_amd import rdx
    rng = np.random.default_rng(100 * S + R)
    mesh = I.box_mesh(4, 3, 6, 0.5e-6, jitter=0.1, seed=S).as_dict()
    T = len(mesh["tets"])
    lhs, rhs = np.zeros((R, S), np.int32), np.zeros((R, S), np.int32)
    for r in range(R):  # species in a ring; the only one grows and shrinks
        lhs[r, r % S] = 1
        rhs[r, (r + 1 + r // S) % S] += 1 if S > 1 else 2 * (r % 2)
    md = dict(D=np.where(np.arange(S) % 5 == 3, 0.0, 1e-12), lhs=lhs, rhs=rhs, kcst=np.ones((1, R)))
    md["kcst"][:] = events / (mean * R * oracle_lib.Instance(mesh, md, 21).tau)
    counts = rng.poisson(mean, (S, T)).astype(np.int32)
    print(f"case: S={S} R={R} mean {mean} events {events}", flush=True)
    ref = oracle_lib.Instance(mesh, md, 21)
    ref.reset(counts)
    sim = rdx.Sim(mesh, md, 21)
    sim.set_counts(counts)
    for _ in range(3):
        ref.step(1)
        sim.step(1)
        np.testing.assert_array_equal(sim.get_counts(), ref.counts)
    assert sim.stats().ssa_events == ref.tallies.ssa_events > T * events / 2
    sim.close()
