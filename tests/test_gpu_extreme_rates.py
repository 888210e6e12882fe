"""Rate constants at the end of the double range, which the model checks accept:
propensities in the last binade (whose power-of-two bound is not finite) and
infinite ones, alone and beside ordinary reactions, against the oracle bit for
bit.  Every reaction uses its reactants up, so that a window ends."""
import numpy as np
import pytest

from paper_1610_02258_amd import inputs as I

HUGE = 1.7e308


def _model(S, R, ks):
    """X_s -> X_S-1 for the first species (s < S - 1), reaction r at ks[r % len(ks)], a species' second one at 1/s."""
    lhs, rhs = np.zeros((R, S), np.int32), np.zeros((R, S), np.int32)
    for r in range(R):
        lhs[r, r % (S - 1)], rhs[r, S - 1] = 1, 1
    return dict(D=np.full(S, 1e-12), lhs=lhs, rhs=rhs, kcst=np.array([[ks[r % len(ks)] if r < S - 1 else 1.0 for r in range(R)]]))


@pytest.mark.gpu
@pytest.mark.parametrize("ks", [[HUGE], [1e308], [HUGE, 1.0], [1e308, 1e300, 1e3], [1.0, HUGE, 1e308, 1e-3, 0.0]])
@pytest.mark.parametrize("S,R", [(3, 4), (5, 8), (9, 12), (15, 24), (16, 32)])
def test_extreme_rates_match_oracle(oracle_lib, S, R, ks):
    from paper_1610_02258_amd import rdx
    mesh = I.box_mesh(3, 2, 4, 1e-6, jitter=0.1, seed=S).as_dict()
    T = len(mesh["tets"])
    md = _model(S, R, ks)
    counts = np.random.default_rng(S + R).integers(0, 4, (S, T)).astype(np.int32)
    print(f"case: S={S} R={R} rates {ks}", flush=True)
    ref = oracle_lib.Instance(mesh, md, 11)
    ref.reset(counts)
    ref.step(3)
    sim = rdx.Sim(mesh, md, 11)
    sim.set_counts(counts)
    sim.step(3)
    np.testing.assert_array_equal(sim.get_counts(), ref.counts)
    st = sim.stats()
    assert (st.ssa_events, st.moves) == (ref.tallies.ssa_events, ref.tallies.moves)
    assert st.ssa_events > 0
    sim.close()


@pytest.mark.gpu
@pytest.mark.parametrize("S,R", [(3, 4), (5, 8), (9, 12), (16, 24)])
def test_rates_whose_sum_overflows_match_oracle(oracle_lib, S, R):
    """Two reactions of one species whose constants add up to infinity, in tets
    that do not hold it: their other reactions have their events all the same."""
    from paper_1610_02258_amd import rdx
    mesh = I.box_mesh(3, 2, 4, 1e-6, jitter=0.1, seed=S).as_dict()
    T = len(mesh["tets"])
    md = _model(S, R, [1.0])
    md["lhs"][:2], md["rhs"][:2], md["kcst"][0, :2] = 0, 0, HUGE
    md["lhs"][:2, 0], md["rhs"][:2, S - 1] = 1, 1
    md["kcst"][0, 2:] = 0.5 / oracle_lib.Instance(mesh, md, 5).tau
    counts = np.random.default_rng(S + R).integers(0, 4, (S, T)).astype(np.int32)
    counts[0] = 0
    print(f"case: S={S} R={R}", flush=True)
    ref = oracle_lib.Instance(mesh, md, 5)
    ref.reset(counts)
    ref.step(2)
    assert ref.tallies.ssa_events > 0
    sim = rdx.Sim(mesh, md, 5)
    sim.set_counts(counts)
    sim.step(2)
    np.testing.assert_array_equal(sim.get_counts(), ref.counts)
    sim.close()
