"""The window kernel's tile passes against the oracle, bit for bit: each of
its instances (groups of 4, 8 and 16 lanes per listed tet, the largest tables
of an instance and tables that fill it partly), ragged last tiles, tiles where
one, some or all tets are listed (more changed items than are held at a time),
items of one call and of every class up to binomial ones, counts too large for
an item's packed field, tets without a neighbour, immobile species and two
regions; plain launches mixed with graphs of odd length, static and claimed
tiles."""
import numpy as np
import pytest

from paper_1610_02258_amd import inputs as I
from tests.randmodels import random_counts, random_model

pytestmark = pytest.mark.gpu


def _mesh(nx, ny, nz, n_regions, seed):
    """A box and, apart from it, three tets without a neighbour (in the ragged
    last tile)."""
    m = I.box_mesh(nx, ny, nz, 0.5e-6, jitter=0.1, seed=seed).as_dict()
    verts, tets = np.asarray(m["verts"], float), np.asarray(m["tets"], np.int32)
    one = verts[tets[0]] - verts[tets[0]].min(0)
    for k in range(3):
        tets = np.vstack([tets, np.arange(4, dtype=np.int32) + len(verts)])
        verts = np.vstack([verts, one + np.array([1e-3 + 1e-5 * k, 0, 0])])
    reg = np.random.default_rng(seed).integers(0, n_regions, len(tets)).astype(np.uint8)
    return dict(verts=verts, tets=tets, region=reg if n_regions > 1 else None)


@pytest.mark.parametrize("mean", [0.4, 3.0, 12.0, 60.0])
@pytest.mark.parametrize("S,R,box", [(1, 1, (1, 1, 1)), (4, 4, (4, 4, 2)), (3, 5, (5, 3, 4)), (8, 8, (3, 3, 7)),
                                     (9, 3, (4, 3, 3)), (12, 12, (4, 4, 3)), (2, 13, (3, 5, 3)), (16, 24, (3, 4, 4)),
                                     (15, 32, (5, 4, 2))])
def test_tiles_match_oracle(oracle_lib, S, R, box, mean):
    from paper_1610_02258_amd import rdx
    rng = np.random.default_rng(int(1000 * S + 10 * R + mean))
    mesh = _mesh(*box, 2, seed=S + R)
    T = len(mesh["tets"])
    md = random_model(rng, S, R, 2)
    counts = random_counts(rng, S, T, mean)
    # a few events per tet and window, whatever the time step
    md["kcst"] *= 3e-4 / oracle_lib.Instance(mesh, md, 77).tau
    md["kcst"][:, md["lhs"].sum(1) == 0] *= 0.01
    if mean == 60.0:  # below, at and above the packed field's end, in a species nothing consumes
        md["kcst"][:, md["lhs"][:, 0] > 0] = 0.0
        counts[0, [0, T // 2, T - 1]] = [(1 << 22) - 1, 1 << 22, 5_000_001]
    print(f"case: T={T} S={S} R={R} mean {mean}", flush=True)
    ref = oracle_lib.Instance(mesh, md, 77)
    ref.reset(counts)
    n = (1, 5, 3)
    want = []
    for k in n:
        ref.step(k)
        want.append(ref.counts.copy())
    for graph, claim in ((1, 0), (3, 0), (2, 1)):
        print(f"  graph_windows {graph} tile_claim {claim}", flush=True)
        sim = rdx.Sim(mesh, md, 77)
        sim.set_exec_options(graph_windows=graph, tile_claim=claim)
        sim.set_counts(counts)
        for k, w in zip(n, want):
            sim.step(k)
            np.testing.assert_array_equal(sim.get_counts(), w)
        st = sim.stats()
        assert (st.ssa_events, st.moves, st.face_moves) == (ref.tallies.ssa_events, ref.tallies.moves,
                                                            ref.tallies.face_moves)
        sim.close()


@pytest.mark.parametrize("claim", [0, 1])
@pytest.mark.parametrize("box", [(15, 15, 15), (20, 20, 15)])
def test_tile_widths_match_oracle(oracle_lib, box, claim):
    """Runs of 317 and 563 tiles on a quarter of the resident blocks, where
    tiles of 32 and of 64 tets are taken (the small runs above take 16)."""
    from paper_1610_02258_amd import rdx
    rng = np.random.default_rng(sum(box))
    mesh = _mesh(*box, 2, seed=3)
    T = len(mesh["tets"])
    md = random_model(rng, 3, 5, 2)
    md["kcst"] *= 3e-4 / oracle_lib.Instance(mesh, md, 5).tau
    md["kcst"][:, md["lhs"].sum(1) == 0] *= 0.01
    counts = random_counts(rng, 3, T, 3.0)
    print(f"case: T={T} tile_claim {claim}", flush=True)
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
