"""Face adjacency of the set-up against a dictionary of faces: vertex numbers
with and without gaps (buckets, or one sort of all faces), a hub vertex shared
by every tet (a bucket sorted as a whole), and meshes it refuses."""
import numpy as np
import pytest

from paper_1610_02258_amd import inputs as I
from paper_1610_02258_amd import rdx
from tests.meshes import model

MODEL = model([1e-12, 0.0, 3e-13], [], ["A", "B", "C"])


def _cone(n, apex_first):
    """2 n^2 tets over a triangulated square, all sharing an apex."""
    x, y = np.meshgrid(np.arange(n + 1.0), np.arange(n + 1.0), indexing="ij")
    base = np.stack([x.ravel(), y.ravel(), 0.01 * x.ravel()], 1)
    v = (np.arange(n)[:, None] * (n + 1) + np.arange(n)).ravel()
    tri = np.vstack([np.stack([v, v + 1, v + n + 1], 1), np.stack([v + 1, v + n + 1, v + n + 2], 1)])
    apex = np.array([[n / 2.0, n / 2.0, n + 1.0]])
    verts = np.vstack([apex, base] if apex_first else [base, apex]) * 1e-6
    tri = tri + 1 if apex_first else tri
    top = 0 if apex_first else len(base)
    return verts, np.column_stack([tri, np.full(len(tri), top)]).astype(np.int32)


def _box(seed, gaps):
    m = I.box_mesh(5, 4, 3, 0.5e-6, jitter=0.1, seed=seed).as_dict()
    verts, tets = np.asarray(m["verts"], float), np.asarray(m["tets"])
    rng = np.random.default_rng(seed)
    to = rng.permutation(len(verts) + gaps)[:len(verts)]
    out = np.zeros((len(verts) + gaps, 3))
    out[to] = verts
    return out, to[tets][rng.permutation(len(tets))].astype(np.int32)


def _neighbours(tets):
    seen, nbr = {}, np.full((len(tets), 4), -1, np.int32)
    for i, t in enumerate(tets):
        for k in range(4):
            key = tuple(sorted(np.delete(t, k)))
            if key in seen:
                j, q = seen[key]
                nbr[i, k], nbr[j, q] = j, i
            else:
                seen[key] = (i, k)
    return nbr


@pytest.mark.parametrize("mesh", [_cone(7, True), _cone(7, False), _cone(2, True), _box(1, 0), _box(2, 900),
                                  _box(3, 20000)])
def test_adjacency(mesh):
    verts, tets = mesh
    out = rdx.setup_geometry(dict(verts=verts, tets=tets, region=None), MODEL)
    nbr = _neighbours(tets)
    np.testing.assert_array_equal(out["nbr"], nbr)
    assert ((out["g"] > 0) == (nbr >= 0)).all()
    assert out["tau"] == 1.0 / max(D * G for D in MODEL["D"] for G in out["G"])


@pytest.mark.parametrize("gaps", [0, 20000])
def test_a_face_of_three_tets_is_refused(gaps):
    verts, tets = _box(4, gaps)
    for bad in (np.vstack([tets, tets[:1]]), np.vstack([tets, tets[:1, [1, 0, 2, 3]]])):
        with pytest.raises(rdx.RdxError, match="shared by more than two"):
            rdx.setup_geometry(dict(verts=verts, tets=bad.astype(np.int32), region=None), MODEL)
