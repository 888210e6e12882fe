"""A count that passes 2^31 within one window (two neighbours of 2^30 molecules
each empty into one tet) is reported as an overflow, and not dropped."""
import numpy as np
import pytest

from tests.meshes import stars


@pytest.mark.gpu
@pytest.mark.parametrize("S", [1, 6, 12, 16])
@pytest.mark.parametrize("senders", [2, 3])
def test_a_wrapped_count_is_an_overflow(S, senders):
    from paper_1610_02258_amd import rdx
    mesh = stars(3)
    none = np.zeros((0, S), np.int32)
    md = dict(D=np.full(S, 1e-12), lhs=none, rhs=none, kcst=np.zeros((1, 0)))
    counts = np.zeros((S, len(mesh["tets"])), np.int32)
    counts[S - 1, 6:6 + senders] = 1 << 30  # neighbours of the second star's centre, tet 5
    sim = rdx.Sim(mesh, md, 3, tau_override=1.0)  # every molecule leaves in a window
    sim.set_counts(counts)
    print(f"case: S={S} senders {senders}", flush=True)
    sim.step(2)
    with pytest.raises(rdx.RdxError) as e:
        sim.sync()
    assert e.value.status == -5
    sim.close()
