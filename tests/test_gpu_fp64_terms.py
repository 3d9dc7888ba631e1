"""FP64 edge terms over the range of cell size against smoothing length.

A part of an edge can be long or short against h, lie on one side of the foot
point or on both, and meet the inner piece, the shell or only the far field;
which of these occur depends on the ratio of h to the cells.  Every pair is
compared with the oracle's direct form.  Tolerance: a pair sums at most some
400 terms, each formed from values of order one with a few roundings
(400 x 4 x 1.1e-16 = 1.8e-13) and the oracle's own sum rounds as much: 1e-12.
"""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dist", [0, 3])
@pytest.mark.parametrize("scale", [0.02, 0.25, 1.0, 3.0])
def test_fp64_pairs_over_scales(scale, dist):
    import oracle
    import paper_2404_17084_amd as em
    import synth

    p, c = synth.workload("clumps", 333, 7)
    q = synth.Particles(p.xyz, p.m, p.h * scale)
    ref = oracle.map_particles(q, c)
    with em.Mapper(device=0, precision=em.MAP_FP64) as mp:
        em.map_set_tune(mp.ctx, em.MAP_FP64, waves=0 if dist == 0 else 3, persistent=dist)
        r = mp.map(q, c, want_pairs=True)
    assert np.array_equal(r["pair_p"], ref["pair_p"]) and np.array_equal(r["pair_c"], ref["pair_c"])
    assert np.abs(r["f"] - ref["f"]).max() < 1e-12
    assert abs(r["M"].sum() - p.m.sum()) < 1e-12


@pytest.mark.parametrize("dist", [0, 3])
@pytest.mark.parametrize("h", [1e-3, 1e-30, 1e-76, 1e-78, 1e-90, 1e-120, 1e-150])
def test_cells_far_larger_than_the_support(h, dist):
    """Particles on the wall between two half boxes, edges up to 1e150 h away: each half holds half of them, whatever
    the smoothing length.  (Lengths square to 1e300 h^2 at most.)"""
    import paper_2404_17084_amd as em
    import synth

    c = synth.voronoi_cells(np.array([[0.25, 0.5, 0.5], [0.75, 0.5, 0.5]]))
    p = synth.Particles(np.array([[0.5, 0.5, 0.5], [0.5, 0.3, 0.7]]), np.array([0.5, 0.5]), np.full(2, h))
    with em.Mapper(device=0, precision=em.MAP_FP64) as mp:
        em.map_set_tune(mp.ctx, em.MAP_FP64, waves=0 if dist == 0 else 3, persistent=dist)
        r = mp.map(p, c, want_pairs=True)
    assert np.abs(r["f"] - 0.5).max() < 1e-12 and r["f"].size == 4
    assert np.abs(r["M"] - 0.5).max() < 1e-12
