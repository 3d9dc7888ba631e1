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


@pytest.mark.parametrize("precision", ["fp64", "mixed"])
@pytest.mark.parametrize("dist", [0, 3])
def test_particles_next_to_an_edge(precision, dist):
    """Particles beside the common edge of four cells, down to distances whose squares, or that themselves, are near
    the smallest doubles: each cell holds a quarter (to the distance), and a particle on a wall plane beside the edge
    as much as one off it.  1e-12 as above; mixed 1e-6, some 40 FP32 terms of order one."""
    import paper_2404_17084_amd as em
    import synth

    c = synth.voronoi_cells(np.array([[x, y, 0.0] for x in (-.25, .25) for y in (-.25, .25)]),
                            (-.5, -.5, -.5, .5, .5, .5))
    prec = em.MAP_FP64 if precision == "fp64" else em.MAP_MIXED
    e = [0.0, 1e-20, 1e-100, 1e-146, 1e-170, 1e-250, 1e-280, 1e-290, 1e-300, 1e-310]
    xyz = np.array([[a, b, z] for a in e for b in e for z in (0.0, 0.1)])
    n = len(xyz)
    p = synth.Particles(xyz, np.full(n, 1.0 / n), np.full(n, 0.1))
    with em.Mapper(device=0, precision=prec) as mp:
        em.map_set_tune(mp.ctx, prec, waves=0 if dist == 0 else (3 if precision == "fp64" else 6), persistent=dist)
        r = mp.map(p, c, want_pairs=True)
    assert r["f"].size == 4 * n
    assert np.abs(r["f"] - 0.25).max() < (1e-12 if precision == "fp64" else 1e-6)
