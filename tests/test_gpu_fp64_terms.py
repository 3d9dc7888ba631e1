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
