"""Pair search: the pair set at the edges of its tree walk.

The walk starts from at most 64 nodes, expands two levels at a time, takes the
particles of 8 leaves of 8 at once for 4 cells of a wavefront and keeps 512
candidates per cell before a second walk.  Sizes about those numbers, stored in
Morton order and shuffled (a wavefront's cells then lie far apart), with
supports from a fraction of a cell to the whole box; pair sets are compared
with the oracle's bit for bit.
"""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("order", ["morton", "shuffled"])
@pytest.mark.parametrize("n,scale", [(1, 1.0), (2, 1.0), (3, 0.1), (9, 1.0), (63, 1.0), (257, 0.05), (513, 1.0),
                                     (1025, 4.0), (4097, 1.0)])
def test_pair_set(n, scale, order):
    import oracle
    import paper_2404_17084_amd as em
    import synth

    p, c = synth.workload("uniform", n, 40 + n)
    xyz, m, h = p.xyz, p.m, p.h * scale
    if order == "shuffled":
        rng = np.random.default_rng(n)
        k = rng.permutation(n)
        xyz, m, h = np.ascontiguousarray(xyz[k]), m[k], np.ascontiguousarray(h[k])
        c = synth.cells_subset(c, rng.permutation(n))
    q = synth.Particles(xyz, m, h)
    ref = oracle.map_particles(q, c)
    with em.Mapper(device=0) as mp:
        pp, pc = mp.pairs(q, c)
    assert np.array_equal(pp, ref["pair_p"]) and np.array_equal(pc, ref["pair_c"])
