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


@pytest.mark.parametrize("walls", [16, 48])
@pytest.mark.parametrize("scale", [2.0 ** -100, 2.0 ** -80, 1.0, 2.0 ** 66, 2.0 ** 70, 2.0 ** 200])
def test_pair_set_in_other_units(scale, walls):
    """Lengths times a power of two, which is exact: the pairs are those of the unit box, also where squared lengths
    leave FP32's range.  One cell among `walls` others on a sphere about it: fewer walls than the test stages in LDS
    (40), and more."""
    import oracle
    import paper_2404_17084_amd as em
    import synth

    k = np.arange(walls) + 0.5
    ph, th = np.arccos(1 - 2 * k / walls), np.pi * (1 + 5 ** 0.5) * k
    s = 0.5 + 0.25 * np.stack([np.cos(th) * np.sin(ph), np.sin(th) * np.sin(ph), np.cos(ph)], 1)
    s = np.concatenate([[[0.5, 0.5, 0.5]], s + 1e-3 * np.random.default_rng(1).standard_normal(s.shape)])
    c = synth.voronoi_cells(s)
    assert np.diff(c.cell_face_off).max() == walls
    x = np.random.default_rng(2).random((3000, 3))
    p = synth.Particles(x, np.full(3000, 1 / 3000.0), np.full(3000, 0.03))
    ref = oracle.map_particles(p, c)
    q = synth.Particles(x * scale, p.m, p.h * scale)
    cs = synth.Cells(c.cell_face_off, c.face_vert_off, c.face_vert, c.face_plane * np.array([1.0, 1.0, 1.0, scale]),
                     c.face_nb, c.verts * scale, c.cell_volume * scale ** 3, tuple(scale * np.array(synth.BOX)))
    with em.Mapper(device=0) as mp:
        pp, pc = mp.pairs(q, cs)
    assert np.array_equal(pp, ref["pair_p"]) and np.array_equal(pc, ref["pair_c"])


@pytest.mark.parametrize("h", [1e-6, 1e-14, 1e-18, 1e-30])
def test_particles_on_the_vertices(h):
    """Particles on the cells' own vertices, supports down to far below the rounding of the cells' coordinates: the
    ball about a cell ends at its farthest vertex, whose particle must not be dropped for the rounding of its
    distance.  Pairs of a particle with the cell whose vertex it is on, as the oracle's test of all pairs has them."""
    import oracle
    import paper_2404_17084_amd as em
    import synth

    c = synth.voronoi_cells(np.random.default_rng(8).random((200, 3)))
    own = np.full(c.n_verts, -1)
    for i in range(c.n_cells):
        a, b = c.face_vert_off[c.cell_face_off[i]], c.face_vert_off[c.cell_face_off[i + 1]]
        own[c.face_vert[a:b]] = i
    n = c.n_verts
    p = synth.Particles(c.verts.copy(), np.full(n, 1.0 / n), np.full(n, h))
    pp, pc = oracle.pairs(p.xyz, p.h, c, brute=True)
    want = set(pp[own[pp] == pc].tolist())
    with em.Mapper(device=0) as mp:
        gp, gc = mp.pairs(p, c)
    got = set(gp[own[gp] == gc].tolist())
    assert len(want) > n // 4 and want - got == set()


@pytest.mark.parametrize("precision", ["fp64", "mixed", "table"])
def test_mapping_in_other_units(precision):
    """A whole mapping with lengths times a power of two: the same bits of the masses and of S_a."""
    import paper_2404_17084_amd as em
    import synth

    prec = {"fp64": em.MAP_FP64, "mixed": em.MAP_MIXED, "table": em.MAP_TABLE}[precision]
    p, c = synth.workload("clumps", 1000, 5)
    with em.Mapper(device=0, precision=prec) as mp:
        ref = mp.map(p, c)
        for scale in (2.0 ** -80, 2.0 ** 70, 2.0 ** 200):
            cs = synth.Cells(c.cell_face_off, c.face_vert_off, c.face_vert,
                             c.face_plane * np.array([1.0, 1.0, 1.0, scale]), c.face_nb, c.verts * scale,
                             c.cell_volume * scale ** 3, tuple(scale * np.array(synth.BOX)))
            r = mp.map(synth.Particles(p.xyz * scale, p.m, p.h * scale), cs)
            assert np.array_equal(r["M"], ref["M"]) and np.array_equal(r["S"], ref["S"])
