"""The octree's one-pass build at its edges: runs of 256 particles and one more
or less, particles in one place (cells that end at the deepest level), leaves of
1 and of 64, against the oracle's tree: node counts, and the set and its order."""

import numpy as np
import pytest

import oracle
import synth
import paper_2404_17084_amd as em

pytestmark = pytest.mark.gpu

BOX = [0.0, 0.0, 0.0, 1.0, 1.0, 1.0]


@pytest.mark.parametrize("leaf", [1, 8, 64])
@pytest.mark.parametrize("n,same", [(1, 0), (8, 0), (9, 0), (64, 64), (65, 65), (255, 0), (256, 30), (257, 100),
                                    (1025, 300), (2048, 0)])
def test_tree_edges(n, same, leaf):
    print(f"case: {n} particles, {same} in one place, leaves of {leaf}", flush=True)
    p, _ = synth.workload("clumps", max(n, 16), 11)
    x, m, h = p.xyz[:n].copy(), p.m[:n].copy(), p.h[:n].copy()
    if same:
        x[n - same:] = x[0]
    src = np.array([[0.4, 0.5, 0.6]])
    with em.Mapper(device=0) as mp:
        G = mp.pseudo(synth.Particles(x, m, h), BOX, src, theta=0.4, r_part=0.05, r_leaf=0.1, leaf_size=leaf)
    O = oracle.pseudo(x, m, h, BOX, src, 0.4, 0.05, 0.1, leaf, 1.1)
    for k in ("kind", "ref"):
        assert np.array_equal(G[k], O[k]), k
    # sums over at most 2048 particles in an order of their own
    for k, o in (("xyz", "xyz"), ("m", "m"), ("size", "s")):
        assert np.abs(np.asarray(G[k]) - np.asarray(O[o])).max() < 1e-12, k
    for k, o in (("n_tree_nodes", "tree_nodes"), ("n_leaves", "leaves"), ("max_level", "max_level")):
        assert G["stats"][k] == O["stats"][o], k
