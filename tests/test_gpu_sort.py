"""The key sort on both sides of its lines (counting up to 32,768 keys; 4, 8 and
16 items per thread up to 524,288, 1,048,576 and more; a tile's last items), seen
through a walk that extracts every particle: the set is the particles in Morton
order, ties by index."""

import numpy as np
import pytest

import synth
import paper_2404_17084_amd as em

pytestmark = pytest.mark.gpu


def morton(x):
    q = np.clip(np.floor(x * 2097152.0), 0, 2097151).astype(np.uint64)

    def spread(v):
        for s, m in ((32, 0x1f00000000ffff), (16, 0x1f0000ff0000ff), (8, 0x100f00f00f00f00f), (4, 0x10c30c30c30c30c3),
                     (2, 0x1249249249249249)):
            v = (v | (v << np.uint64(s))) & np.uint64(m)
        return v

    return (spread(q[:, 0]) << np.uint64(2)) | (spread(q[:, 1]) << np.uint64(1)) | spread(q[:, 2])


@pytest.mark.parametrize("n", [2, 64, 65, 32767, 32768, 32769, 33793, 524288, 524289, 1048576, 1048577, 1052673])
def test_particles_in_morton_order(n):
    print(f"case: {n} particles", flush=True)
    rng = np.random.default_rng(n)
    x = rng.random((n, 3))
    x[n // 2:n // 2 + n // 8] = x[:n // 8]      # pairs of equal keys, far apart in the list
    x[n - n // 16:] = x[n - 1]                  # and many in one place
    p = synth.Particles(x, np.full(n, 1.0 / n), np.full(n, 0.01))
    with em.Mapper(device=0) as mp:
        G = mp.pseudo(p, [0.0, 0.0, 0.0, 1.0, 1.0, 1.0], [[0.5, 0.5, 0.5]], theta=0.5, r_part=10.0, r_leaf=10.0,
                      leaf_size=64)
    assert G["stats"]["n_particles"] == n
    assert np.array_equal(G["ref"], np.argsort(morton(x), kind="stable"))
