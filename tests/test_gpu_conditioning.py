"""The mixed path's conditioning test, edge by edge: particles at distances from
wall planes and edge lines just inside and just outside its margins, the number
of edges sent to the FP64 fixup pass against the definition evaluated on the
host.  Lattice coordinates and smoothing lengths are powers of two, so the
projections are exact and the FP32 values the test uses are the rounded ones."""

import numpy as np
import pytest

import oracle
import synth
import paper_2404_17084_amd as em
from test_gpu_degenerate import cube_lattice

pytestmark = pytest.mark.gpu

E = 2.0 ** -20
H = 0.0625


def flagged_edges(x, h, c, cells):
    """Edges of the listed cells that the definition sends to the fixup pass."""
    n = 0
    f32 = np.float32
    for cell in cells:
        for j in range(c.cell_face_off[cell], c.cell_face_off[cell + 1]):
            nrm, cst = c.face_plane[j, :3], c.face_plane[j, 3]
            r0d = abs(cst - nrm @ x) / h
            if not r0d < 2.0:
                continue
            r0 = f32(r0d)
            ids = c.face_vert[c.face_vert_off[j]:c.face_vert_off[j + 1]]
            for k in range(len(ids)):
                v, w = c.verts[ids[k]], c.verts[ids[(k + 1) % len(ids)]]
                e = (w - v) / np.linalg.norm(w - v)
                rho = np.cross(nrm, e) @ (x - v)
                if rho == 0.0:
                    continue
                R02 = f32(abs(rho) / h) * f32(abs(rho) / h)
                c2 = f32(np.float64(r0) * np.float64(r0) + np.float64(R02))  # one rounding, as a fused operation has
                n += bool(R02 < f32(E * E) * c2 or c2 < f32(2.0 ** -60) or abs(r0 - f32(1)) < f32(E)
                          or abs(c2 - f32(1)) < f32(E) or abs(c2 - f32(4)) < f32(4 * E))
    return n


def place(kind, t):
    """A particle at a place where the test turns over, t margins off it."""
    if kind == "wall at h":
        return (0.5 - H * (1 + t * E), 0.3125 + 2.0 ** -9, 0.40625 - 2.0 ** -10)
    if kind == "line at h":   # c^2 = 1 + t E to first order, 0.6 and 0.8 of it along x and y
        s = 1 + 0.5 * t * E
        return (0.5 - 0.59375 * H * s, 0.25 + np.sqrt(1 - 0.59375 ** 2) * H * s, 0.6015625)
    if kind == "line at 2h":
        s = 2 * (1 + 0.5 * t * E)
        return (0.5 - 0.59375 * H * s, 0.25 + np.sqrt(1 - 0.59375 ** 2) * H * s, 0.6484375)
    if kind == "foot on line":  # R0 = t E c for the wall x = 1/2 and the line y = 1/4 on it
        return (0.5 - 0.5 * H, 0.25 + 0.5 * H * t * E, 0.6015625)
    return (0.5 - 0.25 * H * t * E, 0.25 + 0.25 * H * t * E, 0.6015625)  # close to the line: c of some E


@pytest.mark.parametrize("t", [0.5, -0.5, 2.0, -2.0, 6.0, 24.0])
@pytest.mark.parametrize("kind", ["wall at h", "line at h", "line at 2h", "foot on line", "line"])
def test_flagged_edges_are_those_of_the_definition(kind, t):
    print(f"case: {kind}, {t} margins", flush=True)
    c = cube_lattice(4)
    p = synth.Particles(np.array([place(kind, t)], np.float64), np.ones(1), np.array([H]))
    with em.Mapper(device=0, precision=em.MAP_MIXED) as mp:
        r = mp.map(p, c, want_pairs=True)
    assert r["stats"]["n_fixup_terms"] == flagged_edges(p.xyz[0], H, c, r["pair_c"])
    # and the fractions carry the mixed path's error at most
    assert np.abs(r["f"] - oracle.map_particles(p, c)["f"]).max() < 1e-6
