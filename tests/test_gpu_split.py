"""Pairs shared by four lanes (small jobs) and by one (larger ones): oracle parity
from one pair up to both sides of the two lines (98,304 pairs mixed, 196,608 in
FP64), and the same bits from a second call."""

import numpy as np
import pytest

import oracle
import synth
import paper_2404_17084_amd as em

pytestmark = pytest.mark.gpu

# the bars of the whole-pair kernels: rounding of some hundred terms of order 1 (FP64), FP32 terms (mixed)
PAIR_ABS = {em.MAP_FP64: 1e-12, em.MAP_MIXED: 1e-6}
LINE = {em.MAP_FP64: 196608, em.MAP_MIXED: 98304}


@pytest.mark.parametrize("prec", [em.MAP_FP64, em.MAP_MIXED])
@pytest.mark.parametrize("kind,n", [("uniform", 2), ("clumps", 67), ("uniform", 700),
                                          ("uniform", 1000), ("uniform", 1200), ("uniform", 2000),
                                          ("uniform", 2300)])
def test_pairs_on_both_sides_of_the_line(prec, kind, n):
    print(f"case: {kind} {n}, precision {prec}", flush=True)
    p, c = synth.workload(kind, n, 5)
    o = oracle.map_particles(p, c)
    with em.Mapper(device=0, precision=prec) as mp:
        r = mp.map(p, c, want_pairs=True)
        again = mp.map(p, c, want_pairs=True)
    print(f"  {o['f'].size} pairs, {'split' if o['f'].size <= LINE[prec] else 'whole'}", flush=True)
    assert np.array_equal(r["pair_p"], o["pair_p"]) and np.array_equal(r["pair_c"], o["pair_c"])
    assert np.abs(r["f"] - o["f"]).max() < PAIR_ABS[prec]
    assert np.array_equal(r["f"], again["f"]) and np.array_equal(r["S"], again["S"])
    # the work is the same work: the walls of every pair's cell
    walls = np.diff(c.cell_face_off)[o["pair_c"]].sum()
    assert r["stats"]["n_face_visits"] == walls
