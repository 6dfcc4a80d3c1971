"""Edges of the device kernels: the smallest and largest sizes of each path's
range, remainders of tiles and groups, against the FP64 CPU oracle.

FP64 results are held to the bar of the parity tests (rel-L2 <= 1e-12 against
the oracle FMM of the same tree and order, or the direct sum); the mixed form
to half its accuracy setting against the FP64 result of the same plan.
"""
import numpy as np
import pytest

import workloads as W
from gpu_common import gpu_matvec, log

pytestmark = pytest.mark.gpu


# Target evaluation: coefficient streams of 3, 6 and 21 coefficients (hardly longer
# than the loads that run ahead), the longest, and groups of one and two
# right-hand sides; leaves of 1 to 30 beads, W-list multipoles evaluated.
@pytest.mark.parametrize("p,nrhs", [(1, 1), (1, 4), (2, 5), (5, 3), (27, 1)])
def test_evaluation_streams(orc, p, nrhs):
    w = W.clustered(1201, 6, 10.0, 0.8, 0.05, nrhs, seed=300 + p)
    log(f"evaluation streams p={p} nrhs={nrhs}")
    u, st = gpu_matvec(w.pos, w.forces, w.a, w.eta, 1e-6, order=p, leaf_size=30, w_direct=-1, eval_mode="sets")
    assert st["list_len"]["W"] > 0
    ref = orc.fmm(w.pos, w.forces, w.a, w.eta, p, 30, -1)
    assert orc.rel_l2(u, ref) <= 1e-12


# Interaction lists built by a wave per box, bit-exact against the oracle's:
# leaves of one bead, O lists longer than the sort's LDS buffer (dense beads in
# tiny leaves), a depth cap, and the deepest tree (beads in pairs 2^-19 apart).
def _list_cases():
    g = np.random.default_rng(340)
    pairs = g.uniform(0.0, 1.0, size=(40, 3))
    return [
        ("one-bead-leaves", g.uniform(0.0, 1.0, size=(700, 3)), 1, 14, 0.01),
        ("long-O", g.uniform(0.0, 1.0, size=(2300, 3)), 1, 14, 0.45),
        ("depth-2", g.uniform(0.0, 1.0, size=(3000, 3)), 1, 2, 0.2),
        ("deepest", np.concatenate([pairs, pairs + 2.0**-19]), 1, 21, 1e-6),
    ]


@pytest.mark.parametrize("case", _list_cases(), ids=lambda c: c[0])
def test_lists_bit_exact(orc, case):
    import paper_1711_02976_amd as R
    from gpu_common import to_dev
    name, pos, s, md, a = case
    ref = orc.Tree(pos, s, md, a)
    log(f"lists {name} n={len(pos)} longest O {np.diff(ref.lists['O'][0]).max()}")
    P = R.Plan(to_dev(pos), a, 1.0, 1e-3, leaf_size=s, max_depth=md)
    try:
        got = P.export()
    finally:
        P.free()
    if name == "long-O":
        assert np.diff(ref.lists["O"][0]).max() > 1536
    assert np.array_equal(got["boxes"], ref.boxes)
    for L in "UVWXO":
        assert np.array_equal(got["lists"][L][0], ref.lists[L][0]), L
        assert np.array_equal(got["lists"][L][1], ref.lists[L][1]), L
