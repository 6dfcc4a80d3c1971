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
