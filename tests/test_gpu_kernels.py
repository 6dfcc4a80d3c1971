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


# Near-field tiles split over several blocks (few tiles, or one list much
# longer than the others): one bead, tiles of 1, 127, 128 and 129 beads, a leaf
# of several chunks, on the vector units and the matrix cores; one leaf, so the
# matvec is the direct sum and the far field is empty.
@pytest.mark.parametrize("n,nrhs", [(1, 1), (127, 2), (128, 1), (129, 4), (1025, 1), (2500, 17), (2500, 8)])
def test_split_single_leaf_is_direct(orc, n, nrhs):
    w = W.uniform_cube(n, 1.0, 0.03, nrhs=nrhs, seed=310 + n)
    log(f"split single leaf n={n} nrhs={nrhs}")
    u, st = gpu_matvec(w.pos, w.forces, w.a, w.eta, 1e-6, leaf_size=10_000)
    assert st["nleaf"] == 1
    ref = orc.rpy_direct(w.pos, w.forces, w.a, w.eta)
    assert orc.rel_l2(u, ref) <= 1e-12
    um, _ = gpu_matvec(w.pos, w.forces, w.a, w.eta, 1e-6, leaf_size=10_000, precision="mixed")
    assert orc.rel_l2(um, u) <= 5e-7


# Split U, W and O lists together: clustered beads in leaves of up to 300, with
# overlapping pairs outside U; the W boxes summed directly.
@pytest.mark.parametrize("nrhs", [1, 3, 18])
def test_split_adaptive_lists(orc, nrhs):
    w = W.clustered(9000, 4, 12.0, 0.6, 0.3, nrhs, seed=320)
    log(f"split adaptive lists nrhs={nrhs}")
    u, st = gpu_matvec(w.pos, w.forces, w.a, w.eta, 1e-6, leaf_size=300, order=6, w_direct=10**6)
    assert st["list_len"]["W"] > 0 and st["list_len"]["O"] > 0
    ref = orc.fmm(w.pos, w.forces, w.a, w.eta, 6, 300, 10**6)
    assert orc.rel_l2(u, ref) <= 1e-12


# An empty far field: two leaves next to each other (no V, W or X entries),
# and an injected error is still reported at a far-field phase.
def test_empty_far_field(orc):
    import paper_1711_02976_amd as R
    from gpu_common import to_dev
    w = W.uniform_cube(400, 1.0, 0.02, nrhs=5, seed=330)
    log("empty far field n=400")
    P = R.Plan(to_dev(w.pos), w.a, w.eta, 1e-6, leaf_size=100)
    try:
        st = P.stats()
        assert st["nleaf"] > 1 and st["list_len"]["V"] == 0 and st["list_len"]["X"] == 0
        u = P.matvec(to_dev(w.forces)).cpu().numpy()
        assert orc.rel_l2(u, orc.rpy_direct(w.pos, w.forces, w.a, w.eta)) <= 1e-12
        P.inject_error("eval")
        with pytest.raises(R.RpyError):
            P.matvec(to_dev(w.forces))
    finally:
        P.free()


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


# M->L at the edges of its kernels' order ranges in both precisions, one, two
# and four right-hand sides per pass, V lists that fill batches of 64, 32 and
# 16 columns unevenly; the FP64 form against the oracle FMM, the mixed form
# against the FP64 one.
@pytest.mark.parametrize("p,nrhs", [(10, 3), (11, 1), (16, 4), (17, 2), (21, 1), (21, 4), (22, 1), (27, 2)])
def test_m2l_order_ranges(orc, p, nrhs):
    for w in (W.uniform_cube(3000, 1.0, 0.005, nrhs=nrhs, seed=350), W.clustered(2500, 8, 10.0, 0.8, 0.05, nrhs, seed=351)):
        log(f"M->L p={p} nrhs={nrhs} {w.name}")
        kw = dict(order=p, leaf_size=40, w_direct=(p + 1) * (p + 2))
        u, st = gpu_matvec(w.pos, w.forces, w.a, w.eta, 1e-6, **kw)
        assert st["list_len"]["V"] > 0
        ref = orc.fmm(w.pos, w.forces, w.a, w.eta, p, 40, (p + 1) * (p + 2))
        assert orc.rel_l2(u, ref) <= 1e-12
        um, _ = gpu_matvec(w.pos, w.forces, w.a, w.eta, 1e-6, precision="mixed", **kw)
        assert orc.rel_l2(um, u) <= 5e-7


# Matrix-core P2P staging: source chunks of 1, 3, 125..129 and 256 beads and
# every number of vector-unit right-hand sides in the same launch.
@pytest.mark.parametrize("n,nrhs", [(17, 16), (131, 17), (253, 18), (129, 20), (257, 24), (384, 16)])
def test_matrix_core_staging(orc, n, nrhs):
    w = W.uniform_cube(n, 1.0, 0.05, nrhs=nrhs, seed=360 + n)
    log(f"matrix-core staging n={n} nrhs={nrhs}")
    u, st = gpu_matvec(w.pos, w.forces, w.a, w.eta, 1e-6, leaf_size=10_000)
    assert orc.rel_l2(u, orc.rpy_direct(w.pos, w.forces, w.a, w.eta)) <= 1e-12
    um, _ = gpu_matvec(w.pos, w.forces, w.a, w.eta, 1e-6, leaf_size=10_000, precision="mixed")
    assert orc.rel_l2(um, u) <= 5e-7


# Small far fields: S->M, S->L, M->M, L->L and the evaluation cut into finer work
# items, with one, two and five right-hand sides (groups of 4 + 1), in both
# evaluation forms and at orders whose polynomials have no room for the M->M
# shares; an adaptive tree with leaves of many chunks, and a full one of 64 leaves.
_SMALL = [(1, 1), (3, 2), (4, 5), (5, 1), (16, 2)]


@pytest.mark.parametrize("p,nrhs,mode", [(p, q, m) for m in ("sets", "poly") for p, q in _SMALL] +
                         [(22, 1, "sets"), (23, 5, "sets")])  # polynomials end at order 21
def test_small_far_field(orc, p, nrhs, mode):
    for w, leaf in ((W.clustered(4000, 5, 12.0, 0.5, 0.02, nrhs, seed=350 + p), 700),
                    (W.uniform_cube(5000, 1.0, 0.01, nrhs=nrhs, seed=351 + p), 150)):
        log(f"small far field p={p} nrhs={nrhs} {mode} leaf={leaf}")
        u, st = gpu_matvec(w.pos, w.forces, w.a, w.eta, 1e-6, order=p, leaf_size=leaf, eval_mode=mode)
        ref = orc.fmm(w.pos, w.forces, w.a, w.eta, p, leaf, st["w_direct"])
        assert orc.rel_l2(u, ref) <= 1e-12


# Lanczos vectors scaled on the device: right-hand sides that end at different
# steps (a general one, zero, an eigenvector of D, whose next vector is rounding
# noise) in one call, one bead, and a vector of just over two chunks of the dot
# products.
@pytest.mark.parametrize("n", [1, 60, 683])
def test_lanczos_mixed_ends(orc, n):
    import paper_1711_02976_amd as R
    from gpu_common import to_dev
    g = np.random.default_rng(360 + n)
    pos = g.uniform(0.0, 20.0, size=(n, 3))
    z = g.standard_normal((3, n, 3))
    z[1] = 0.0
    if n == 60:
        D = orc.rpy_direct(pos, np.eye(3 * n).reshape(3 * n, n, 3), 0.4, 1.0).reshape(3 * n, 3 * n)
        z[2] = np.linalg.eigh(0.5 * (D + D.T))[1][:, 7].reshape(n, 3)
    log(f"lanczos mixed ends n={n}")
    P = R.Plan(to_dev(pos), 0.4, 1.0, 1e-6, leaf_size=1000)
    try:
        y, info = P.sqrt_matvec(to_dev(z), tol=1e-11, max_iter=100)
        y = y.cpu().numpy()
    finally:
        P.free()
    ref = orc.rpy_sqrt(pos, z, 0.4, 1.0)
    assert info["converged"] and np.all(y[1] == 0.0)
    for r in (0, 2):
        assert orc.rel_l2(y[r], ref[r]) <= 1e-9


# Dot products over more chunks than a wave has lanes: D^{1/2} twice is D, to
# the plan's accuracy (its matvec is symmetric to 1e-6).
def test_lanczos_many_chunks(orc):
    import paper_1711_02976_amd as R
    from gpu_common import to_dev
    w = W.uniform_cube(45000, 1.0, 0.0005, nrhs=1, seed=370)  # 45 steps; of radius .004, over 100
    log("lanczos many chunks n=45000")
    P = R.Plan(to_dev(w.pos), w.a, w.eta, 1e-6)
    try:
        y, _ = P.sqrt_matvec(to_dev(w.forces), tol=1e-9, max_iter=100)
        y, info = P.sqrt_matvec(y, tol=1e-9, max_iter=100)
        u = P.matvec(to_dev(w.forces))
        assert info["converged"]
        assert orc.rel_l2(y.cpu().numpy(), u.cpu().numpy()) <= 1e-5
    finally:
        P.free()


# Memory, streams and host pages kept between plans: plans of several sizes made,
# used and freed by two threads on streams of their own, blocks of one reused by
# the other, give what a plan on its own gives, bit for bit.
def test_plans_share_kept_memory():
    import threading

    import paper_1711_02976_amd as R
    import torch
    from gpu_common import to_dev
    log("kept memory: two threads, two streams")
    work = []
    for i, (n, nrhs, leaf) in enumerate([(300, 1, 40), (5000, 3, 60), (20000, 1, 0), (900, 2, 25)]):
        w = W.clustered(n, 4, 12.0, 0.7, 0.05, nrhs, seed=380 + i)
        work.append((to_dev(w.pos), to_dev(w.forces), w.a, w.eta, leaf))

    def one(c, stream):
        pos, F, a, eta, leaf = c
        P = R.Plan(pos, a, eta, 1e-6, leaf_size=leaf, stream=stream.cuda_stream)
        try:
            return P.matvec(F).clone()
        finally:
            P.free()

    torch.cuda.synchronize()
    ref = [one(c, torch.cuda.current_stream()) for c in work]
    torch.cuda.synchronize()
    bad = []

    def run(k):
        st = torch.cuda.Stream()
        with torch.cuda.stream(st):
            for it in range(6):
                i = (it * (k + 1) + k) % len(work)
                got = one(work[i], st)
                st.synchronize()
                if not torch.equal(got, ref[i]):
                    bad.append((k, it, i))

    ts = [threading.Thread(target=run, args=(k,)) for k in range(2)]
    for t in ts:
        t.start()
    for t in ts:
        t.join()
    assert not bad


# Plans without a far field in two launches, forces read and velocities written
# in the caller's order: systems of 0 to 1,300 beads side by side, every group of
# right-hand sides, the velocities written over the forces, and many small
# systems (one part per block, then more blocks than are taken at all).
@pytest.mark.parametrize("counts,nrhs", [([5, 0, 130, 1300], 1), ([64, 700], 7), ([1, 129, 33], 11),
                                         ([7] * 1500, 2), ([3] * 2500, 1)])
@pytest.mark.parametrize("precision", ["fp64", "mixed"])
def test_direct_plans(orc, counts, nrhs, precision):
    import paper_1711_02976_amd as R
    from gpu_common import to_dev
    n = sum(counts)
    w = W.uniform_cube(n, 1.0, 0.02, nrhs=nrhs, seed=390 + n)
    log(f"direct plans {len(counts)} systems n={n} nrhs={nrhs} {precision}")
    P = R.Plan(to_dev(w.pos), w.a, w.eta, 1e-6, leaf_size=10_000, counts=counts, precision=precision)
    try:
        F = to_dev(w.forces)
        u = P.matvec(F).cpu().numpy()
        R.rpy_matvec(P.handle, nrhs, F.data_ptr(), F.data_ptr())
        over = F.cpu().numpy()
    finally:
        P.free()
    assert np.array_equal(over, u)
    ref, at = np.empty_like(u), 0
    for c in counts:
        if c:
            ref[:, at:at + c] = orc.rpy_direct(w.pos[at:at + c], w.forces[:, at:at + c], w.a, w.eta)
        at += c
    assert orc.rel_l2(u, ref) <= (1e-12 if precision == "fp64" else 5e-7)


# A captured matvec replayed with eager work in between equals the eager result
# each time: direct launches, and split phases of a small adaptive tree.
@pytest.mark.parametrize("n,leaf,nrhs", [(700, 1000, 2), (4000, 300, 3)])
def test_captured_matvec(n, leaf, nrhs):
    import paper_1711_02976_amd as R
    import torch
    from gpu_common import to_dev
    w = W.clustered(n, 4, 12.0, 0.6, 0.05, nrhs, seed=395)
    log(f"captured matvec n={n} leaf={leaf} nrhs={nrhs}")
    st = torch.cuda.Stream()
    with torch.cuda.stream(st):
        P = R.Plan(to_dev(w.pos), w.a, w.eta, 1e-6, leaf_size=leaf, stream=st.cuda_stream)
        F = to_dev(w.forces)
        ref = P.matvec(F).clone()
    torch.cuda.synchronize()
    try:
        g = torch.cuda.CUDAGraph()
        with torch.cuda.graph(g, stream=st):
            out = P.matvec(F)
        for it in range(4):
            g.replay()
            torch.cuda.synchronize()
            assert torch.equal(out, ref)
            out.zero_()
            with torch.cuda.stream(st):
                assert torch.equal(P.matvec(F), ref)
            torch.cuda.synchronize()
    finally:
        P.free()


# Non-finite forces stay where they belong: a call with NaN and infinite forces
# leaves nothing behind for the plan's next calls (wider passes first, whose
# charges lie where narrower ones have their rows past the last bead), reaches no
# other right-hand side of its call and no other system of its plan.  Leaves of
# odd sizes on adaptive trees: S->M and S->L on the vector units and the matrix
# cores, the allocating and the allocation-free call.
def _poison(F):
    F = F.copy()
    F[..., 0] = np.nan
    F[..., 1] = np.inf
    return F


@pytest.mark.parametrize("noalloc", [False, True])
def test_nonfinite_forces_leave_nothing_behind(noalloc):
    import paper_1711_02976_amd as R
    import torch
    from gpu_common import to_dev
    w = W.clustered(3001, 5, 12.0, 0.6, 0.05, 4, seed=400)
    log(f"non-finite forces, later calls, noalloc={noalloc}")
    kw = dict(leaf_size=37, order=8, w_direct=20, eval_mode="sets")

    def call(P, F):
        U = torch.full_like(F, float("nan"))
        (R.rpy_matvec_noalloc if noalloc else R.rpy_matvec)(P.handle, F.shape[0], F.data_ptr(), U.data_ptr())
        return U.cpu().numpy()

    F, bad = to_dev(w.forces), to_dev(_poison(w.forces))
    P, Q = (R.Plan(to_dev(w.pos), w.a, w.eta, 1e-6, **kw) for _ in range(2))
    try:
        assert P.stats()["list_len"]["X"] > 0
        call(Q, F)  # the workspace of four right-hand sides, as P's
        ref = {k: call(Q, F[:k].contiguous()) for k in (1, 2, 3, 4)}
        assert all(np.isfinite(r).all() for r in ref.values())
        for k in (1, 2, 3, 4):
            call(P, bad)
            assert np.array_equal(call(P, F[:k].contiguous()), ref[k]), k
        mix = F[:3].clone()
        mix[:2] = bad[:2]  # a pass of two, then the third right-hand side alone
        assert np.array_equal(call(P, mix)[2], ref[3][2])
    finally:
        P.free()
        Q.free()


@pytest.mark.parametrize("nrhs", [1, 2, 4])
def test_nonfinite_forces_stay_in_their_system(nrhs):
    import paper_1711_02976_amd as R
    from gpu_common import to_dev
    counts = [1501, 1499]
    w = W.clustered(sum(counts), 5, 12.0, 0.6, 0.05, nrhs, seed=401)
    log(f"non-finite forces, other systems, nrhs={nrhs}")
    P = R.Plan(to_dev(w.pos), w.a, w.eta, 1e-6, leaf_size=37, order=8, counts=counts, eval_mode="sets")
    try:
        ref = P.matvec(to_dev(w.forces)).cpu().numpy()
        F = w.forces.copy()
        F[:, counts[0]:] = _poison(F[:, counts[0]:])
        u = P.matvec(to_dev(F)).cpu().numpy()
        assert np.isfinite(ref).all() and np.array_equal(u[:, :counts[0]], ref[:, :counts[0]])
        F = w.forces.copy()
        F[:, :counts[0]] = _poison(F[:, :counts[0]])
        u = P.matvec(to_dev(F)).cpu().numpy()
        assert np.array_equal(u[:, counts[0]:], ref[:, counts[0]:])
    finally:
        P.free()


# Pairs of the FP64 form as far apart as the FP32 range of their squared distances
# allows in the units of the pair kernels (r of 1.3e19 to 1.8e19 times a power of
# two near the diameter): the far terms are there in full.  The forces are on one
# bead, so that its own term does not hide them.
@pytest.mark.parametrize("nrhs", [1, 4, 16])
def test_most_distant_pairs(orc, nrhs):
    g = np.random.default_rng(410)
    a, m = 2.0**-64, 2.0**63  # 2 a m = 1
    v = g.standard_normal((40, 3))
    pos = np.concatenate([np.zeros((1, 3)), v / np.linalg.norm(v, axis=1, keepdims=True) * g.uniform(1.45, 1.95, (40, 1))])
    assert 1.3e19 < 1.45 * m and 1.95 * m < np.sqrt(np.finfo(np.float32).max)
    F = np.zeros((nrhs, 41, 3))
    F[:, 0] = g.standard_normal((nrhs, 3))
    log(f"most distant pairs nrhs={nrhs}")
    u, st = gpu_matvec(pos, F, a, leaf_size=1000)
    ref = orc.rpy_direct(pos, F, a, 1.0)
    assert st["nleaf"] == 1
    assert orc.rel_l2(u[:, 1:], ref[:, 1:]) <= 1e-12


# A workspace whose partial-sum slots do not fit: the matvec runs in whole tiles
# and coarse items instead, as before there were slots.  Adaptive trees with
# split U, W and O lists, S->M, S->L and evaluation items (FP64 and mixed, on the
# vector units and the matrix cores), and a plan of direct launches.
@pytest.mark.parametrize("n,leaf,nrhs", [(9000, 300, 3), (9000, 300, 18), (4000, 700, 1), (700, 1000, 2)])
def test_workspace_without_slots(orc, n, leaf, nrhs):
    import paper_1711_02976_amd as R
    import torch
    from gpu_common import to_dev
    w = W.clustered(n, 4, 12.0, 0.6, 0.3, nrhs, seed=420)
    log(f"workspace without slots n={n} leaf={leaf} nrhs={nrhs}")
    F = to_dev(w.forces)
    ref = None
    for precision in ("fp64", "mixed"):
        P, Q = (R.Plan(to_dev(w.pos), w.a, w.eta, 1e-6, leaf_size=leaf, order=12, w_direct=60, precision=precision)
                for _ in range(2))
        try:
            P.inject_error("slots")
            u = P.matvec(F)
            v = Q.matvec(F)
            st, sq = P.stats(), Q.stats()
            assert st["device_bytes"] < sq["device_bytes"]
            if n > leaf:
                assert st["list_len"]["X"] > 0
            if n == 9000:
                assert st["list_len"]["O"] > 0
            if ref is None:
                ref = orc.fmm(w.pos, w.forces, w.a, w.eta, 12, leaf, 60)
            u, v = u.cpu().numpy(), v.cpu().numpy()
            if precision == "fp64":
                assert orc.rel_l2(u, ref) <= 1e-12
            else:
                assert orc.rel_l2(u, ref) <= 5e-7
            assert orc.rel_l2(u, v) <= 1e-13
            # the next call needs no new workspace; a larger one has its slots again
            assert torch.equal(P.matvec(F), to_dev(u))
            if nrhs < 16:
                F24 = to_dev(np.resize(w.forces, (24, n, 3)))
                assert torch.equal(P.matvec(F24), Q.matvec(F24))
                assert P.stats()["device_bytes"] == Q.stats()["device_bytes"]
        finally:
            P.free()
            Q.free()


# Positions produced by the default stream for a plan on a stream of its own that
# does not wait for it (the plan's: no wait on the caller's side either): the plan
# is of the new positions.  The old ones are as good, so that a plan of them would
# be whole, and wrong.
def test_positions_of_the_default_stream():
    import paper_1711_02976_amd as R
    import torch
    from gpu_common import to_dev
    w, old = (W.uniform_cube(3000, 1.0, 0.01, nrhs=1, seed=s) for s in (430, 431))
    log("positions of the default stream")
    side = torch.cuda.Stream()
    new, pos = to_dev(w.pos), to_dev(old.pos)
    R.Plan(pos, w.a, w.eta, 1e-6, leaf_size=40, stream=side.cuda_stream).free()  # the kernels are loaded
    torch.cuda.synchronize()
    torch.cuda._sleep(100_000_000)  # 40 ms at the least
    pos.copy_(new)
    P = R.Plan(pos, w.a, w.eta, 1e-6, leaf_size=40, stream=side.cuda_stream)
    try:
        torch.cuda.synchronize()
        keys = P.export()["keys"]
    finally:
        P.free()
    Q = R.Plan(new, w.a, w.eta, 1e-6, leaf_size=40)
    try:
        assert np.array_equal(keys, Q.export()["keys"])
    finally:
        Q.free()


# What the statistics count: a pass per far-field chunk of right-hand sides, with
# and without a far field, and the S->L items of the workspace in use.
@pytest.mark.parametrize("n,leaf", [(300, 1000), (3000, 40)])
def test_timed_passes(n, leaf):
    import paper_1711_02976_amd as R
    from gpu_common import to_dev
    log(f"timed passes n={n}")
    w = W.uniform_cube(n, 1.0, 0.01, nrhs=20, seed=440)
    P = R.Plan(to_dev(w.pos), w.a, w.eta, 1e-3, leaf_size=leaf)
    try:
        P.set_timing(1)
        done = 0
        for nrhs, passes in ((1, 1), (3, 2), (8, 2), (11, 4), (20, 5)):  # 2 + 1; 4 + 4; 4 + 4, 2, 1; five of 4
            P.matvec(to_dev(w.forces[:nrhs]))
            done += passes
            assert P.timings()["passes"] == done, nrhs
    finally:
        P.free()


def test_counted_s2l_items():
    import paper_1711_02976_amd as R
    from gpu_common import to_dev
    w = W.clustered(9000, 4, 12.0, 0.6, 0.05, 1, seed=441)
    log("counted S->L items")
    F = to_dev(w.forces)
    P, Q = (R.Plan(to_dev(w.pos), w.a, w.eta, 1e-6, leaf_size=700, order=8) for _ in range(2))
    try:
        Q.inject_error("slots")
        P.matvec(F)
        Q.matvec(F)
        assert 0 < Q.stats()["p2l_items"] < P.stats()["p2l_items"]
        assert Q.stats()["p2l_split_boxes"] <= P.stats()["p2l_split_boxes"]
    finally:
        P.free()
        Q.free()


# The allocation-free matvec of plans whose workspace fits its 128 MiB only without
# partial-sum slots: whole tiles and coarse items.  A uniform plan of 20 right-hand
# sides, and an adaptive one with W, X and O lists, evaluated W multipoles and
# S->L items that would be finer; FP64 against the oracle FMM, the mixed form
# against it to half its accuracy setting.
@pytest.mark.parametrize("precision", ["fp64", "mixed"])
@pytest.mark.parametrize("kind", ["uniform", "adaptive"])
def test_noalloc_without_slots(orc, kind, precision):
    import paper_1711_02976_amd as R
    import torch
    from gpu_common import to_dev
    if kind == "uniform":
        w, leaf, p, wd = W.uniform_cube(12000, 1.0, 0.005, nrhs=20, seed=450), 250, 12, 0
    else:
        w, leaf, p, wd = W.clustered(9000, 4, 12.0, 0.6, 0.3, 18, seed=451), 300, 12, 60
    log(f"noalloc without slots {kind} {precision}")
    P, Q = (R.Plan(to_dev(w.pos), w.a, w.eta, 1e-6, leaf_size=leaf, order=p, w_direct=wd, precision=precision)
            for _ in range(2))
    try:
        F = to_dev(w.forces)
        st = P.stats()
        if kind == "adaptive":
            assert st["list_len"]["W"] > 0 and st["list_len"]["X"] > 0 and st["list_len"]["O"] > 0
        U = torch.full_like(F, float("nan"))
        R.rpy_matvec_noalloc(P.handle, w.nrhs, F.data_ptr(), U.data_ptr())
        u = U.cpu().numpy()
        assert P.stats()["device_bytes"] == st["device_bytes"]  # nothing allocated
        Q.inject_error("slots")
        v = Q.matvec(F).cpu().numpy()
        without = Q.stats()["device_bytes"] - st["device_bytes"]
        x = P.matvec(F).cpu().numpy()
        full = P.stats()["device_bytes"] - st["device_bytes"]
        log(f"  workspace {full >> 20} MiB with slots, {without >> 20} without, items {P.stats()['p2l_items']} {Q.stats()['p2l_items']}")
        assert without < 127 << 20 and full > 128 << 20
    finally:
        P.free()
        Q.free()
    ref = orc.fmm(w.pos, w.forces, w.a, w.eta, p, leaf, st["w_direct"])
    assert orc.rel_l2(u, ref) <= (1e-12 if precision == "fp64" else 5e-7)
    assert np.array_equal(u, v) and orc.rel_l2(u, x) <= 1e-13


# More boxes than one launch of a block per box takes (fewer than 2^32 threads
# along x).  Coincident pairs in leaves of one bead: a chain of boxes per pair down
# to the deepest level.
def _pairs(m, seed):
    import torch
    from gpu_common import torch_cuda
    torch_cuda()
    g = torch.Generator(device="cuda").manual_seed(seed)
    return torch.rand((m, 3), generator=g, device="cuda", dtype=torch.float64).repeat(2, 1)


# M->L of 12 waves (FP64, order 11) over more than 2^32 / 768 boxes, against the
# dense operator on the same tree, whose blocks of 256 threads fit one launch.
def test_more_boxes_than_a_launch_m2l():
    import paper_1711_02976_amd as R
    import torch
    log("M->L over more boxes than a launch takes")
    pos = _pairs(430_000, 460)
    F = torch.randn((1, pos.shape[0], 3), generator=torch.Generator(device="cuda").manual_seed(461), device="cuda",
                    dtype=torch.float64)
    u = []
    for mode in ("dense", "rotation"):
        P = R.Plan(pos, 2e-3, 1.0, 3e-5, leaf_size=1, order=11, max_depth=21, m2l=mode)
        try:
            st = P.stats()
            u.append(P.matvec(F))
            torch.cuda.synchronize()
        finally:
            P.free()
    assert st["nbox"] - st["nleaf"] > 2**32 // 768 and st["list_len"]["V"] > 0
    assert float((u[1] - u[0]).norm() / u[0].norm()) <= 1e-12


# The tree and its lists over more than 2^32 / 64 boxes: the two levels more add a
# box each per pair and no list entries (the pairs are far apart there).
def test_more_boxes_than_a_launch_tree():
    import paper_1711_02976_amd as R
    log("tree over more boxes than a launch takes")
    pos = _pairs(5_300_000, 462)
    st = []
    for depth in (19, 21):
        P = R.Plan(pos, 1e-12, 1.0, 1e-3, leaf_size=1, order=1, max_depth=depth)
        try:
            st.append(P.stats())
        finally:
            P.free()
    a, b = st
    log(f"  boxes {a['nbox']} {b['nbox']}, plans {a['plan_ms']:.0f} {b['plan_ms']:.0f} ms")
    assert a["nbox"] <= 2**32 // 64 - 8 < b["nbox"]
    assert a["nleaf"] == b["nleaf"] == 5_300_000 and b["nbox"] == a["nbox"] + 2 * a["nleaf"]
    assert a["list_len"] == b["list_len"] and a["list_len"]["U"] == a["nleaf"]


# What freed plans left with the library goes back to the device when the program
# asks for it, and a plan in use and the next one are none the worse.
def test_release_memory(orc):
    import paper_1711_02976_amd as R
    import torch
    from gpu_common import to_dev
    w = W.uniform_cube(20000, 1.0, 0.005, nrhs=2, seed=470)
    log("released memory")
    pos, F = to_dev(w.pos), to_dev(w.forces)

    def free_bytes():
        torch.cuda.synchronize()
        return torch.cuda.mem_get_info()[0]

    P = R.Plan(pos, w.a, w.eta, 1e-6, leaf_size=100, order=8)
    try:
        u = P.matvec(F)
        u2 = torch.empty_like(u)
        for _ in range(2):  # the first time, the runtime makes its hardware queues
            R.rpy_release_memory()
            before = free_bytes()
            Q = R.Plan(pos, w.a, w.eta, 1e-6, leaf_size=100, order=8)
            R.rpy_matvec(Q.handle, 2, F.data_ptr(), u2.data_ptr())
            Q.free()
            kept = before - free_bytes()
            R.rpy_release_memory()
        log(f"  kept {kept >> 10} KiB, after the release {(before - free_bytes()) >> 10}")
        assert kept >= 8 << 20 and before - free_bytes() <= 2 << 20
        R.rpy_matvec(P.handle, 2, F.data_ptr(), u2.data_ptr())
        assert torch.equal(u2, u)
        Q = R.Plan(pos, w.a, w.eta, 1e-6, leaf_size=100, order=8)
        assert torch.equal(Q.matvec(F), u)
        Q.free()
    finally:
        P.free()
