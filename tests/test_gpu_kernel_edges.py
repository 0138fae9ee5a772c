"""Edges of the kernels' tiles and dispatch rules, against the oracle: sizes
where a tile, slice or chunk ends, is nearly empty or is exceeded.  Both sides
compute the same truncated sums in another order, so the bounds are those of
the FP64 and MIXED parity tests."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():  # pragma: no cover
    pytest.skip("no GPU", allow_module_level=True)

from paper_2005_12351_amd import fmm  # noqa: E402
from paper_2005_12351_amd import workloads as W  # noqa: E402
from tests.gpu_helpers import PHI_FLOOR, to_dev, within  # noqa: E402

FP64, MIXED = fmm.FMM_PREC_FP64, fmm.FMM_PREC_MIXED


@pytest.fixture(scope="module")
def ctx():
    c = fmm.Context(0)
    yield c
    c.close()


def _workload(seed, order, n, kind, p, ncrit, theta=0.5):
    if order >= 16:
        return W.small_mixed(seed, n, order - 16, kind, p=p, theta=theta, ncrit=ncrit)
    return W.small_random(seed, n, order, kind, p=p, theta=theta, ncrit=ncrit)


# leaves above 256 targets (a second pass over the lists), of one particle,
# of 129 (one slice), lists above 256 entries (a second window), every single
# order and the run-time mask
@pytest.mark.parametrize("order,n,ncrit,kind", [(0, 300, 512, "uniform"), (1, 260, 300, "uniform"), (2, 129, 130, "uniform"),
                                                (3, 600, 40, "plummer"), (16 + 9, 700, 300, "plummer"),
                                                (1, 900, 1, "uniform"), (16 + 7, 65, 64, "uniform")])
def test_derivatives_tiles(orc, ctx, order, n, ncrit, kind):
    p = 6
    w = _workload(4100 + n, order, n, kind, p, ncrit)
    print(f"[derivs tiles] order={order} n={n} ncrit={ncrit} {kind}", flush=True)
    t = fmm.Tree(ctx, to_dev(w.pos), ncrit, w.theta)
    t.upward(w.order, to_dev(w.moments), p, FP64)
    ot = orc.Tree(w.pos, ncrit, w.theta)
    ok = True
    for K in (1, 2, 3):
        d = t.evaluate_derivs(K)
        torch.cuda.synchronize()
        # pooled and per target: the bounds of the FP64 derivative parity test
        ok &= within(d.cpu().numpy(), ot.fmm_derivs(w.order, w.moments, p, K), FP64, f"order {K}", (1e-10, 1e-12))
    t.close()
    assert ok


# the matrix-core M2L over its row chunks (one to four lines), LDS buffers
# (odd and even chunk counts of two buffers, one buffer) and pieces with fewer
# entries than waves; ncrit 4 at n = 700 gives pieces of a few hundred entries
@pytest.mark.parametrize("p,s", [(1, 0), (4, 0), (5, 0), (6, 1), (7, 2), (8, 0), (8, 1), (8, 3), (9, 1), (10, 0), (10, 1),
                                 (10, 2), (10, 3)])
@pytest.mark.parametrize("n,ncrit", [(150, 16), (700, 4)])
def test_matrix_core_m2l_chunks(orc, ctx, p, s, n, ncrit):
    w = _workload(4200 + 10 * p + s, s, n, "uniform", p, ncrit)
    print(f"[mfma m2l] p={p} s={s} n={n}", flush=True)
    ctx.set_m2l_engine(fmm.FMM_M2L_ENGINE_MFMA)
    try:
        t = fmm.Tree(ctx, to_dev(w.pos), ncrit, w.theta)
        phi, E = t.run(s, to_dev(w.moments), p, MIXED)
        torch.cuda.synchronize()
    finally:
        ctx.set_m2l_engine(fmm.FMM_M2L_ENGINE_AUTO)
    assert t.info()["n_m2l"] > 0
    ophi, oE = orc.Tree(w.pos, ncrit, w.theta).fmm(w.order, w.moments, p)[:2]
    ok = within(E.cpu().numpy(), oE, MIXED, "E")
    ok &= within(phi.cpu().numpy(), ophi, MIXED, "phi", floor=PHI_FLOOR)
    t.close()
    assert ok


# the combine's split of a tile's row sets: one tile of hundreds of sets (32
# threads a sum), a few tiles (8), many (1); fewer cells than a workgroup holds
@pytest.mark.parametrize("n,ncrit,p,s", [(100, 4, 1, 0), (1000, 64, 4, 0), (1000, 64, 6, 1), (3000, 16, 5, 2),
                                         (8000, 8, 4, 1)])
@pytest.mark.parametrize("prec,basis", [(FP64, fmm.FMM_M2L_HARMONIC), (MIXED, fmm.FMM_M2L_HARMONIC),
                                        (FP64, fmm.FMM_M2L_FULL)])
def test_combine_parts(orc, ctx, n, ncrit, p, s, prec, basis):
    w = _workload(4300 + n + p, s, n, "uniform", p, ncrit)
    print(f"[combine] n={n} ncrit={ncrit} p={p} s={s} precision={prec} basis={basis}", flush=True)
    ctx.set_m2l_basis(basis)
    try:
        t = fmm.Tree(ctx, to_dev(w.pos), ncrit, w.theta)
        phi, E = t.run(s, to_dev(w.moments), p, prec)
        torch.cuda.synchronize()
    finally:
        ctx.set_m2l_basis(fmm.FMM_M2L_HARMONIC)
    ophi, oE = orc.Tree(w.pos, ncrit, w.theta).fmm(w.order, w.moments, p)[:2]
    ok = within(E.cpu().numpy(), oE, prec, "E")
    ok &= within(phi.cpu().numpy(), ophi, prec, "phi", floor=PHI_FLOOR)
    t.close()
    assert ok


def _tree_equal(gt, o):
    g = gt.export()
    assert np.array_equal(g["geom"][:3], o.lo) and g["geom"][3] == o.W
    for k in ("key", "perm", "level", "ix", "first", "count", "parent", "child0", "nchild", "m2l_ptr", "m2l_src",
              "p2p_ptr", "p2p_src"):
        assert g[k].shape == getattr(o, k).shape, k
        assert np.array_equal(g[k].astype(np.int64), getattr(o, k).astype(np.int64)), k


def _points(kind, n):
    rng = np.random.default_rng(4400 + n)
    if kind == "cluster":       # one dense cube and a few far particles: long lists, pairs that split the source alone
        return np.concatenate([0.05 * rng.random((n, 3)), rng.random((40, 3))])
    if kind == "multi":         # clusters of very different sizes: more pair geometries than are ranked by counting
        rng = np.random.default_rng(1)
        return np.concatenate([rng.random(3) + 10.0 ** (-k) * rng.random((n // 6, 3)) for k in (0.5, 1, 1.5, 2, 2.5, 3)])
    if kind == "same":          # many particles at one place: a chain of cells to the depth cap
        return np.concatenate([rng.random((n - 20, 3)), np.tile(rng.random((1, 3)), (20, 1))])
    return rng.random((n, 3))


# the tree and the lists against the oracle, whole numbers: workgroups of 256
# particles (just below, at and above), windows beyond LDS (ncrit > 3840) and
# beyond the input, one cell, a depth-cap chain, lists of several thousand P2P
# sources (beyond LDS, with the open pairs: test_gpu_list_capacities)
@pytest.mark.parametrize("kind,n,ncrit,theta", [("uniform", 255, 8, 0.5), ("uniform", 256, 256, 0.5),
                                                ("uniform", 257, 256, 0.5), ("uniform", 513, 1, 0.6),
                                                ("uniform", 9000, 4000, 0.5), ("uniform", 9000, 3840, 0.5),
                                                ("uniform", 9000, 9000, 0.5), ("same", 300, 3, 0.5),
                                                ("cluster", 4000, 1, 0.3), ("cluster", 4000, 4, 0.7),
                                                ("multi", 9000, 8, 0.5), ("uniform", 3000, 2, 0.15)])
def test_tree_and_lists_edges(orc, ctx, kind, n, ncrit, theta):
    pos = np.ascontiguousarray(_points(kind, n))
    print(f"[tree edges] {kind} n={n} ncrit={ncrit} theta={theta}", flush=True)
    gt = fmm.Tree(ctx, torch.from_numpy(pos).cuda(), ncrit, theta)
    _tree_equal(gt, orc.Tree(pos, ncrit, theta).dump())
    gt.close()


# the device's schedule against the host's where the classes are sorted
# instead of counted (more than 8192), and just with few of them
@pytest.mark.parametrize("kind,n,ncrit,theta,many", [("multi", 9000, 1, 0.3, True), ("cluster", 4000, 4, 0.7, False)])
def test_schedule_class_paths(kind, n, ncrit, theta, many):
    pos = torch.from_numpy(np.ascontiguousarray(_points(kind, n))).cuda()
    print(f"[schedule classes] {kind} n={n} ncrit={ncrit} theta={theta}", flush=True)
    dev, host = fmm.Context(0), fmm.Context(0)
    host.set_m2l_schedule(fmm.FMM_SCHEDULE_HOST)
    td, th = fmm.Tree(dev, pos, ncrit, theta), fmm.Tree(host, pos, ncrit, theta)
    a, b = td.m2l_schedule(), th.m2l_schedule()
    assert a["where"] == fmm.FMM_SCHEDULE_DEVICE and (td.info()["n_classes"] > 8192) == many
    for k in ("tile_cell", "tile_uoff", "ucls", "usrc", "cls_geom"):
        assert a[k].shape == b[k].shape and np.array_equal(a[k], b[k]), k
    for t in (td, th):
        t.close()
    dev.close()
    host.close()


# Barnes-Hut: one wavefront a group, two and eight; rows through places in LDS
# (the MIXED field from p 6 on) and not (the others, from p 8 or 9 on in
# test_gpu_bh_orders); a root that is a leaf, a tree that ends above and below the
# level whose cells are shared out, a last group of one particle
@pytest.mark.parametrize("n,ncrit,p,s,kind", [(1, 8, 6, 0, "uniform"), (40, 64, 6, 1, "uniform"), (65, 8, 6, 1, "uniform"),
                                              (129, 4, 5, 2, "plummer"), (2000, 64, 7, 1, "uniform"),
                                              (3000, 2, 6, 3, "plummer"), (9000, 16, 6, 0, "plummer"),
                                              (20001, 32, 6, 1, "uniform"), (40000, 64, 4, 1, "plummer")])
@pytest.mark.parametrize("prec", [FP64, MIXED])
def test_barnes_hut_shares(orc, ctx, n, ncrit, p, s, kind, prec):
    w = _workload(4500 + n, s, n, kind, p, ncrit)
    print(f"[bh shares] n={n} ncrit={ncrit} p={p} s={s} {kind} precision={prec}", flush=True)
    t = fmm.Tree(ctx, to_dev(w.pos), ncrit, 0.5, fmm.FMM_METHOD_BH)
    t.upward(s, to_dev(w.moments), p, prec)
    phi, E = t.evaluate()
    _, _, G = t.evaluate_grad()
    torch.cuda.synchronize()
    tg = np.arange(n) if n <= 3000 else np.sort(np.random.default_rng(3).choice(n, 1500, replace=False))
    ophi, oE, oG = orc.Tree(w.pos, ncrit).bh(w.order, w.moments, p, 0.5, targets=tg, want_grad=True)
    ok = within(E.cpu().numpy()[tg], oE, prec, "E")
    ok &= within(phi.cpu().numpy()[tg], ophi, prec, "phi", floor=PHI_FLOOR)
    # the gradient's bounds: as in the gradient parity test
    ok &= within(G.cpu().numpy()[tg], oG, prec, "G", None if prec == FP64 else (2e-6, 1e-4))
    t.close()
    assert ok


# the shifts' row cuts (lowest and highest p and s), parents of one to eight
# children, chains of single children, both bases
@pytest.mark.parametrize("basis", [fmm.FMM_M2L_HARMONIC, fmm.FMM_M2L_FULL])
@pytest.mark.parametrize("p,s,n,ncrit,kind", [(1, 0, 90, 1, "plummer"), (2, 1, 200, 2, "uniform"), (4, 3, 300, 4, "plummer"),
                                              (10, 0, 500, 8, "plummer"), (10, 3, 400, 8, "uniform")])
def test_shift_edges(orc, ctx, basis, p, s, n, ncrit, kind):
    w = _workload(4700 + n, s, n, kind, p, ncrit)
    print(f"[shift] p={p} s={s} n={n} ncrit={ncrit} {kind} basis={basis}", flush=True)
    ctx.set_m2l_basis(basis)
    try:
        ok = True
        for prec in (FP64, MIXED):
            t = fmm.Tree(ctx, to_dev(w.pos), ncrit, w.theta)
            t.upward(w.order, to_dev(w.moments), p, prec)
            phi, E = t.evaluate()
            torch.cuda.synchronize()
            rphi, rE = orc.Tree(w.pos, ncrit, w.theta).fmm(w.order, w.moments, p)[:2]
            ok &= within(phi.cpu().numpy(), rphi, prec, "phi", floor=PHI_FLOOR)
            ok &= within(E.cpu().numpy(), rE, prec, "field")
            t.close()
    finally:
        ctx.set_m2l_basis(fmm.FMM_M2L_HARMONIC)
    assert ok


# L2P of harmonic rows at the orders where its unrolled length changes most
# (one, two, the longest), packs of as many leaves as a wavefront takes, leaves
# of more than 64 targets
@pytest.mark.parametrize("p,s,n,ncrit,kind", [(2, 1, 60, 4, "uniform"), (1, 0, 300, 4, "plummer"), (3, 1, 500, 2, "uniform"),
                                              (9, 2, 700, 200, "uniform"), (10, 1, 900, 130, "plummer"),
                                              (10, 0, 400, 3, "uniform")])
def test_l2p_edges(orc, ctx, p, s, n, ncrit, kind):
    w = _workload(4800 + n, s, n, kind, p, ncrit)
    print(f"[l2p] p={p} s={s} n={n} ncrit={ncrit} {kind}", flush=True)
    t = fmm.Tree(ctx, to_dev(w.pos), ncrit, w.theta)
    t.upward(s, to_dev(w.moments), p, FP64)
    grad = p - s >= 2
    if grad:
        phi, E, G = t.evaluate_grad()
    else:
        phi, E = t.evaluate()
    torch.cuda.synchronize()
    o = orc.Tree(w.pos, ncrit, w.theta).fmm(w.order, w.moments, p, want_grad=grad)
    ok = within(phi.cpu().numpy(), o[0], FP64, "phi", floor=PHI_FLOOR)
    ok &= within(E.cpu().numpy(), o[1], FP64, "E")
    if grad:
        ok &= within(G.cpu().numpy(), o[2], FP64, "G")
    t.close()
    assert ok


# P2M of harmonic rows: every set of source orders, orders below and above the
# source's (a mixed set with p under its highest order), the bounds of its
# kernels' orders, leaves of one particle, of 64 (one pass), 65 and more
@pytest.mark.parametrize("mask,p,n,ncrit,kind", [(1, 1, 130, 1, "plummer"), (2, 4, 500, 65, "uniform"), (4, 5, 520, 64, "uniform"),
                                                 (8, 6, 600, 66, "plummer"), (3, 7, 900, 200, "uniform"), (5, 8, 700, 30, "plummer"),
                                                 (6, 9, 700, 130, "uniform"), (9, 2, 400, 8, "uniform"), (10, 10, 600, 64, "plummer"),
                                                 (12, 4, 500, 40, "uniform"), (7, 10, 900, 300, "uniform"), (15, 3, 500, 16, "plummer"),
                                                 (11, 6, 500, 33, "uniform"), (13, 8, 500, 20, "plummer"), (14, 9, 500, 70, "uniform")])
@pytest.mark.parametrize("prec", [FP64, MIXED])
def test_p2m_edges(orc, ctx, mask, p, n, ncrit, kind, prec):
    w = _workload(4900 + mask, 16 + mask, n, kind, p, ncrit)
    print(f"[p2m] mask={mask} p={p} n={n} ncrit={ncrit} {kind} precision={prec}", flush=True)
    t = fmm.Tree(ctx, to_dev(w.pos), ncrit, w.theta)
    t.upward(w.order, to_dev(w.moments), p, prec)
    phi, E = t.evaluate()
    torch.cuda.synchronize()
    ophi, oE = orc.Tree(w.pos, ncrit, w.theta).fmm(w.order, w.moments, p)[:2]
    ok = within(phi.cpu().numpy(), ophi, prec, "phi", floor=PHI_FLOOR)
    ok &= within(E.cpu().numpy(), oE, prec, "E")
    t.close()
    assert ok


# the FP64 M2L on the matrix cores (p - s of 8 and 9) beside the vector kernels on
# both sides of its range; few entries a wave, many, and levels that differ
@pytest.mark.parametrize("p,s", [(7, 0), (8, 0), (9, 0), (10, 0), (9, 1), (10, 1), (10, 2), (10, 3)])
@pytest.mark.parametrize("n,ncrit,kind", [(150, 16, "uniform"), (900, 8, "uniform"), (1500, 12, "plummer")])
def test_fp64_m2l_range(orc, ctx, p, s, n, ncrit, kind):
    w = _workload(5000 + 10 * p + s, s, n, kind, p, ncrit)
    print(f"[fp64 m2l] p={p} s={s} n={n} ncrit={ncrit} {kind}", flush=True)
    t = fmm.Tree(ctx, to_dev(w.pos), ncrit, w.theta)
    phi, E = t.run(s, to_dev(w.moments), p, FP64)
    torch.cuda.synchronize()
    assert t.info()["n_m2l"] > 0
    ophi, oE = orc.Tree(w.pos, ncrit, w.theta).fmm(w.order, w.moments, p)[:2]
    ok = within(E.cpu().numpy(), oE, FP64, "E")
    ok &= within(phi.cpu().numpy(), ophi, FP64, "phi", floor=PHI_FLOOR)
    t.close()
    assert ok


# a Barnes-Hut tree whose limit has no room for the shared groups' sums: the call
# is accepted as it is without them, and gives the same sums in another order
def test_barnes_hut_without_share_scratch():
    n, p = 3001, 7
    w = _workload(5200, 1, n, "plummer", p, 32)
    pos, mom = to_dev(w.pos), to_dev(w.moments)
    out = []
    for cut in (0, 1):
        c = fmm.Context(0)
        if cut:
            c.set_tree_limit(out[0][2] - 1)   # one byte less than with the sums
        t = fmm.Tree(c, pos, 32, 0.6, fmm.FMM_METHOD_BH)
        t.upward(1, mom, p, FP64)
        phi, E = t.evaluate()
        torch.cuda.synchronize()
        out.append((phi.cpu().numpy(), E.cpu().numpy(), t.info()["bytes"]))
        t.close()
        c.close()
    assert out[1][2] < out[0][2]
    assert within(out[1][0], out[0][0], FP64, "phi", floor=PHI_FLOOR) & within(out[1][1], out[0][1], FP64, "E")
