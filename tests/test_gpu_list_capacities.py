"""Tree and lists against the oracle where a list or a target's open pairs go
beyond what the kernels keep in LDS, and where the buffers' first sizes do not
do; each case says by the lists themselves that it gets there."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():  # pragma: no cover
    pytest.skip("no GPU", allow_module_level=True)

from paper_2005_12351_amd import fmm  # noqa: E402
from tests.test_gpu_kernel_edges import _points, _tree_equal  # noqa: E402

M2L_LDS, P2P_LDS, OPEN_LDS = 3072, 2048, 2048   # tree_gpu.hip: kM2LBuf, kP2PBuf, kOpenBuf
SORT_BATCH = 1 << 22                             # kLongBatch


def _unsorted_lists(o, which, above):
    """entries of lists longer than `above` whose sources are of several levels (the walk's order is not theirs)"""
    ptr, src = (o.m2l_ptr, o.m2l_src) if which == "m2l" else (o.p2p_ptr, o.p2p_src)
    tot = 0
    for c in np.nonzero(np.diff(ptr) > above)[0]:
        lev = o.level[src[ptr[c]:ptr[c + 1]]]
        if lev.min() != lev.max():
            tot += int(ptr[c + 1] - ptr[c])
    return tot


# lists that are sorted outside LDS: P2P lists of every cell of a dense cube
# (one batch of the sort), and M2L and P2P lists with more entries in all than
# a batch takes
@pytest.mark.parametrize("kind,n,ncrit,theta,m2l,batches", [("cluster", 9000, 1, 0.2, False, False),
                                                            ("uniform", 9000, 2, 0.12, True, True)])
def test_lists_beyond_lds(orc, kind, n, ncrit, theta, m2l, batches):
    pos = np.ascontiguousarray(_points(kind, n))
    print(f"[long lists] {kind} n={n} ncrit={ncrit} theta={theta}", flush=True)
    o = orc.Tree(pos, ncrit, theta).dump()
    p = _unsorted_lists(o, "p2p", P2P_LDS)
    m = _unsorted_lists(o, "m2l", M2L_LDS)
    assert p > 0 and (m > 0) == m2l and (p + m > SORT_BATCH) == batches, (p, m)
    for where in (fmm.FMM_SCHEDULE_AUTO, fmm.FMM_SCHEDULE_HOST):
        ctx = fmm.Context(0)
        ctx.set_m2l_schedule(where)
        gt = fmm.Tree(ctx, torch.from_numpy(pos).cuda(), ncrit, theta)
        _tree_equal(gt, o)
        gt.close()
        ctx.close()


def _open_pairs(o, theta):
    """pairs (source, target) that each target cell leaves open to its children: neither accepted nor of two leaves,
    and split at the target"""
    lev, ix = o.level.astype(np.int64), o.ix.astype(np.int64).reshape(-1, 3)
    ch0, nch = o.child0.astype(np.int64), o.nchild.astype(np.int64)
    count = np.zeros(len(lev), np.int64)
    a = b = np.zeros(1, np.int64)

    def split(x, y):
        """x's children, each with its y"""
        k = nch[x]
        return np.repeat(ch0[x], k) + np.arange(k.sum()) - np.repeat(np.cumsum(k) - k, k), np.repeat(y, k)

    while len(a):
        ra, rb = 1 << (21 - lev[a]), 1 << (21 - lev[b])
        d = (2 * ix[b] + 1) * rb[:, None] - (2 * ix[a] + 1) * ra[:, None]
        near = ~((ra + rb).astype(float) ** 2 < theta * theta * (d.astype(float) ** 2).sum(1))
        la, lb = nch[a] == 0, nch[b] == 0
        rest = near & ~(la & lb)
        source = rest & (lb | (~la & (ra > rb)))
        target = rest & ~source
        np.add.at(count, b[target], 1)
        both = target & ~la & (ra == rb)
        only = target & ~both
        a1, b1 = split(a[source], b[source])
        b2, a2 = split(b[only], a[only])
        b3, a3 = split(b[both], a[both])
        a3, b3 = split(a3, b3)
        a, b = np.concatenate([a1, a2, a3]), np.concatenate([b1, b2, b3])
    return count


# a target with more open pairs than its LDS buffer takes walks twice
def test_open_pairs_beyond_lds(orc):
    n, ncrit, theta = 4100, 1, 0.1
    pos = np.ascontiguousarray(_points("uniform", n))
    print(f"[open pairs] n={n} ncrit={ncrit} theta={theta}", flush=True)
    o = orc.Tree(pos, ncrit, theta).dump()
    assert _open_pairs(o, theta).max() > OPEN_LDS
    ctx = fmm.Context(0)
    gt = fmm.Tree(ctx, torch.from_numpy(pos).cuda(), ncrit, theta)
    _tree_equal(gt, o)
    gt.close()
    ctx.close()


# a context whose budget leaves the open pairs' buffer fewer entries than they
# need (1/512 of it in bytes) runs the levels again with more
@pytest.mark.parametrize("kind,n,ncrit,theta,budget", [("uniform", 9000, 1, 0.5, 1 << 20), ("cluster", 4000, 4, 0.4, 1 << 16),
                                                       ("same", 300, 3, 0.5, 1 << 10)])
@pytest.mark.parametrize("where", [fmm.FMM_SCHEDULE_AUTO, fmm.FMM_SCHEDULE_HOST])
def test_open_pairs_beyond_their_buffer(orc, kind, n, ncrit, theta, budget, where):
    pos = np.ascontiguousarray(_points(kind, n))
    print(f"[open buffer] {kind} n={n} ncrit={ncrit} theta={theta} budget={budget}", flush=True)
    o = orc.Tree(pos, ncrit, theta).dump()
    assert _open_pairs(o, theta).sum() > max(1, budget // 8 // 64)
    ctx = fmm.Context(0, budget_bytes=budget)
    ctx.set_m2l_schedule(where)
    gt = fmm.Tree(ctx, torch.from_numpy(pos).cuda(), ncrit, theta)
    _tree_equal(gt, o)
    gt.close()
    ctx.close()
