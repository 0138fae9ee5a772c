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
