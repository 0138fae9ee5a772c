"""Device memory against a tree limit: what a set-up may hold, and calls that a
limit allows by what their result needs."""
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


# the host-made tables of a tree count with their own bytes: a system of one
# cell and one of a few hundred in the bytes that each took with every table an
# allocation of its own (dipoles, p 4, MIXED, harmonic basis; FMM)
@pytest.mark.parametrize("n,where,build,total", [(1, fmm.FMM_SCHEDULE_DEVICE, 180, 9960), (1, fmm.FMM_SCHEDULE_HOST, 176, 9956),
                                                 (300, fmm.FMM_SCHEDULE_DEVICE, 121860, 1714708),
                                                 (300, fmm.FMM_SCHEDULE_HOST, 112780, 1705628)])
def test_tables_count_their_own_bytes(n, where, build, total):
    w = W.small_random(3, n, 1, "uniform", p=4, theta=0.5, ncrit=32)
    pos, mom = to_dev(w.pos), to_dev(w.moments)
    c = fmm.Context(0)
    c.set_m2l_schedule(where)
    c.set_tree_limit(total)
    t = fmm.Tree(c, pos, 32, 0.5)
    assert t.info()["bytes"] <= build
    t.upward(1, mom, 4, MIXED)
    assert t.info()["bytes"] <= total
    phi, E = t.evaluate()
    torch.cuda.synchronize()
    assert torch.isfinite(phi).all() and torch.isfinite(E).all()
    t.close()
    c.close()


# FP64 M2L of p - s 8 and 9: limits of what the trees held with the vector
# kernels (rows of a multiple of four, their own cut of the work)
@pytest.mark.parametrize("n,s,p,limit", [(100, 0, 9, None), (300, 0, 8, 17475176), (300, 0, 9, 20311404), (300, 2, 10, 18624648),
                                         (3000, 0, 8, 24360672), (3000, 0, 9, 28383604), (3000, 1, 9, 25496400),
                                         (3000, 1, 10, 29937364), (20000, 1, 9, 44753720)])
def test_fp64_m2l_rows_fit_the_limit(orc, n, s, p, limit):
    w = W.small_random(3, n, s, "uniform", p=4, theta=0.5, ncrit=32)
    pos, mom = to_dev(w.pos), to_dev(w.moments)
    out = []
    for cut in (0, 1):
        c = fmm.Context(0)
        if cut:
            c.set_tree_limit(limit or out[0][2] - 300)
        t = fmm.Tree(c, pos, 32, 0.5)
        t.upward(s, mom, p, FP64)
        phi, E = t.evaluate()
        torch.cuda.synchronize()
        out.append((phi.cpu().numpy(), E.cpu().numpy(), t.info()["bytes"]))
        t.close()
        c.close()
    ok = within(out[1][0], out[0][0], FP64, "phi", floor=PHI_FLOOR) & within(out[1][1], out[0][1], FP64, "E")
    if n <= 3000:
        po, Eo = orc.Tree(w.pos, 32, 0.5).fmm(s, w.moments, p)[:2]
        ok &= within(out[1][0], po, FP64, "phi (oracle)", floor=PHI_FLOOR) & within(out[1][1], Eo, FP64, "E (oracle)")
    assert ok


# a tree whose M2L schedule the device gives up (more than 4096 pair geometries
# in a tile): it holds what a tree with the host's schedule holds, fits its
# limit and has the same schedule
@pytest.mark.parametrize("n,ncrit,theta", [(3000, 4, 0.2)])
def test_schedule_given_up_holds_what_the_host_s_does(n, ncrit, theta):
    pos = torch.from_numpy(np.random.default_rng(5 + n).random((n, 3))).cuda()
    dev, host = fmm.Context(0), fmm.Context(0)
    host.set_m2l_schedule(fmm.FMM_SCHEDULE_HOST)
    th = fmm.Tree(host, pos, ncrit, theta)
    dev.set_tree_limit(th.info()["bytes"])
    td = fmm.Tree(dev, pos, ncrit, theta)
    a, b = td.m2l_schedule(), th.m2l_schedule()
    assert a["where"] == b["where"] == fmm.FMM_SCHEDULE_HOST
    assert td.info()["bytes"] == th.info()["bytes"]
    for k in ("tile_cell", "tile_uoff", "ucls", "usrc", "cls_geom"):
        assert np.array_equal(a[k], b[k]), k
    x, y = td.export(), th.export()
    for k in ("m2l_ptr", "m2l_src", "p2p_ptr", "p2p_src"):
        assert np.array_equal(x[k], y[k]), k
    for t in (td, th):
        t.close()
    dev.close()
    host.close()


# Barnes-Hut set up at one p and then at a higher one, under a limit that the
# second reaches without the shared groups' sums: those of the first must not
# count against it
def test_barnes_hut_set_up_again_at_a_higher_order(orc):
    n, ncrit = 2000, 1
    w = W.small_random(6100, n, 1, "uniform", p=4, theta=0.6, ncrit=ncrit)
    pos, mom = to_dev(w.pos), to_dev(w.moments)

    def held(p, limit):
        c = fmm.Context(0)
        c.set_tree_limit(limit)
        t = fmm.Tree(c, pos, ncrit, 0.6, fmm.FMM_METHOD_BH)
        t.upward(1, mom, p, FP64)
        b = t.info()["bytes"]
        t.close()
        c.close()
        return b

    bare = held(10, held(10, 0) - 1)   # p 10 without the sums
    assert held(4, 0) < bare           # p 4 has room for them
    c = fmm.Context(0)
    c.set_tree_limit(bare)
    t = fmm.Tree(c, pos, ncrit, 0.6, fmm.FMM_METHOD_BH)
    out = []
    for p in (4, 10, 4):
        t.upward(1, mom, p, FP64)
        phi, E = t.evaluate()
        torch.cuda.synchronize()
        out.append((phi.cpu().numpy(), E.cpu().numpy()))
    assert np.array_equal(out[0][0], out[2][0]) and np.array_equal(out[0][1], out[2][1])
    po, Eo = orc.Tree(w.pos, ncrit).bh(1, w.moments, 10, 0.6)[:2]
    assert within(out[1][0], po, FP64, "phi", floor=PHI_FLOOR) & within(out[1][1], Eo, FP64, "E")
    t.close()
    c.close()


# larger sums of shared groups belong to the context: they take nothing of a
# tree's limit or of a request's footprint, and two trees of one context in turn
# give what each gives alone, also as replayed graphs
def test_barnes_hut_sums_of_the_context(orc):
    ctx = fmm.Context(0)
    trees = []
    for n, s in ((8192, 1), (20001, 0)):
        w = W.small_random(6200 + n, n, s, "plummer", p=6, theta=0.6, ncrit=64)
        own = fmm.Context(0)
        t = fmm.Tree(own, to_dev(w.pos), 64, 0.6, fmm.FMM_METHOD_BH)
        t.upward(s, to_dev(w.moments), 6, FP64)
        phi, E, G = (x.cpu().numpy() for x in t.evaluate_grad())
        held = t.info()["bytes"]
        # 8 to 2 wavefronts of 80 bytes a particle would be 5.2 and 3.2 MB more
        assert held < 8 * n * (3 + 1 + 0.5 + 3 + 4 + 4) + t.info()["ncells"] * (64 + 8 * 52)
        t.close()
        own.close()
        t = fmm.Tree(ctx, to_dev(w.pos), 64, 0.6, fmm.FMM_METHOD_BH)
        trees.append((t, s, to_dev(w.moments), phi, E, G, [torch.empty_like(torch.from_numpy(x)).cuda() for x in (phi, E, G)]))
    for _ in range(3):
        for t, s, mom, phi, E, G, out in trees:
            t.upward(s, mom, 6, FP64)
            t.evaluate_grad(fmm.FMM_POT | fmm.FMM_FIELD | fmm.FMM_GRAD, *out)
        torch.cuda.synchronize()
        for t, s, mom, phi, E, G, out in trees:
            for a, b in zip(out, (phi, E, G)):
                assert np.array_equal(a.cpu().numpy(), b)
    for x in trees:
        x[0].close()
    ctx.close()


# a Barnes-Hut request of few cells holds no more than it was admitted with
@pytest.mark.parametrize("n", [3000, 8192, 32768])
def test_barnes_hut_request_within_its_footprint(n):
    w = W.small_random(6300, n, 0, "uniform", p=4, theta=0.5, ncrit=n)
    ctx = fmm.Context(0, budget_bytes=1 << 30)
    ctx.serve_start(1)
    pos, mom = to_dev(w.pos), to_dev(w.moments)
    phi, E = torch.empty(n, dtype=torch.float64, device="cuda"), torch.empty((n, 3), dtype=torch.float64, device="cuda")
    k = ctx.submit(n=n, order=0, p=4, theta=0.5, ncrit=n, pos=pos, moments=mom, phi=phi, field=E, method=fmm.FMM_METHOD_BH)
    ctx.wait(k, 60.0)
    t = ctx.request_times(k)
    assert 0 < t["bytes_used"] <= t["footprint"]
    ctx.close()
