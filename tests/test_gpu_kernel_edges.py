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
