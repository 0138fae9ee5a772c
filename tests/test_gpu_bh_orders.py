"""Barnes-Hut at the orders from which cells wait in LDS (MIXED field p 6,
gradient 8; FP64 field 8, gradient 9, of dipoles 10), with one and two wavefronts a group of
particles, and the FP64 gradient just below, where the M2P is written out (both
bases, charges to octupoles), against the oracle."""
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


def _check(orc, w, order, n, ncrit, p, prec, basis, sample):
    ctx = fmm.Context(0)
    ctx.set_m2l_basis(basis)
    t = fmm.Tree(ctx, to_dev(w.pos), ncrit, 0.5, fmm.FMM_METHOD_BH)
    t.upward(order, to_dev(w.moments), p, prec)
    phi, E = t.evaluate()
    gphi, gE, G = t.evaluate_grad()
    torch.cuda.synchronize()
    tg = np.arange(n) if n <= sample else np.sort(np.random.default_rng(3).choice(n, sample, replace=False))
    ophi, oE, oG = orc.Tree(w.pos, ncrit).bh(order, w.moments, p, 0.5, targets=tg, want_grad=True)
    ok = within(E.cpu().numpy()[tg], oE, prec, "E") & within(gE.cpu().numpy()[tg], oE, prec, "E beside G")
    ok &= within(phi.cpu().numpy()[tg], ophi, prec, "phi", floor=PHI_FLOOR)
    ok &= within(gphi.cpu().numpy()[tg], ophi, prec, "phi beside G", floor=PHI_FLOOR)
    # the gradient's bounds: as in the gradient parity test
    ok &= within(G.cpu().numpy()[tg], oG, prec, "G", None if prec == FP64 else (2e-6, 1e-4))
    t.close()
    ctx.close()
    assert ok


# two wavefronts a group at 20 001 particles, one at 40 000
@pytest.mark.parametrize("n,ncrit,p,s", [(20001, 32, 8, 1), (40000, 64, 8, 0), (20001, 32, 9, 0), (40000, 64, 9, 2),
                                         (20001, 64, 10, 0), (40000, 64, 10, 1)])
@pytest.mark.parametrize("prec", [FP64, MIXED])
def test_places_by_precision(orc, n, ncrit, p, s, prec):
    w = W.small_random(7000 + n + p, n, s, "plummer", p=p, theta=0.5, ncrit=ncrit)
    print(f"[bh places] n={n} ncrit={ncrit} p={p} s={s} precision={prec}", flush=True)
    _check(orc, w, s, n, ncrit, p, prec, fmm.FMM_M2L_HARMONIC, 300)


@pytest.mark.parametrize("order", [0, 1, 2, 3, 16 + 7])
@pytest.mark.parametrize("p", [5, 8, 10])
@pytest.mark.parametrize("basis", [fmm.FMM_M2L_HARMONIC, fmm.FMM_M2L_FULL])
@pytest.mark.parametrize("n", [130, 2000])
def test_fp64_gradient_written_out(orc, order, p, basis, n):
    w = W.small_mixed(7100, n, order - 16, "plummer", p=p, theta=0.5, ncrit=8) if order >= 16 else \
        W.small_random(7100 + order, n, order, "plummer", p=p, theta=0.5, ncrit=8)
    print(f"[bh fp64 gradient] order={order} p={p} basis={basis} n={n}", flush=True)
    _check(orc, w, w.order, n, 8, p, FP64, basis, 300)


# dipoles at p 9: the one order and p whose gradient waits with places only from the next p on
@pytest.mark.parametrize("n,ncrit", [(130, 8), (2000, 8), (20001, 32), (40000, 64)])
def test_fp64_gradient_dipoles_below_places(orc, n, ncrit):
    w = W.small_random(7200 + n, n, 1, "plummer", p=9, theta=0.5, ncrit=ncrit)
    print(f"[bh fp64 gradient] dipoles p=9 n={n}", flush=True)
    _check(orc, w, 1, n, ncrit, 9, FP64, fmm.FMM_M2L_HARMONIC, 300)
