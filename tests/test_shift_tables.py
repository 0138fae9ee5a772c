"""The M2M and L2L tables (csrc/gen_shift.py), used as the kernels use them,
against the oracle's shifts: every octant, both bases, every cut by order."""
import os
import sys

import numpy as np
import pytest

from tests.test_oracle_reduced import fold, rebuild

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2005_12351_amd", "csrc")


@pytest.fixture(scope="module")
def tables():
    sys.path.insert(0, CSRC)
    import gen_shift
    sys.path.remove(CSRC)
    out = {}
    for harm in (True, False):
        comps, m2m, l2l = gen_shift.matrices(harm)
        out[harm] = comps, gen_shift.entries(comps, m2m), gen_shift.entries(comps, l2l)
    return out


def _char(x, c):
    return -1.0 if bin(x & c).count("1") & 1 else 1.0


def _product(tab, h, x, lo, hi, src):
    """class sum of output h, and the sum of its terms' magnitudes"""
    idx, val, off = tab
    e = range(off[8 * h + x][lo], off[8 * h + x][hi])
    t = [val[i] * src[idx[i]] for i in e]
    return sum(t), sum(map(abs, t))


def _offset(c):
    return np.array([(1 if c & 4 else -1), (1 if c & 2 else -1), (1 if c & 1 else -1)]) * 0.25


# at most 8 x 18 terms (M2M) or 8 x 56 (L2L) an output and as many in the
# oracle: (2 x 448 + 50) x 1.2e-16 < 2e-13 of the magnitudes' sum, which the
# fold and the rebuild (weights up to 10, 21 terms) may raise tenfold
TOL = 2e-12


@pytest.mark.parametrize("harm", [True, False])
@pytest.mark.parametrize("p,s", [(1, 0), (2, 1), (5, 2), (4, 3), (8, 1), (10, 0), (10, 3)])
def test_shift_tables(orc, tables, harm, p, s):
    comps, m2m, l2l = tables[harm]
    rng = np.random.default_rng(100 * p + s)
    q = p - s
    order = np.array([sum(orc.multi_index(i)) for i in range(orc.nterms(p))])
    outs = [h for h, c in enumerate(comps) if s <= sum(c) <= p]
    pos = [orc.index(*c) for c in comps]
    # M2M of children in some octants together (orders below s absent)
    for kids in ([0, 1, 2, 3, 4, 5, 6, 7], [5], [2, 7]):
        rows = {c: rng.standard_normal(orc.nterms(p)) * (order >= s) for c in kids}
        ref = np.zeros(orc.nterms(p))
        W = np.zeros((8, len(comps)))
        for c, m in rows.items():
            if harm:
                m = fold(orc, m, p)
            ref += orc.m2m(p, _offset(c), m * 0.25 ** order, np.zeros(3)) / 0.5 ** order
            for h in range(len(comps)):
                if sum(comps[h]) <= p:
                    for x in range(8):
                        W[x, h] += _char(x, c) * m[pos[h]]
        ref = fold(orc, ref, p) if harm else ref
        for h in outs:
            r = [_product(m2m, h, x, s, -1, W[x]) for x in range(8)]
            scale = max(sum(b for _, b in r), np.abs(ref).max())
            assert abs(sum(a for a, _ in r) - ref[pos[h]]) <= TOL * scale
    # L2L of one row to each octant
    lo = order[:orc.nterms(q)]
    L = rng.standard_normal(orc.nterms(q))
    src = np.zeros(len(comps))
    if harm:
        L = rebuild(orc, L, q)
    for h, c in enumerate(comps):
        if sum(c) <= q:
            src[h] = L[pos[h]]
    for c in range(8):
        ref = orc.l2l(p, s, np.zeros(3), L / 0.5 ** (lo + 1.0), _offset(c)) * 0.25 ** (lo + 1.0)
        for h in range(len(comps)):
            if sum(comps[h]) > q:
                continue
            r = [_product(l2l, h, x, 0, q + 1, src) for x in range(8)]
            v = sum(_char(x, c) * a for x, (a, _) in enumerate(r))
            scale = max(sum(b for _, b in r), np.abs(ref).max())
            assert abs(v - ref[pos[h]]) <= TOL * scale
