"""Writes the tables of the M2M and L2L shifts (a build step).

In the normalised form of the expansions (M~_n = M_n / r^|n|, L~_n = L_n
r^(|n|+1)) moving one between a parent and its child of octant c (Eq. 4 of
Pepper & Fangohr, arXiv 2005.12351, read with new minus old centre; the Taylor
shift of the locals) multiplies by a fixed matrix:

    M2M  M~_n(P) += 2^-|n| sum_{m <= n} prod_d (-s_d)^(n_d - m_d) / (n_d - m_d)! M~_m(C),
    L2L  L~_n(C) += sum_a prod_d s_d^a_d / a_d! 2^-(|n+a|+1) L~_{n+a}(P),

with s_d = +1 in the child's upper half of axis d and -1 in its lower.  The sign
of an entry depends on the octant only through the parities x of n - m (of a):
prod_d (-1)^(x_d c_d), a character of the octant.  So one matrix serves all
octants: M2M contracts, for every class x, the entries of that class with the
children's rows summed under character x, and L2L sums each class once and
combines the eight class sums under the characters (both eight-point
Walsh-Hadamard transforms).

Harmonic basis: rows hold the components with third index <= 1.  A multipole
row is lifted with zeros, shifted and folded (component (a, b, r + 2j) goes to
(a + 2i, b + 2(j - i), r) with (-1)^j C(j, i)); a local row's other components
are rebuilt by the same weights before the shift.  Both keep parities, so the
products are matrices of the same form.

Entries of (output h, class x) lie together, by input, so an expansion that
starts at order s (M2M) or ends at order q (L2L) takes a suffix or a prefix of
them; the matrices do not depend on p.  Computed in rationals.

Usage: python gen_shift.py OUTDIR -> OUTDIR/shift_tables.h
"""
import os
import sys
from fractions import Fraction
from math import comb, factorial

P_MAX = 10


def orders(p):
    return [(x, y, k - x - y) for k in range(p + 1) for x in range(k, -1, -1) for y in range(k - x, -1, -1)]


def folded(n):
    """(component, weight) pairs that component n folds onto"""
    j, r = n[2] // 2, n[2] % 2
    return [((n[0] + 2 * i, n[1] + 2 * (j - i), r), (-1) ** j * comb(j, i)) for i in range(j + 1)]


def matrices(harmonic):
    """{(out, in): value} of M2M and L2L over all components up to P_MAX"""
    full = orders(P_MAX)
    comps = [n for n in full if not harmonic or n[2] <= 1]
    pos = {n: i for i, n in enumerate(comps)}
    m2m, l2l = {}, {}

    def add(m, o, i, v):
        if v:
            m[(o, i)] = m.get((o, i), Fraction(0)) + v

    for n in full:
        outs = folded(n) if harmonic else [(n, 1)]
        for m in ((a, b, c) for a in range(n[0] + 1) for b in range(n[1] + 1) for c in range(n[2] + 1)):
            if m not in pos:
                continue
            v = Fraction(1, 2 ** sum(n))
            for d in range(3):
                v /= factorial(n[d] - m[d])
            for o, w in outs:
                add(m2m, pos[o], pos[m], w * v)
    for n in comps:
        for k in full:
            a = [k[d] - n[d] for d in range(3)]
            if min(a) < 0:
                continue
            # s_d^a_d = (-1)^a_d (-1)^(a_d c_d): the first factor is the entry's
            v = Fraction((-1) ** sum(a), 2 ** (sum(k) + 1))
            for d in range(3):
                v /= factorial(a[d])
            for i, w in (folded(k) if harmonic else [(k, 1)]):
                add(l2l, pos[n], pos[i], w * v)
    return comps, m2m, l2l


def entries(comps, mat):
    """(inputs, values, offsets): the entries of (output h, class x) by input;
    offsets[8 h + x][k], k = 0..P_MAX + 1, ends those with an input of order < k"""
    n = len(comps)
    par = [(c[0] & 1) << 2 | (c[1] & 1) << 1 | (c[2] & 1) for c in comps]
    rows = [[[] for _ in range(8)] for _ in range(n)]
    for (o, i), v in mat.items():
        if v:
            rows[o][par[o] ^ par[i]].append((i, v))
    idx, val, off = [], [], []
    for h in range(n):
        for x in range(8):
            ent = sorted(rows[h][x])
            off.append([len(idx) + sum(1 for i, _ in ent if sum(comps[i]) < k) for k in range(P_MAX + 2)])
            idx += [i for i, _ in ent]
            val += [float(v) for _, v in ent]
    assert len(idx) < 65536
    return idx, val, off


def table(name, comps, mat):
    idx, val, off = entries(comps, mat)
    return [f"static __device__ const uint16_t k{name}_idx[{len(idx)}] = {{{','.join(map(str, idx))}}};",
            f"static __device__ const double k{name}_val[{len(val)}] = {{{','.join(map(repr, val))}}};",
            f"static __device__ const uint16_t k{name}_off[{len(off)}][{P_MAX + 2}] = {{"
            + ",".join("{" + ",".join(map(str, o)) + "}" for o in off) + "};"]


def main(outdir):
    os.makedirs(outdir, exist_ok=True)
    parts = ["// Generated by gen_shift.py; do not edit.", "#pragma once", "#include <cstdint>", "", f"constexpr int kShiftOrders = {P_MAX};"]
    for harm in (True, False):
        comps, m2m, l2l = matrices(harm)
        parts += table("M2M" + ("H" if harm else "F"), comps, m2m)
        parts += table("L2L" + ("H" if harm else "F"), comps, l2l)
    fn = os.path.join(outdir, "shift_tables.h")
    txt = "\n".join(parts) + "\n"
    old = open(fn).read() if os.path.exists(fn) else None
    if old != txt:
        with open(fn, "w") as f:
            f.write(txt)


if __name__ == "__main__":
    main(sys.argv[1] if len(sys.argv) > 1 else "_build/gen")
