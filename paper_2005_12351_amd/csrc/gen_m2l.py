"""Writes the unrolled M2L kernels of libfmm.so (a build step).

The multipole-to-local translation (Eq. 8 of Pepper & Fangohr, arXiv
2005.12351) is, for target cell B and source cell A,

    L_n(B) += sum_{s <= |m| <= p - |n|} M_m(A) D_{n+m}(z_B - z_A),  |n| <= p - s,

with D_k the derivatives of 1/r.  In the normalised form used on the GPU
(M~_m = M_m / r_A^|m|, L~_n = L_n r_B^(|n|+1), rho = r_A / r_B) it reads

    L~_n(B) += sum_m D_{n+m}((z_B - z_A) / r_B) * rho^|m| * M~_m(A).

In each generated kernel a 64-wide wavefront works on one tile: lane l owns
the target cell of tile slot l and keeps its local coefficients (or one block
of them) in registers; the wave walks the tile's translation classes, and at
each step every lane streams the multipole of its own source while the
derivative tensor of the class, identical for all lanes, comes through scalar
loads.  The contraction is written out term by term (one fused multiply-add
each), so no index arithmetic is left at run time.  The grid has exactly as
many workgroups as the device keeps resident; the host cuts the concatenated
(tile, output block, entry) work into equally expensive pieces, one per
workgroup, so every SIMD finishes together although the blocks differ in
work by up to 10x.  The wgw waves of a workgroup split each piece's entries
and add their sums in LDS; a piece writes partial sums only where it crosses
a (tile, block) boundary.

Harmonic basis.  The derivative tensor of 1/r is harmonic: for every k,
D_{k+2e_x} + D_{k+2e_y} + D_{k+2e_z} = 0, hence
D_{k+2j e_z} = (-1)^j sum_i C(j,i) D_{k+2i e_x+2(j-i) e_y}.  A multipole
row folded onto the components with m_z <= 1 (done once per cell, as P2M
and M2M write the row) therefore gives the same sums, and the locals, whose
truncation |m| <= p - |n| is the same for n+2e_x, n+2e_y and n+2e_z, obey
the same identity, so only their components with n_z <= 1 are computed and
the rest is rebuilt afterwards.  Order l then holds 2l+1 components instead
of (l+1)(l+2)/2: the irreducible count the paper's Discussion refers to.
The "_h" kernels contract these reduced rows; the term lists are the same
construction restricted to the reduced components.

Matrix cores.  The "_hm" kernels compute the same FP32 harmonic-basis
contraction on the MFMA units.  v_mfma_f32_4x4x1_16b_f32 is a batch of
sixteen 4x4 outer products: block b of the wave gets D[r][c] += A[r] B[c],
with A[r] from lane 4b+r and B[c] from lane 4b+c.  Lane l = 4b+c holds the
scaled multipole coefficient m_j of its own target's source (B) and four
accumulators, the local outputs 4g..4g+3 of its target; the class operand
A[r] = D_{n_{4g+r}+m_j} is the same for every block, so it is broadcast from
one block (CBSZ = 4, ABID = k): a single VGPR holds the operands of sixteen
consecutive multiply-add slots (j, g), gathered per lane from the class's
derivative row through a fixed index table (an index past the tensor reads a
zero for outputs a slot does not reach).  Per slot: 64 targets x 4 outputs
in one instruction, twice the FP32 multiply-add rate of the vector unit.
The rows come through LDS: a lane that loads its own row touches 64 cache
lines an instruction, which kept the address units busier than the matrix
pipe.  Eight lanes that share a row's 128-byte line copy it straight to LDS,
swizzled so that each lane then reads its own row without bank conflicts; the
copies of later chunks land while the current one multiplies, and need no
registers.  What bounds it now is the issue of the 4x4x1 instruction (6.5 to
6.9 ns each per SIMD, 4.8 in a loop of nothing else).  2x10^6 quadrupoles,
theta 0.5, p 10: 1.07 -> 0.81 ms a launch; 100k dipoles, theta 0.3, p 10:
0.384 -> 0.373 ms.

FP64 matrix cores.  For p - s of 8 and 9 the "_f64_h" kernels use
v_mfma_f64_4x4x4_4b_f64, a product of four outputs by four inputs for sixteen
targets: A[i][k] = D_{n_{4g+i}+m} is the same for all targets, so one operand,
gathered from the class's row in LDS through a table of offsets (a zero where
n + m is past the tensor), serves the four instructions of the tile's 64
targets; B holds the multipoles, lane j + 16k the coefficients of target j,
two neighbours a load, so a load touches 16 rows and not 64.  The next
coefficients, and the next entry's rows, load while the current ones multiply.
The instruction reaches 72 TFLOP/s alone, multiply-adds 60 with two waves a
SIMD, and the vector form here 34 (scalar loads of the derivatives, row
gathers); 12 % of the products are padding at p 10, s 1.  100k particles: dipoles,
theta 0.3, p 10: 779 -> 664 us; charges, p 8: 518 -> 427; theta 0.5, p 10: 191 -> 170.

Usage: python gen_m2l.py OUTDIR  -> OUTDIR/m2l_s{0,1,2}_{f32,f64}[_h].hip, m2l_s{0,1,2}_f32_hm.hip
"""
import os
import sys

P_MAX = 10
TILE = 64

# code-shape options (register blocking, scalar-load pipelining, waves per
# workgroup); the defaults are the measured best on gfx950
DEFAULTS = {"acc32": 128, "m32": 64, "acc64": 64, "m64": 32, "dgroup32": 32, "dgroup64": 16, "pipeline": 1,
            "mpre": 0, "launder": 1, "scale_branch": 0, "minwaves": 0, "wgw": 4, "fairprio": 1,
            "mdist": 4}

ROW_LINE = 32           # FP32 coefficients of a 128-byte line: the chunk of the matrix-core kernels
NQ = ROW_LINE // 4      # its float4s
GROUPS64 = 13           # groups of four outputs an FP64 matrix-core block holds


def orders(p):
    out = []
    for k in range(p + 1):
        for nx in range(k, -1, -1):
            for ny in range(k - nx, -1, -1):
                out.append((nx, ny, k - nx - ny))
    return out


def nterms(p):
    return 0 if p < 0 else (p + 1) * (p + 2) * (p + 3) // 6


def idx(n):
    k = sum(n)
    a = n[1] + n[2]
    return nterms(k - 1) + a * (a + 1) // 2 + n[2]


def pad(x, m):
    return (x + m - 1) // m * m


def reduced(mis):
    """The components with n_z <= 1 (the harmonic basis), in storage order."""
    return [n for n in mis if n[2] <= 1]


def split_blocks(nl, max_acc):
    """Fewest contiguous n-ranges [a, b) of nearly equal size with at most
    max_acc accumulators each (every block re-reads the multipole
    coefficients it needs, so fewer blocks means less gather traffic)."""
    nb = max(1, -(-nl // max_acc))
    assert nb <= 16, 'at most 16 output blocks'
    return [(nl * i // nb, nl * (i + 1) // nb) for i in range(nb)]


def gen_kernel(p, s, fp32, opt=None, harmonic=False):
    """One kernel per (p, s, precision).  Work split: blockIdx.x = work item
    (tile, entry range, output row), blockIdx.y = block of output
    coefficients.  Inside a block the needed multipole coefficients are loaded
    into registers in chunks; within a chunk the multiply-adds are emitted in
    bands of equal total derivative order |n| + |m|, so that only one band of
    the (uniform) derivative tensor is live in scalar registers at a time; an
    scheduling barrier (not a memory clobber, so the tensor stays eligible
    for scalar loads) separates the groups so that the compiler cannot hoist
    every scalar load to the top of the loop."""
    T = "float" if fp32 else "double"
    V = "float4" if fp32 else "double2"
    VW = 4 if fp32 else 2
    fma = "__builtin_fmaf" if fp32 else "__builtin_fma"
    suf = "f32" if fp32 else "f64"
    ns = orders(p - s)
    ms = orders(p)[nterms(s - 1):]
    if harmonic:
        ns, ms = reduced(ns), reduced(ms)
    nm = len(ms)
    nl = len(ns)
    nmp = pad(nm, 4)
    nlp = pad(nl, 4)
    nd = pad(nterms(p), 16)
    scw = pad(p + 1, 4)
    opt = dict(DEFAULTS, **(opt or {}))
    max_acc = opt["acc32"] if fp32 else opt["acc64"]
    max_m = opt["m32"] if fp32 else opt["m64"]
    dgroup = opt["dgroup32"] if fp32 else opt["dgroup64"]
    blocks = split_blocks(nl, max_acc)
    name = f"m2l_p{p}_s{s}_{suf}" + ("_h" if harmonic else "")
    L = []
    # minwaves > 0: resident waves per SIMD the register allocation must allow
    wgw = opt["wgw"]
    NT = TILE * wgw
    lb = f"{NT}, {opt['minwaves']}" if opt["minwaves"] else f"{NT}"
    L.append(f"__global__ __launch_bounds__({lb}) void {name}(M2LArgs a)")
    L.append("{")
    L.append(f"    const int lane = threadIdx.x % {TILE};")
    if wgw > 1:
        # the waves of a workgroup split every item's entries and add their
        # partial sums in LDS (in wave order) before one row set is written;
        # the wave index is read from the first lane so that the compiler
        # knows it is uniform (else the piece bounds, class ids and table
        # pointer derived from it leave the scalar unit)
        L.append(f"    const int wv = __builtin_amdgcn_readfirstlane((int)threadIdx.x / {TILE});")
        L.append(f"    __shared__ {T} red[{max(b - a for a, b in blocks)} * {TILE}];")
    L.append(f"    const {T} *__restrict__ Mb = (const {T} *)a.M;")
    L.append(f"    const {T} *__restrict__ Db = (const {T} *)a.D;")
    L.append(f"    const {T} *__restrict__ Sb = (const {T} *)a.sc;")
    L.append("    // this wave's pieces (equal total cost per wave, fixed by the host)")
    L.append("    const int p0 = a.wave_ptr[blockIdx.x], p1 = a.wave_ptr[blockIdx.x + 1];")
    L.append("    for (int item = p0; item < p1; ++item) {")
    L.append("    const int4 w = a.work[item];")
    L.append("    const int blk = w.x >> 24;")
    L.append(f"    {T} *__restrict__ out = ({T} *)a.part + ((size_t)w.w + lane) * {nlp};")
    for bi, (n0, n1) in enumerate(blocks):
        kw = "if" if bi == 0 else "else if"
        L.append(f"    {kw} (blk == {bi}) {{")
        for i in range(n0, n1):
            L.append(f"        {T} c{i} = 0;")
        minord = min(sum(ns[i]) for i in range(n0, n1))
        need = [j for j, m in enumerate(ms) if sum(m) + minord <= p]
        # chunks of the needed m, aligned to the vector width
        chunks, cur = [], []
        for j in need:
            if cur and (len(cur) >= max_m and j % VW == 0):
                chunks.append(cur)
                cur = []
            cur.append(j)
        if cur:
            chunks.append(cur)
        if wgw > 1:
            L.append(f"        const int uspan = w.z - w.y;")
            L.append(f"        const int ub = w.y + uspan * wv / {wgw}, ue = w.y + uspan * (wv + 1) / {wgw};")
            L.append("        for (int u = ub; u < ue; ++u) {")
        else:
            L.append("        for (int u = w.y; u < w.z; ++u) {")
        if opt["fairprio"] and wgw > 1:
            # issue priority falls as the wave works through its entries, so
            # a wave that lags (the younger workgroup's, which loses the
            # age-ordered arbitration) catches up instead of finishing alone
            L.append("            {")
            L.append("                const int stage = (u - ub) * 4 / (ue - ub);")
            L.append("                if (stage == 0) __builtin_amdgcn_s_setprio(3);")
            L.append("                else if (stage == 1) __builtin_amdgcn_s_setprio(2);")
            L.append("                else if (stage == 2) __builtin_amdgcn_s_setprio(1);")
            L.append("                else __builtin_amdgcn_s_setprio(0);")
            L.append("            }")
        L.append("            const int cls = a.ucls[u];")
        # the class tables are read-only for the whole kernel: reading them
        # through the constant address space lets the uniform loads go
        # through the scalar unit into SGPRs (an operand of every FMA)
        L.append(f"            const {T} __attribute__((address_space(4))) *const D = "
                 f"(const {T} __attribute__((address_space(4))) *)(Db + (size_t)cls * {nd});")
        L.append(f"            const {T} __attribute__((address_space(4))) *sc = "
                 f"(const {T} __attribute__((address_space(4))) *)(Sb + (size_t)cls * {scw});")
        L.append(f"            const {T} *__restrict__ Mr = Mb + (size_t)a.usrc[(size_t)u * {TILE} + lane] * {nmp};")
        comps = "xyzw"
        SB = '            __builtin_amdgcn_sched_barrier(0);'

        def mload(ch):
            return [f"            const {V} v{g} = *(const {V} *)(Mr + {g * VW});" for g in sorted(set(j // VW for j in ch))]

        def mscale(ch):
            if opt["scale_branch"]:
                # rho = r_A / r_B is 1 for pairs of one level: skip the scaling then
                out = [f"            {T} m{j} = v{j // VW}.{comps[j % VW]};" for j in ch]
                out.append("            if (sc[1] != 1) {")
                out += [f"                m{j} *= sc[{sum(ms[j])}];" for j in ch]
                out.append("            }")
                return out
            return [f"            const {T} m{j} = v{j // VW}.{comps[j % VW]} * sc[{sum(ms[j])}];" for j in ch]

        def chunk_groups(ch):
            # multiply-adds of this chunk, ordered by derivative index k = n + m
            # (bands of equal |k| are contiguous in the coefficient order),
            # in groups of at most dgroup distinct k, never spanning two bands
            terms = []
            for i in range(n0, n1):
                n = ns[i]
                for j in ch:
                    m = ms[j]
                    if sum(n) + sum(m) > p:
                        continue
                    terms.append((idx((n[0] + m[0], n[1] + m[1], n[2] + m[2])), i, j))
            terms.sort()
            groups, cur, curk = [], [], []
            for k, i, j in terms:
                band = sum(orders(p)[k])
                if curk and k != curk[-1] and (len(curk) >= dgroup or sum(orders(p)[curk[-1]]) != band):
                    groups.append((curk, cur))
                    cur, curk = [], []
                if not curk or curk[-1] != k:
                    curk.append(k)
                cur.append((k, i, j))
            if cur:
                groups.append((curk, cur))
            return groups

        def loads(g):
            base = f"D{g[2]}" if opt["launder"] else "D"
            return [f"            const {T} d{g[2]}_{k} = {base}[{k}];" for k in g[0]]

        def fmas(g):
            return [f"            c{i} = {fma}(d{g[2]}_{k}, m{j}, c{i});" for k, i, j in g[1]]

        mode = opt["pipeline"]
        mpre = opt["mpre"]
        if mpre:
            L.extend(mload(chunks[0]))
        for ci, ch in enumerate(chunks):
            if opt["launder"]:
                # a table pointer per chunk that the compiler cannot prove
                # equal to the previous one: it reloads the derivatives each
                # chunk needs instead of keeping the whole tensor live in
                # scalar registers
                L.append(f"            const {T} __attribute__((address_space(4))) *const D{ci} = D + (size_t)(a.zero * {ci + 1});")
            if not mpre:
                L.extend(mload(ch))
            L.extend(mscale(ch))
            groups = [(ks, ts, ci) for ks, ts in chunk_groups(ch)]
            mid = len(groups) // 2
            nxt = chunks[ci + 1] if ci + 1 < len(chunks) else None
            if mode == 0:
                for gi, g in enumerate(groups):
                    L.append(SB)
                    L.extend(loads(g))
                    L.extend(fmas(g))
                    if mpre and nxt and gi == mid:
                        L.append(SB)
                        L.extend(mload(nxt))
            elif mode == 1:
                # loads of group g+1 are issued before the multiply-adds of group g
                L.append(SB)
                L.extend(loads(groups[0]))
                for gi, g in enumerate(groups):
                    L.append(SB)
                    if gi + 1 < len(groups):
                        L.extend(loads(groups[gi + 1]))
                    L.extend(fmas(g))
                    if mpre and nxt and gi == mid:
                        L.append(SB)
                        L.extend(mload(nxt))
            else:
                # loads of group g+1 are issued half way through the
                # multiply-adds of group g: scalar loads complete out of
                # order, so the wait before group g+1 covers every scalar
                # load in flight; this way only group g+1's are
                L.append(SB)
                L.extend(loads(groups[0]))
                for gi, g in enumerate(groups):
                    f_ = fmas(g)
                    h = len(f_) // 2
                    L.append(SB)
                    L.extend(f_[:h])
                    L.append(SB)
                    if gi + 1 < len(groups):
                        L.extend(loads(groups[gi + 1]))
                    if mpre and nxt and gi == mid:
                        L.extend(mload(nxt))
                    L.append(SB)
                    L.extend(f_[h:])
        L.append("        }")
        if wgw > 1:
            for q in range(wgw):
                last = q == wgw - 1
                L.append(f"        if (wv == {q}) {{")
                for i in range(n0, n1):
                    slot = f"red[{i - n0} * {TILE} + lane]"
                    if q == 0:
                        L.append(f"            {slot} = c{i};")
                    elif not last:
                        L.append(f"            {slot} += c{i};")
                    else:
                        L.append(f"            out[{i}] = {slot} + c{i};")
                L.append("        }")
                if not last:
                    L.append("        __syncthreads();")
            L.append("        __syncthreads();   // red is reused by the next item")
        else:
            for i in range(n0, n1):
                L.append(f"        out[{i}] = c{i};")
        L.append("    }")
    L.append("    }")
    L.append("}")
    launcher = f"""
static hipError_t launch_{name}(const M2LArgs &a, int nwaves, hipStream_t st)
{{
    hipLaunchKernelGGL({name}, dim3(nwaves), dim3({NT}), 0, st, a);
    return hipGetLastError();
}}

static int occ_{name}()
{{
    int per_cu = 0;
    if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, {name}, {NT}, 0) != hipSuccess) return 1;
    return per_cu > 0 ? per_cu : 1;
}}
"""
    fma_per_block = []
    for (n0, n1) in blocks:
        fma_per_block.append(sum(1 for i in range(n0, n1) for m in ms if sum(m) + sum(ns[i]) <= p))
    meta = dict(name=name, nl_pad=nlp, nm_pad=nmp, nd=nd, nblocks=len(blocks), scw=scw,
                blo=[b[0] for b in blocks] + [blocks[-1][1]], bfma=fma_per_block)
    return "\n".join(L) + "\n" + launcher, meta


def mfma_schedule(p, s, mch, dist):
    """Multiply-add slots (j, g) of the harmonic contraction for the matrix
    cores, in issue order, with accumulator copies: a slot whose output group
    was used fewer than `dist` slots before goes to another copy of that
    group's accumulators (added together at the end), so that no MFMA waits
    for the previous one's result.  Returns the chunks of the multipole row
    (lists of j, at most `mch`, starting at multiples of 4) and per chunk the
    slots as (j, g, copy)."""
    ns = reduced(orders(p - s))
    ms = reduced(orders(p)[nterms(s - 1):])
    nl = len(ns)
    ng = (nl + 3) // 4
    chunks = [list(range(c, min(len(ms), c + mch))) for c in range(0, len(ms), mch)]
    out = []
    for ch in chunks:
        queues = {}
        for j in ch:
            for g in range(ng):
                if any(sum(ns[i]) + sum(ms[j]) <= p for i in range(4 * g, min(nl, 4 * g + 4))):
                    queues.setdefault(g, []).append(j)
        last = {}            # (g, copy) -> step of its last use
        ncopy = {g: 1 for g in queues}
        seq, step = [], 0
        while any(queues.values()):
            # the group with the most remaining slots that has a free copy
            best = None
            for g, q in sorted(queues.items(), key=lambda kv: -len(kv[1])):
                if not q:
                    continue
                free = [c for c in range(ncopy[g]) if step - last.get((g, c), -dist) >= dist]
                if free:
                    best = (g, free[0])
                    break
            if best is None:
                g = max((g for g in queues if queues[g]), key=lambda g: len(queues[g]))
                if ncopy[g] < 4:
                    ncopy[g] += 1
                    best = (g, ncopy[g] - 1)
                else:
                    best = (g, min(range(ncopy[g]), key=lambda c: last.get((g, c), -dist)))
            g, c = best
            j = queues[g].pop(0)
            seq.append((j, g, c))
            last[(g, c)] = step
            step += 1
        out.append(seq)
    return chunks, out


def mfma_waves(p, s):
    """Waves per SIMD (= workgroups per CU) of the matrix-core kernels, held
    by the launch bound: what the registers allow with the accumulators (one
    per local output, and copies) beside a chunk of rows and its operands.
    The host cuts the work into that many pieces per CU, so this number also
    fixes the order of the FP32 sums."""
    nl = pad(len(reduced(orders(p - s))), 4)
    return 4 if nl <= 40 else 3 if nl <= 64 else 2


def gen_kernel_mfma(p, s, opt=None):
    """FP32 harmonic-basis M2L on the matrix cores (see the module header).
    Same arguments, work items, waves per workgroup and partial rows as the
    vector kernels (one output block holding every local output)."""
    opt = dict(DEFAULTS, **(opt or {}))
    ns = reduced(orders(p - s))
    ms = reduced(orders(p)[nterms(s - 1):])
    nl, nm = len(ns), len(ms)
    # rows aligned to 128-byte lines: a chunk of 32 coefficients is one line
    nlp, nmp = pad(nl, 4), pad(nm, ROW_LINE)
    nd = pad(nterms(p), 16)
    scw = pad(p + 1, 4)
    zero = nterms(p)          # an entry of every derivative row that is zero (nd > nterms(p))
    assert zero < nd
    ng = (nl + 3) // 4
    assert 4 * ng == nlp
    mch = ROW_LINE           # a chunk is one line of the rows
    chunks, sched = mfma_schedule(p, s, mch, opt["mdist"])
    # operand groups: 16 consecutive slots of a chunk share one VGPR
    groups = []              # per group: list of (j, g, copy)
    for seq in sched:
        for k in range(0, len(seq), 16):
            groups.append(seq[k:k + 16])
    nw = len(groups)
    itab = []
    for grp in groups:
        row = []
        for slot in range(16):
            for r in range(4):
                v = zero
                if slot < len(grp):
                    j, g, _ = grp[slot]
                    i = 4 * g + r
                    if i < nl and sum(ns[i]) + sum(ms[j]) <= p:
                        n, m = ns[i], ms[j]
                        v = idx((n[0] + m[0], n[1] + m[1], n[2] + m[2]))
                row.append(4 * v)      # byte offset in the class's row
        itab.append(row)
    copies = {}
    for seq in sched:
        for j, g, c in seq:
            copies[g] = max(copies.get(g, 0), c + 1)
    wgw = opt["wgw"]
    NT = TILE * wgw
    name = f"m2l_p{p}_s{s}_f32_hm"
    nchunk = len(chunks)
    assert mch == ROW_LINE
    # two chunks in LDS where two workgroups share a CU's 160 KB
    nbuf = 2 if mfma_waves(p, s) == 2 else 1
    assert nbuf == 1 or nchunk >= 3
    # Kernels whose registers the launch bound just allows: the addresses of the
    # permutations and LDS reads are made where they are used (the compiler keeps
    # one a copy and one a quad through the loop otherwise), the class numbers come
    # through the scalar unit, and with three or four waves a SIMD the scales when
    # their entry begins.  Spilled registers cost more than their moves: a reload
    # waits for every copy under way.  us with 28 to 188 bytes spilled / now, theta
    # 0.3, 100k: quadrupoles p 9 307 / 231, octupoles p 8 166 / 141, p 10 319 / 270,
    # charges p 10 376 / 364, dipoles p 8 204 / 197.  The kernels with registers to
    # spare lose 2 to 3 % by it (dipoles p 10 342 / 350).
    tight = nbuf == 1 or nl > 100
    late_scales = nbuf == 1
    L = []
    # operand byte offsets, two 16-bit values per word: group 2k in the low half
    words = []
    for k in range(0, nw, 2):
        lo = itab[k]
        hi = itab[k + 1] if k + 1 < nw else [0] * 64
        words.append([a | (b << 16) for a, b in zip(lo, hi)])
    assert max(max(r) for r in itab) < 65536
    flat = ", ".join(str(v) for w_ in words for v in w_)
    L.append(f"static __device__ const unsigned kIdx_{name}[{len(words) * 64}] = {{{flat}}};")
    L.append(f"__global__ __launch_bounds__({NT}, {mfma_waves(p, s)}) void {name}(M2LArgs a)")
    L.append("{")
    L.append(f"    const int lane = threadIdx.x % {TILE};")
    L.append(f"    const int wv = __builtin_amdgcn_readfirstlane((int)threadIdx.x / {TILE});")
    # the operand index table, read from LDS where a group of slots needs it
    L.append(f"    __shared__ unsigned ixs[{len(words) * 64}];")
    # per wave one or two chunks of the 64 source rows, and the sums of an
    # item's waves when its entries are done
    # (on a line boundary: the swizzled reads flip address bits 4 to 6)
    L.append(f"    __shared__ alignas({4 * ROW_LINE}) float4 area[{max(nbuf * wgw * TILE * NQ, nlp * TILE // 4)}];")
    L.append("    float *const red = (float *)area;")
    if tight:
        L.append("    const int __attribute__((address_space(4))) *const ucls = "
                 "(const int __attribute__((address_space(4))) *)a.ucls;")
    else:
        L.append("    const int32_t *__restrict__ ucls = a.ucls;")
    L.append(f"    for (int k = threadIdx.x; k < {len(words) * 64}; k += {NT}) ixs[k] = kIdx_{name}[k];")
    L.append("    __syncthreads();")
    L.append("    const float *__restrict__ Mb = (const float *)a.M;")
    L.append("    const char *__restrict__ Db = (const char *)a.D;")
    L.append("    const float *__restrict__ Sb = (const float *)a.sc;")
    # copy k of a chunk: eight rows of one line each, straight to LDS (lane i to
    # slot i of the copy's 64); lane i takes quad (i % 8) ^ (i / 8) of row
    # 8k + i / 8, so that the lanes' reads of one quad of their own rows fall
    # on different banks
    L.append(f"    const int sr = lane / {NQ}, sq = lane % {NQ};")
    L.append(f"    const float *const Mq = Mb + 4 * (sq ^ sr);")
    L.append(f"    float4 *const stage = area + wv * {nbuf * TILE * NQ};")
    L.append(f"    const unsigned srd = lds_address(stage + {NQ} * lane + sq);   // quad q at srd ^ 16 q")
    L.append("    const int p0 = a.wave_ptr[blockIdx.x], p1 = a.wave_ptr[blockIdx.x + 1];")
    L.append("    for (int item = p0; item < p1; ++item) {")
    L.append("    const int4 w = a.work[item];")
    L.append(f"    float *__restrict__ out = a.part ? (float *)a.part + ((size_t)w.w + lane) * {nlp} : nullptr;")
    for g in range(ng):
        for c in range(copies.get(g, 1)):
            L.append(f"    f32x4 acc{g}_{c} = {{0.f, 0.f, 0.f, 0.f}};")
    L.append("    const int uspan = w.z - w.y;")
    L.append(f"    const int ub = w.y + uspan * wv / {wgw}, ue = w.y + uspan * (wv + 1) / {wgw};")
    # operand groups of each chunk (first global group index, count)
    gstart, gi = [], 0
    for seq in sched:
        gstart.append(gi)
        gi += (len(seq) + 15) // 16
    ords = sorted(set(sum(m) for m in ms))
    ng0 = (len(sched[0]) + 15) // 16

    def chunk_copies(src, ci, buf):
        # row 8k + sr is the source of lane 8k + sr
        if tight:
            out = ["{", "    int at = 4 * sr;", '    asm volatile("" : "+v"(at));']
            out += [f"    const int src{k} = __builtin_amdgcn_ds_bpermute(at + {4 * (TILE // NQ) * k}, {src});" for k in range(NQ)]
            out += [f"    copy_to_lds(Mq + (size_t)src{k} * {nmp} + {ROW_LINE * ci}, stage + {buf} + {TILE * k});"
                    for k in range(NQ)]
            return out + ["}"]
        return [f"copy_to_lds(Mq + (size_t)__builtin_amdgcn_ds_bpermute(4 * sr + {4 * (TILE // NQ) * k}, {src}) * {nmp} + "
                f"{ROW_LINE * ci}, stage + {buf} + {TILE * k});" for k in range(NQ)]

    def operands(ci, dr, decl, suf=""):
        out = []
        for k in range((len(sched[ci]) + 15) // 16):
            wk = gstart[ci] + k
            word = f"ixs[{(wk // 2) * 64} + lane]"
            half = f"({word} & 0xffffu)" if wk % 2 == 0 else f"({word} >> 16)"
            out.append(f"{decl}w{wk}{suf} = *(const float *)({dr} + {half});")
        return out

    def scales(decl, cls, suf=""):
        ptr = (f"const float __attribute__((address_space(4))) *sp{suf} = "
               f"(const float __attribute__((address_space(4))) *)(Sb + (size_t){cls} * {scw});")
        return [ptr] + [f"{decl}s{o}{suf} = sp{suf}[{o}];" for o in ords]

    def mfmas(ci):
        ch, seq = chunks[ci], sched[ci]
        out = []
        for j in ch:
            out.append(f"const float m{j} = v{j // 4}[{j % 4}] * s{sum(ms[j])};")
        for k in range((len(seq) + 15) // 16):
            wk = gstart[ci] + k
            for slot, (j, g, c) in enumerate(seq[16 * k:16 * k + 16]):
                out.append(f"acc{g}_{c} = __builtin_amdgcn_mfma_f32_4x4x1f32(w{wk}, m{j}, acc{g}_{c}, 4, {slot}, 0);")
        return out

    def emit(lines, ind):
        L.extend(" " * ind + x for x in lines)

    SB = "__builtin_amdgcn_sched_barrier(0);"
    CH4 = TILE * NQ          # float4s of a chunk
    # LDS offset of chunk ci of the entry `ahead` entries on: its number among
    # all chunks modulo the buffers (flip: this entry's first, 0 or CH4)
    flips = nbuf == 2 and nchunk % 2 == 1

    def buf(ci, ahead=0):
        if nbuf == 1:
            return "0"
        k = (ci + ahead * nchunk) % 2
        return f"({CH4} - flip)" if flips and k else "flip" if flips else str(CH4 * k)

    # the first entry's sources, operands, scales and first chunks
    emit(["int src = 0;"] + [f"float w{gstart[0] + k};" for k in range(ng0)] +
         ([] if late_scales else [f"float s{o};" for o in ords]), 4)
    if flips:
        emit(["int flip = 0;"], 4)
    emit(["if (ub < ue) {"], 4)
    emit([f"src = a.usrc[(size_t)ub * {TILE} + lane];", "const int cls = ucls[ub];",
         f"const char *__restrict__ Dr = Db + (size_t)cls * {nd * 4};"] + operands(0, "Dr", "") +
         ([] if late_scales else scales("", "cls")) + [SB], 8)
    for ci in range(nbuf):
        emit(chunk_copies("src", ci, buf(ci)), 8)
    emit(["}"], 4)
    emit(["for (int u = ub; u < ue; ++u) {"], 4)
    if opt["fairprio"]:
        emit(["{",
              "    const int stage_ = (u - ub) * 4 / (ue - ub);",
              "    if (stage_ == 0) __builtin_amdgcn_s_setprio(3);",
              "    else if (stage_ == 1) __builtin_amdgcn_s_setprio(2);",
              "    else if (stage_ == 2) __builtin_amdgcn_s_setprio(1);",
              "    else __builtin_amdgcn_s_setprio(0);",
              "}"], 8)
    emit(["// the entry loaded ahead (this one again at the end of the range)",
          "const int un = u + 1 < ue ? u + 1 : u;",
          "const int cls = ucls[u], clsn = ucls[un];",
          f"const char *__restrict__ Dr = Db + (size_t)cls * {nd * 4};",
          f"const char *__restrict__ Drn = Db + (size_t)clsn * {nd * 4};"], 8)
    if late_scales:
        emit(scales("const float ", "cls"), 8)
    # where the operands are loaded: with registers to spare all but the first
    # chunk's one phase after their registers fall free, the next entry's in
    # the second phase (the later ones are too short to cover the loads);
    # otherwise each in the phase before its use
    early = nbuf == 2 and nl < 100
    ahead = 1 if early else nchunk - 1
    for ci in range(nchunk):
        # this chunk's rows are in LDS: each lane reads its own, then the copies
        # of the chunk nbuf later are issued over them and land while this and
        # the chunks between multiply.  Waits are spelled out: all but the
        # NQ copies of the chunk between are done before the reads, the reads
        # before the next copies, which are the phase's last memory operations.
        quads = sorted(set(j // 4 for j in chunks[ci]))
        emit([SB, f"wait_copies<{NQ * (nbuf - 1)}>();", SB] + [f"f32x4 v{q};" for q in quads], 8)
        outs = ", ".join(f'"=&v"(v{q})' for q in quads)
        ins = ", ".join(f'"v"(({"rd" if tight else "srd"} + 16 * {buf(ci)}) ^ {16 * (q - NQ * ci)}u)' for q in quads)
        code = "".join(f"ds_read_b128 %{k}, %{k + len(quads)}\\n" for k in range(len(quads))) + "s_waitcnt lgkmcnt(0)"
        read = [f'asm volatile("{code}" : {outs} : {ins} : "memory");']
        if tight:
            read = ["{", "    unsigned rd = srd;", '    asm volatile("" : "+v"(rd));', "    " + read[0], "}"]
        emit(read + [SB], 8)
        if ci == 0:
            emit([f"const int srcn = a.usrc[(size_t)un * {TILE} + lane];"], 8)
        for cj in range(1, nchunk):
            if ci == (min(cj - 1, 1) if early else cj - 1):
                emit(operands(cj, "Dr", "const float "), 8)
        if ci == ahead:
            emit(operands(0, "Drn", "const float ", "n") +
                 ([] if late_scales else scales("const float ", "clsn", "n")), 8)
        cn, an = (ci + nbuf) % nchunk, (ci + nbuf) // nchunk
        emit([SB] + chunk_copies("srcn" if an else "src", cn, buf(cn, an)), 8)
        emit(mfmas(ci), 8)
    emit(["src = srcn;"] + [f"w{gstart[0] + k} = w{gstart[0] + k}n;" for k in range(ng0)] +
         ([] if late_scales else [f"s{o} = s{o}n;" for o in ords]), 8)
    if flips:
        emit([f"flip = {CH4} - flip;"], 8)
    emit(["}"], 4)
    for g in range(ng):
        for c in range(1, copies.get(g, 1)):
            L.append(f"    acc{g}_0 += acc{g}_{c};")
    # the last copies (of an entry loaded ahead that does not come) are done
    # before the area is used for the sums
    L.append("    wait_copies<0>();")
    L.append("    __syncthreads();")
    for q in range(wgw):
        last = q == wgw - 1
        L.append(f"    if (wv == {q}) {{")
        for g in range(ng):
            for r in range(4):
                i = 4 * g + r
                slot_ = f"red[{i} * {TILE} + lane]"
                if q == 0:
                    L.append(f"        {slot_} = acc{g}_0[{r}];")
                elif not last:
                    L.append(f"        {slot_} += acc{g}_0[{r}];")
                else:
                    L.append(f"        out[{i}] = {slot_} + acc{g}_0[{r}];")
        L.append("    }")
        if not last:
            L.append("    __syncthreads();")
    L.append("    __syncthreads();   // red is reused by the next item")
    L.append("    }")
    L.append("}")
    launcher = f"""
static hipError_t launch_{name}(const M2LArgs &a, int nwaves, hipStream_t st)
{{
    hipLaunchKernelGGL({name}, dim3(nwaves), dim3({NT}), 0, st, a);
    return hipGetLastError();
}}

static int occ_{name}()
{{
    int per_cu = 0;
    if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, {name}, {NT}, 0) != hipSuccess) return 1;
    return per_cu > 0 ? per_cu : 1;
}}
"""
    nslots = sum(len(q) for q in sched)
    meta = dict(name=name, nl_pad=nlp, nm_pad=nmp, nd=nd, nblocks=1, scw=scw, blo=[0, nl], bfma=[4 * nslots])
    return "\n".join(L) + "\n" + launcher, meta


def mfma64_pays(p, s):
    """FP64 harmonic contractions the matrix cores take: two blocks of outputs,
    p - s = 8 and 9.  With fewer outputs one vector block holds them all and the
    padding of the tiles costs more than the unit gives (100k particles, theta
    0.5, p 7: 76 us vector, 89 matrix; p 6: 61 and 66; p 4: 35 and 40); with more
    (p - s = 10) a third block reads the rows again, and two blocks of 16 groups
    leave no registers (10k: 75.5 us vector, 80 matrix; 300k: 887 and 944)."""
    return 4 * GROUPS64 + 12 < len(reduced(orders(p - s))) <= 8 * GROUPS64


def mfma64_blocks(p, s):
    """Output blocks of the FP64 matrix-core kernels: ranges of groups of four
    outputs, at most GROUPS64 (two accumulation registers a group and
    sixteen targets)."""
    ng = (len(reduced(orders(p - s))) + 3) // 4
    nb = -(-ng // GROUPS64)
    return [(ng * i // nb, ng * (i + 1) // nb) for i in range(nb)]


def mfma64_steps(p, s, g0, g1):
    """Tiles of a block in issue order: [(Q, e, [g, ...])].  Step (Q, e) multiplies
    the coefficients 8Q + 2k + e, k = 0..3 (a lane loads two neighbours at once),
    into the groups g that any of them reaches."""
    ns = reduced(orders(p - s))
    ms = reduced(orders(p)[nterms(s - 1):])
    out = []
    for Q in range((len(ms) + 7) // 8):
        for e in (0, 1):
            js = [8 * Q + 2 * k + e for k in range(4) if 8 * Q + 2 * k + e < len(ms)]
            gs = [g for g in range(g0, g1)
                  if any(sum(ns[i]) + sum(ms[j]) <= p for i in range(4 * g, min(len(ns), 4 * g + 4)) for j in js)]
            if gs:
                out.append((Q, e, gs))
    return out


def gen_kernel_mfma64(p, s, opt=None):
    """FP64 harmonic contraction on the matrix cores (see the module's text)."""
    opt = dict(DEFAULTS, **(opt or {}))
    ns = reduced(orders(p - s))
    ms = reduced(orders(p)[nterms(s - 1):])
    nl, nm = len(ns), len(ms)
    nlp, nmp, nd, scw = pad(nl, 4), pad(nm, 8), pad(nterms(p), 16), pad(p + 1, 4)
    blocks = mfma64_blocks(p, s)
    wgw = opt["wgw"]
    NT = TILE * wgw
    name = f"m2l_p{p}_s{s}_f64_h"
    ND = -(-nd // TILE)          # derivative row: registers a lane
    NS = -(-nmp // TILE)         # scale row
    # byte offsets of the operand A of every tile: [tile / 4][lane % 4 + 4 (lane / 16)][tile % 4]
    zero = nd
    tab, first = [], []
    for g0, g1 in blocks:
        first.append(len(tab) // 64)
        tiles = [(Q, e, g) for Q, e, gs in mfma64_steps(p, s, g0, g1) for g in gs]
        for b in range(0, len(tiles), 4):
            for pos in range(16):
                i, kk = pos % 4, pos // 4
                for x in range(4):
                    off = zero
                    if b + x < len(tiles):
                        Q, e, g = tiles[b + x]
                        j, n = 8 * Q + 2 * kk + e, 4 * g + i
                        if j < nm and n < nl and sum(ns[n]) + sum(ms[j]) <= p:
                            off = idx(tuple(a + c for a, c in zip(ns[n], ms[j])))
                    tab.append(8 * off)
    assert max(tab) < 65536
    red = max(g1 - g0 for g0, g1 in blocks) * 4 * TILE
    L = []
    L.append(f"static __device__ const __align__(8) unsigned short tab_{name}[{len(tab)}] = {{{','.join(map(str, tab))}}};")
    L.append(f"static __device__ const unsigned char ord_{name}[{nmp}] = "
             f"{{{','.join(str(sum(ms[j])) if j < nm else '0' for j in range(nmp))}}};")
    L.append(f"__global__ __launch_bounds__({NT}, 2) void {name}(M2LArgs a)")
    L.append("{")
    L.append(f"    __shared__ double red[{red}];")
    L.append(f"    __shared__ double drow[{wgw}][{nd + 1}];")
    L.append(f"    __shared__ __align__(16) double srow[{wgw}][{nmp}];")
    L.append(f"    __shared__ __align__(16) unsigned short tab[{len(tab)}];")
    L.append(f"    const int lane = threadIdx.x % {TILE};")
    L.append(f"    const int wv = __builtin_amdgcn_readfirstlane((int)threadIdx.x / {TILE});")
    L.append("    const int col = lane & 15, kk = lane >> 4, pos = (lane & 3) + 4 * kk;")
    L.append(f"    for (int i = threadIdx.x; i < {len(tab) // 4}; i += {NT}) ((ushort4 *)tab)[i] = ((const ushort4 *)tab_{name})[i];")
    L.append(f"    if (lane == 0) drow[wv][{zero}] = 0.0;")
    L.append("    __syncthreads();")
    L.append("    const double *__restrict__ Mb = (const double *)a.M;")
    L.append("    const double *__restrict__ Db = (const double *)a.D;")
    L.append("    const double *__restrict__ Sb = (const double *)a.sc;")
    L.append("    const char *const dl = (const char *)drow[wv];")
    L.append("    const int p0 = a.wave_ptr[blockIdx.x], p1 = a.wave_ptr[blockIdx.x + 1];")
    L.append("    for (int item = p0; item < p1; ++item) {")
    L.append("    const int4 w = a.work[item];")
    L.append("    const int blk = w.x >> 24;")
    L.append(f"    double *__restrict__ out = (double *)a.part + (size_t)w.w * {nlp};")
    L.append("    const int uspan = w.z - w.y;")
    L.append(f"    const int ub = w.y + uspan * wv / {wgw}, ue = w.y + uspan * (wv + 1) / {wgw};")
    SB = "            __builtin_amdgcn_sched_barrier(0);"

    def rows(Q, suf, ptr):
        return [f"            {'const ' if suf != 'N' else ''}{'double2 ' if suf != 'N' else ''}v{suf}_{x} = *(const double2 *)({ptr}{x} + {8 * Q});"
                for x in range(4)]

    for bi, (g0, g1) in enumerate(blocks):
        steps = mfma64_steps(p, s, g0, g1)
        L.append(f"    {'if' if bi == 0 else 'else if'} (blk == {bi}) {{")
        for g in range(g0, g1):
            L.append("        double " + ", ".join(f"c{g}_{x} = 0" for x in range(4)) + ";")
        L.append("        if (ub < ue) {")
        # the first entry's operands
        L.append("        double2 vN_0, vN_1, vN_2, vN_3;")
        L.append(f"        double dn[{ND}], sn[{NS}];")

        def fetch_src(u):
            return [f"            const double *r{x} = Mb + (size_t)a.usrc[(size_t){u} * {TILE} + {16 * x} + col] * {nmp} + 2 * kk;"
                    for x in range(4)]

        def fetch_rows(u):
            o = [f"            const int cls = a.ucls[{u}];"]
            for x in range(ND):
                o.append(f"            dn[{x}] = Db[(size_t)cls * {nd} + min(lane + {TILE * x}, {nd - 1})];")
            for x in range(NS):
                o.append(f"            sn[{x}] = Sb[(size_t)cls * {scw} + ord_{name}[min(lane + {TILE * x}, {nmp - 1})]];")
            return o

        L.append("        {")
        L.extend(fetch_src("ub"))
        L.extend(rows(steps[0][0], "N", "r"))
        L.extend(fetch_rows("ub"))
        L.append("        }")
        L.append("        for (int u = ub; u < ue; ++u) {")
        # this entry's rows to LDS: the wave's own, in order with its reads
        L.append("            __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, \"wavefront\");")
        L.append("            __builtin_amdgcn_wave_barrier();")
        for x in range(ND):
            c = f"if (lane + {TILE * x} < {nd}) " if TILE * (x + 1) > nd else ""
            L.append(f"            {c}drow[wv][lane + {TILE * x}] = dn[{x}];")
        for x in range(NS):
            c = f"if (lane + {TILE * x} < {nmp}) " if TILE * (x + 1) > nmp else ""
            L.append(f"            {c}srow[wv][lane + {TILE * x}] = sn[{x}];")
        L.append("            __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, \"wavefront\");")
        L.append("            __builtin_amdgcn_wave_barrier();")
        L.append("            const int un = min(u + 1, ue - 1);   // the next entry (the last: itself again)")
        L.extend(fetch_src("u"))
        L.extend(x.replace("const double *r", "const double *q") for x in fetch_src("un"))
        L.append("            {")
        L.extend(fetch_rows("un"))
        L.append("            }")
        Qs = sorted(set(Q for Q, _, _ in steps))
        L.extend(f"            const double2 v{Qs[0]}_{x} = vN_{x};" for x in range(4))
        tile = 0
        for Q in Qs:
            nxt = Qs[Qs.index(Q) + 1] if Q != Qs[-1] else None
            L.append(SB)
            if nxt is not None:
                L.extend(rows(nxt, str(nxt), "r"))
            else:
                L.extend(rows(Qs[0], "N", "q"))
            L.append(f"            const double2 s{Q} = *(const double2 *)&srow[wv][{8 * Q} + 2 * kk];")
            for _, e, gs in [st for st in steps if st[0] == Q]:
                comp = "xy"[e]
                for x in range(4):
                    L.append(f"            const double b{Q}{comp}_{x} = v{Q}_{x}.{comp} * s{Q}.{comp};")
                for g in gs:
                    if tile % 4 == 0:
                        L.append(f"            const ushort4 t{tile // 4} = *(const ushort4 *)&tab[{(first[bi] + tile // 4) * 64} + 4 * pos];")
                    L.append(f"            const double a{tile} = *(const double *)(dl + t{tile // 4}.{'xyzw'[tile % 4]});")
                    for x in range(4):
                        L.append(f"            c{g}_{x} = __builtin_amdgcn_mfma_f64_4x4x4f64(a{tile}, b{Q}{comp}_{x}, c{g}_{x}, 0, 0, 0);")
                    tile += 1
        L.append("        }")
        L.append("        }")
        # the waves' sums, in wave order: row 4 (g - g0) + lane / 16, target 16 x + lane % 16
        for q in range(wgw):
            L.append(f"        if (wv == {q}) {{")
            for g in range(g0, g1):
                for x in range(4):
                    slot = f"red[{(g - g0) * 4 * TILE} + kk * {TILE} + {16 * x} + col]"
                    if q == 0:
                        L.append(f"            {slot} = c{g}_{x};")
                    elif q < wgw - 1:
                        L.append(f"            {slot} += c{g}_{x};")
                    else:
                        L.append(f"            out[(size_t)({16 * x} + col) * {nlp} + {4 * g} + kk] = {slot} + c{g}_{x};")
            L.append("        }")
            L.append("        __syncthreads();")
        L.append("    }")
    L.append("    }")
    L.append("}")
    launcher = f"""
static hipError_t launch_{name}(const M2LArgs &a, int nwaves, hipStream_t st)
{{
    hipLaunchKernelGGL({name}, dim3(nwaves), dim3({NT}), 0, st, a);
    return hipGetLastError();
}}

static int occ_{name}()
{{
    int per_cu = 0;
    if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, {name}, {NT}, 0) != hipSuccess) return 1;
    return per_cu > 0 ? per_cu : 1;
}}
"""
    work = [16 * sum(len(gs) for _, _, gs in mfma64_steps(p, s, g0, g1)) for g0, g1 in blocks]
    meta = dict(name=name, nl_pad=nlp, nm_pad=nmp, nd=nd, nblocks=len(blocks), scw=scw,
                blo=[4 * g0 for g0, _ in blocks] + [nl], bfma=work)
    return "\n".join(L) + "\n" + launcher, meta


def gen_file(s, fp32, opt=None, harmonic=False, mfma=False):
    suf = ("f32" if fp32 else "f64") + ("_h" if harmonic else "") + ("m" if mfma else "")
    parts = ["// Generated by gen_m2l.py; do not edit.", "#include <algorithm>", '#include "fmm_internal.h"', ""]
    if mfma:
        parts.append("typedef float f32x4 __attribute__((ext_vector_type(4)));")
        parts.append("")
        parts.append("""// 16 bytes a lane from global memory to LDS (the lanes' data back to back from `lds`, the same for the whole wave)
static __device__ __forceinline__ void copy_to_lds(const float *g, float4 *lds)
{
    __builtin_amdgcn_global_load_lds((const __attribute__((address_space(1))) void *)g,
                                     (__attribute__((address_space(3))) void *)lds, 16, 0, 0);
}
static __device__ __forceinline__ unsigned lds_address(const float4 *p)
{
    return (unsigned)(size_t)(const __attribute__((address_space(3))) void *)p;
}
// s_waitcnt vmcnt(N): all but the wave's last N copies and loads are done
template <int N>
static __device__ __forceinline__ void wait_copies()
{
    static_assert(N < 16, "vmcnt's low bits");
    __builtin_amdgcn_s_waitcnt(0x0f70 | N);
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}""")
    metas = []
    for p in range(s + 1, P_MAX + 1):
        if mfma:
            code, meta = gen_kernel_mfma(p, s, opt)
        elif harmonic and not fp32 and mfma64_pays(p, s):
            code, meta = gen_kernel_mfma64(p, s, opt)
        else:
            code, meta = gen_kernel(p, s, fp32, opt, harmonic)
        parts.append(code)
        metas.append((p, meta))
    parts.append(f"bool m2l_lookup_s{s}_{suf}(int p, M2LVariant *v)")
    parts.append("{")
    parts.append("    switch (p) {")
    for p, m in metas:
        blo = ", ".join(str(x) for x in m["blo"] + [0] * (17 - len(m["blo"])))
        bf = ", ".join(str(x) for x in m["bfma"] + [0] * (16 - len(m["bfma"])))
        parts.append(f"    case {p}: *v = M2LVariant{{launch_{m['name']}, occ_{m['name']}, {m['nl_pad']}, {m['nm_pad']}, "
                     f"{m['nd']}, {m['nblocks']}, {{{blo}}}, {{{bf}}}}}; return true;")
    parts.append("    default: return false;")
    parts.append("    }")
    parts.append("}")
    return "\n".join(parts) + "\n"


def main(outdir, opt=None):
    os.makedirs(outdir, exist_ok=True)
    written = []
    for s in (0, 1, 2, 3):
        for fp32, h, mf in ((True, False, False), (False, False, False), (True, True, False), (False, True, False),
                            (True, True, True)):
            fn = os.path.join(outdir, f"m2l_s{s}_{'f32' if fp32 else 'f64'}{'_h' if h else ''}{'m' if mf else ''}.hip")
            txt = gen_file(s, fp32, opt, h, mf)
            old = open(fn).read() if os.path.exists(fn) else None
            if old != txt:
                with open(fn, "w") as f:
                    f.write(txt)
            written.append(fn)
    return written


if __name__ == "__main__":
    main(sys.argv[1] if len(sys.argv) > 1 else "_build/gen")
