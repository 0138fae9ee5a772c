// Multipolar Barnes-Hut evaluation kernel (Section 3.2 of Pepper & Fangohr,
// arXiv 2005.12351), shared by bh.hip (potential and field) and bh_grad.hip
// (with the field gradient): every particle walks the tree from the root; a
// cell that satisfies r_A < theta |x - z_A| (Eq. 12; r = half the side, z =
// geometric centre) and does not contain the particle contributes through
// M2P (Eq. 6), an unaccepted leaf through direct interaction, any other cell
// is opened.
//
// GPU layout: one wavefront = 64 consecutive particles in Morton order, which
// are spatially close.  The wave walks the union of its particles' traversals
// with an LDS stack of (cell, lane mask); each lane takes its own acceptance
// decision, in FP64 with the same rounding sequence as the definition above,
// so every particle accepts exactly the cells it would accept alone and sees
// them in the same depth-first order.  The leaf's sources are identical for
// all lanes and are read through scalar loads.
//
// What bounds it is the vector issue of the M2P evaluation (about 600
// operations at p 6), which half the lanes sat out: neighbours accept the same
// regions at different cells, one the parent, the other its children.  So in
// the harmonic basis an accepted cell's row is copied to one of kSlots places
// in LDS and each accepting lane only marks the place; when the places run out
// every lane evaluates the lowest place it has marked, in rounds, as long as
// most lanes take part.  A lane then still evaluates its own cells with the
// same operations; its sums add up in another order (FP64).  The places cost
// LDS and registers, which the M2P has to be long enough to repay: see
// bh_places_from.  Otherwise each cell is evaluated as it is accepted, its row
// through scalar loads.
//
// A small system fills few wavefronts and then waits for the longest: `split`
// of them share a group of particles.  All walk the cells above level
// kOwnLevel; of those and of that level's each takes the cells (and all below
// them) whose index has its residue.  bh_reduce_kernel adds their sums in order.
#pragma once
#include <cmath>

#include "fmm_internal.h"
#include "pair_kernels.h"
#include "bh_m2p.h"

struct BHGeo {
    double lo[3];
    double h;
};

struct BHArgs {
    const DevCell *cells;
    const double *xs;       // sorted positions, SoA
    const double *m64;      // sorted moments FP64 (w per particle)
    const float *m32;       // sorted moments FP32 (8 per particle)
    const void *M;          // normalised multipoles (harmonic basis: folded), rows of nmp
    const int32_t *perm;
    double *phi, *field;
    int n, nmp, outputs;
    double theta2;
    BHGeo g;
    unsigned long long *counts;   // [0] accepted (particle, cell) pairs, [1] direct pairs
    int mask, w;                  // source orders present (bit mask), FP64 moments per particle
    double *grad;                 // field gradient (n x 6), kernels with GRAD only
    int split;                    // wavefronts that share a group of 64 particles (1, 2, 4 or 8)
    double *part;                 // their sums, split x n x (4 or, with GRAD, 10)
};

constexpr int kStack = 8 * (kMaxLevel + 3);

typedef void (*bh_fn)(BHArgs);

__device__ __forceinline__ void wave_sync_bh()
{
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// lowest p from which cells wait in LDS (harmonic basis).  us with / without
// places, theta 0.6, Plummer: MIXED p 6, 10^6 dipoles 3550 / 3750, p 4, 100k
// quadrupoles 790 / 760; MIXED gradient p 8, 100k charges 2489 / 3278, but p 6,
// 10^6 10588 / 7844; FP64 p 8 1752 / 2488, p 10, 300k dipoles 6701 / 22438, but p
// 6, 10^6 7911 / 5876; FP64 gradient p 9, 70k charges 10530 / 11310, quadrupoles
// 9900 / 12370, octupoles 10220 / 10590, but dipoles 11410 / 10340 (their kernel
// spills a third more with places), and charges p 8, 100k 6003 / 5050.
constexpr int bh_places_from(bool f32, bool grad, int s)
{
    return f32 ? (grad ? 8 : 6) : (grad ? (s == 1 ? 10 : 9) : 8);
}
// row places of a wave, and the lanes below which a round waits for more marks
constexpr int kSlots = 32;
constexpr int kRoundLanes = 36;
constexpr int kOwnLevel = 3;

// 16 bytes a lane from global memory to LDS, the lanes' data back to back
__device__ __forceinline__ void copy_row(const void *g, void *lds)
{
    __builtin_amdgcn_global_load_lds((const __attribute__((address_space(1))) void *)g,
                                     (__attribute__((address_space(3))) void *)lds, 16, 0, 0);
}

// H: the rows are folded onto the harmonic basis and contracted by M2PEvalH
// GRAD: also the field gradient, G_ij = -(1/r^3) sum M~ D_{n+e_i+e_j}(u) for
// an accepted cell and the pairs' closed forms for a leaf
template <int P, int S, typename T, bool H, bool GRAD>
__global__ __launch_bounds__(64) void bh_kernel(BHArgs a)
{
    constexpr bool F32 = sizeof(T) == 4;
    constexpr bool PLACES = H && P >= bh_places_from(F32, GRAD, S);
    // FP64 with the gradient: more terms than registers from p 5 or so on
    // (86 spilled at p 8, 1800 at p 10 in the full basis), and what else lives
    // through the M2P costs.  These kernels keep the share's numbers in LDS, and
    // have the M2P written out where the cell is accepted: called, its terms are
    // ordered before they meet this kernel's registers.  us, 70k Plummer
    // charges, theta 0.6: p 8 5380 -> 4850, full basis p 8 22 480 -> 20 000, p 10
    // 104 000 -> 88 600; dipoles p 8 5690 -> 5250, full basis p 10 107 100 -> 89 700
    // (octupoles of the harmonic basis are better called: p 8 4870 and 4280).
    constexpr bool FULL = !F32 && GRAD && !PLACES;
    constexpr bool CALLED = !FULL || (H && S == 3);
    constexpr int W = (S + 1) * (S + 2) / 2;
    __shared__ int stk_c[kStack], own_[2];
    __shared__ unsigned long long stk_m[kStack];
    const int lane = threadIdx.x;
    const int share = blockIdx.x & (a.split - 1), group = blockIdx.x / a.split;
    const int i = group * 64 + lane;
    const bool valid = i < a.n;
    const int ii = valid ? i : a.n - 1;
    const size_t n = a.n;
    const double xi = a.xs[ii], yi = a.xs[n + ii], zi = a.xs[2 * n + ii];
    double ph = 0.0, ex = 0.0, ey = 0.0, ez = 0.0;
    double g[6] = {0.0, 0.0, 0.0, 0.0, 0.0, 0.0};
    const unsigned long long live = __ballot(valid);
    int sp = 0;
    if (lane == 0) {
        stk_c[0] = 0;
        stk_m[0] = live;
        if constexpr (FULL) {
            own_[0] = a.split - 1;
            own_[1] = share;
        }
    }
    sp = 1;
    wave_sync_bh();
    const T *Mb = (const T *)a.M;
    unsigned int n_m2p = 0, n_p2p = 0;
    // M2P of one cell in the normalised form: u = (x - z)/r,
    // phi = (1/r) sum M~ D(u), E = -(1/r^2) sum M~ D_{+e}(u)
    auto m2p = [&](const T *Mc, double dx, double dy, double dz, double r) {
        const double ir = 1.0 / r;
        T p_, x_, y_, z_;
        const T ux = (T)(dx * ir), uy = (T)(dy * ir), uz = (T)(dz * ir);
        if constexpr (GRAD) {
            T gg[6];
            if constexpr (H) M2PEvalGH<P, S, T>::eval(Mc, ux, uy, uz, p_, x_, y_, z_, gg);
            else M2PEvalG<P, S, T>::eval(Mc, ux, uy, uz, p_, x_, y_, z_, gg);
            const double ir3 = ir * ir * ir;
#pragma unroll
            for (int q = 0; q < 6; ++q) g[q] -= (double)gg[q] * ir3;
        } else if constexpr (H) {
            M2PEvalH<P, S, T>::eval(Mc, ux, uy, uz, p_, x_, y_, z_);
        } else {
            M2PEval<P, S, T>::eval(Mc, ux, uy, uz, p_, x_, y_, z_);
        }
        ph += (double)p_ * ir;
        const double ir2 = ir * ir;
        ex -= (double)x_ * ir2;
        ey -= (double)y_ * ir2;
        ez -= (double)z_ * ir2;
    };
    // places: rows of 16-byte units, an odd number of them apart so that
    // lanes at different places read different banks
    constexpr int kRow16 = (int)((hterms(P) - hterms(S - 1)) * sizeof(T) + 15) / 16;
    constexpr int kStride = (kRow16 | 1) * 16 / (int)sizeof(T);
    static_assert(kRow16 <= 64, "one copy a row");
    __shared__ alignas(16) T rows[PLACES ? kSlots : 1][PLACES ? kStride : 4];
    __shared__ alignas(16) double geo[PLACES ? kSlots : 1][4];   // centre, half side
    unsigned used = 0;       // places taken (the same for the wave)
    unsigned pend = 0;       // places this lane has marked
    // rounds of evaluations; all: until no lane has a mark, else while most
    // lanes do or no place is free
    auto rounds = [&](bool all) {
        __builtin_amdgcn_s_waitcnt(0x0f70);   // vmcnt(0): the rows are in LDS
        wave_sync_bh();
        for (;;) {
            const unsigned long long m = __ballot(pend != 0);
            if (m == 0) break;
            if (!all && __popcll(m) < kRoundLanes) {
                unsigned u = pend;
                for (int o = 1; o < 64; o <<= 1) u |= __shfl_xor(u, o, 64);
                if (u != 0xffffffffu) break;
            }
            if (pend) {
                const int s = __builtin_ctz(pend);
                pend &= pend - 1;
                m2p(rows[s], __dsub_rn(xi, geo[s][0]), __dsub_rn(yi, geo[s][1]), __dsub_rn(zi, geo[s][2]), geo[s][3]);
            }
        }
        used = pend;
        for (int o = 1; o < 64; o <<= 1) used |= __shfl_xor(used, o, 64);
        used = __builtin_amdgcn_readfirstlane(used);
        wave_sync_bh();
    };
    while (sp > 0) {
        --sp;
        const int c = stk_c[sp];
        const unsigned long long mask = stk_m[sp];
        wave_sync_bh();
        const DevCell cell = a.cells[c];
        const bool mine = (mask >> lane) & 1ull;
        const double rc = ldexp(1.0, kMaxLevel - cell.level);
        const double zx = __dadd_rn(a.g.lo[0], __dmul_rn((double)(2 * cell.ix + 1) * rc, a.g.h));
        const double zy = __dadd_rn(a.g.lo[1], __dmul_rn((double)(2 * cell.iy + 1) * rc, a.g.h));
        const double zz = __dadd_rn(a.g.lo[2], __dmul_rn((double)(2 * cell.iz + 1) * rc, a.g.h));
        const double r = __dmul_rn(rc, a.g.h);
        const double dx = __dsub_rn(xi, zx), dy = __dsub_rn(yi, zy), dz = __dsub_rn(zi, zz);
        const double d2 = __dadd_rn(__dadd_rn(__dmul_rn(dx, dx), __dmul_rn(dy, dy)), __dmul_rn(dz, dz));
        const bool inside = i >= cell.first && i < cell.first + cell.count;
        const bool accept = mine && !inside && (__dmul_rn(r, r) < __dmul_rn(a.theta2, d2));
        const unsigned long long acc_m = __ballot(accept);
        const unsigned long long rest = mask & ~acc_m;
        const bool own = cell.level >= kOwnLevel || (c & (FULL ? own_[0] : a.split - 1)) == (FULL ? own_[1] : share);
        if constexpr (PLACES) {
            if (acc_m && own) {
                if (used == 0xffffffffu) rounds(false);
                const int s = __builtin_ctz(~used);
                used |= 1u << s;
                if (lane < kRow16) copy_row((const char *)(Mb + (size_t)c * a.nmp) + 16 * lane, rows[s]);
                if (lane == 0) {
                    geo[s][0] = zx;
                    geo[s][1] = zy;
                    geo[s][2] = zz;
                    geo[s][3] = r;
                }
                if (accept) {
                    ++n_m2p;
                    pend |= 1u << s;
                }
            }
        } else if (accept && own) {
            ++n_m2p;
            if constexpr (CALLED) {
                m2p(Mb + (size_t)c * a.nmp, dx, dy, dz, r);
            } else {
                const double ir = 1.0 / r;
                T p_, x_, y_, z_, gg[6];
                const T *Mc = Mb + (size_t)c * a.nmp;
                const T ux = (T)(dx * ir), uy = (T)(dy * ir), uz = (T)(dz * ir);
                if constexpr (H) M2PEvalGH<P, S, T>::eval(Mc, ux, uy, uz, p_, x_, y_, z_, gg);
                else M2PEvalG<P, S, T>::eval(Mc, ux, uy, uz, p_, x_, y_, z_, gg);
                const double ir3 = ir * ir * ir;
#pragma unroll
                for (int q = 0; q < 6; ++q) g[q] -= (double)gg[q] * ir3;
                ph += (double)p_ * ir;
                const double ir2 = ir * ir;
                ex -= (double)x_ * ir2;
                ey -= (double)y_ * ir2;
                ez -= (double)z_ * ir2;
            }
        }
        if (rest) {
            if (cell.nchild == 0) {
                if (own && ((rest >> lane) & 1ull)) {
                    n_p2p += (unsigned)cell.count - (inside ? 1u : 0u);
                    if (a.mask != (1 << S)) {
                        // several source orders: each order's closed form, FP64
                        for (int j = cell.first; j < cell.first + cell.count; ++j) {
                            if (j == i) continue;
                            const double *mj = a.m64 + (size_t)j * a.w;
                            const double rx = xi - a.xs[j], ry = yi - a.xs[n + j], rz = zi - a.xs[2 * n + j];
                            int off = 0;
                            if (a.mask & 1) {
                                p2p_pair_f64<0>(rx, ry, rz, mj + off, ph, ex, ey, ez);
                                if constexpr (GRAD) p2p_pair_grad_f64<0>(rx, ry, rz, mj + off, g);
                                off += 1;
                            }
                            if (a.mask & 2) {
                                p2p_pair_f64<1>(rx, ry, rz, mj + off, ph, ex, ey, ez);
                                if constexpr (GRAD) p2p_pair_grad_f64<1>(rx, ry, rz, mj + off, g);
                                off += 3;
                            }
                            if (a.mask & 4) {
                                p2p_pair_f64<2>(rx, ry, rz, mj + off, ph, ex, ey, ez);
                                if constexpr (GRAD) p2p_pair_grad_f64<2>(rx, ry, rz, mj + off, g);
                                off += 6;
                            }
                            if (a.mask & 8) {
                                p2p_pair_oct_f64(rx, ry, rz, mj + off, ph, ex, ey, ez);
                                if constexpr (GRAD) p2p_pair_grad_oct_f64(rx, ry, rz, mj + off, g);
                            }
                        }
                    } else if (F32) {
                        // sources in units of the leaf radius, FP32 block sum
                        const double ir = 1.0 / r;
                        float bp = 0.f, bx = 0.f, by = 0.f, bz = 0.f;
                        float bg[6] = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
                        for (int j = cell.first; j < cell.first + cell.count; ++j) {
                            if (j == i) continue;
                            const float rx = (float)((xi - a.xs[j]) * ir), ry = (float)((yi - a.xs[n + j]) * ir),
                                        rz = (float)((zi - a.xs[2 * n + j]) * ir);
                            const float r2 = __builtin_fmaf(rx, rx, __builtin_fmaf(ry, ry, rz * rz));
                            const float4 *m4 =
                                reinterpret_cast<const float4 *>(a.m32) + (size_t)(m32_width(1 << S) / 4) * j;
                            const float inv = __builtin_amdgcn_rsqf(r2);
                            if constexpr (S == 3) {
                                p2p_pair_oct_f32(rx, ry, rz, inv, m4[0], m4[1], m4[2], m4[3], bp, bx, by, bz);
                                if constexpr (GRAD) p2p_pair_grad_oct_f32(rx, ry, rz, inv, m4[0], m4[1], m4[2], m4[3], bg);
                            } else {
                                p2p_pair_f32<S>(rx, ry, rz, r2, inv, m4[0], m4[1], bp, bx, by, bz);
                                if constexpr (GRAD) p2p_pair_grad_f32<S>(rx, ry, rz, inv, m4[0], m4[1], bg);
                            }
                        }
                        double sphi = ir;
#pragma unroll
                        for (int q = 0; q < S; ++q) sphi *= ir;
                        const double sfld = sphi * ir;
                        ph += (double)bp * (p2p_phi_scale(S) * sphi);
                        ex += (double)bx * sfld;
                        ey += (double)by * sfld;
                        ez += (double)bz * sfld;
                        if constexpr (GRAD) {
                            const double sgrd = sfld * ir;
#pragma unroll
                            for (int q = 0; q < 6; ++q) g[q] += (double)bg[q] * sgrd;
                        }
                    } else {
                        for (int j = cell.first; j < cell.first + cell.count; ++j) {
                            if (j == i) continue;
                            const double rx = xi - a.xs[j], ry = yi - a.xs[n + j], rz = zi - a.xs[2 * n + j];
                            if constexpr (S == 3) {
                                p2p_pair_oct_f64(rx, ry, rz, a.m64 + (size_t)j * W, ph, ex, ey, ez);
                                if constexpr (GRAD) p2p_pair_grad_oct_f64(rx, ry, rz, a.m64 + (size_t)j * W, g);
                            } else {
                                p2p_pair_f64<S>(rx, ry, rz, a.m64 + (size_t)j * W, ph, ex, ey, ez);
                                if constexpr (GRAD) p2p_pair_grad_f64<S>(rx, ry, rz, a.m64 + (size_t)j * W, g);
                            }
                        }
                    }
                }
            } else {
                // children in reverse, so that they are visited in octant
                // order, a lane each; of those at kOwnLevel this wavefront's
                const bool keep = lane < cell.nchild && (cell.level != kOwnLevel - 1 ||
                                                         ((cell.child0 + lane) & (FULL ? own_[0] : a.split - 1)) ==
                                                             (FULL ? own_[1] : share));
                const unsigned long long km = __ballot(keep);
                if (keep) {
                    const int at = sp + __popcll(km >> lane) - 1;   // those after it lie below
                    stk_c[at] = cell.child0 + lane;
                    stk_m[at] = rest;
                }
                sp += __popcll(km);
                wave_sync_bh();
            }
        }
    }
    if constexpr (PLACES) rounds(true);
    // interaction counts of the wave, one atomic per wave
    unsigned long long c0 = n_m2p, c1 = n_p2p;
    for (int o = 32; o > 0; o >>= 1) {
        c0 += __shfl_down(c0, o, 64);
        c1 += __shfl_down(c1, o, 64);
    }
    if (lane == 0) {
        atomicAdd(&a.counts[0], c0);
        atomicAdd(&a.counts[1], c1);
    }
    if (valid && a.split > 1) {
        constexpr int NO = GRAD ? 10 : 4;
        double *o = a.part + ((size_t)share * n + i) * NO;
        o[0] = ph;
        o[1] = ex;
        o[2] = ey;
        o[3] = ez;
        if constexpr (GRAD)
#pragma unroll
            for (int q = 0; q < 6; ++q) o[4 + q] = g[q];
        return;
    }
    if (valid) {
        const size_t o = (size_t)a.perm[i];
        if (a.outputs & FMM_POT) a.phi[o] = ph;
        if (a.outputs & FMM_FIELD) {
            a.field[3 * o] = ex;
            a.field[3 * o + 1] = ey;
            a.field[3 * o + 2] = ez;
        }
        if constexpr (GRAD) {
            if (a.outputs & FMM_GRAD)
#pragma unroll
                for (int q = 0; q < 6; ++q) a.grad[6 * o + q] = g[q];
        }
    }
}

// the kernel for (p, s, precision, basis), p in [max(s,1), FMM_P_MAX]
template <bool GRAD, int P, int S>
bh_fn bh_pick(bool f32, bool h)
{
    if (h) return f32 ? (bh_fn)bh_kernel<P, S, float, true, GRAD> : (bh_fn)bh_kernel<P, S, double, true, GRAD>;
    return f32 ? (bh_fn)bh_kernel<P, S, float, false, GRAD> : (bh_fn)bh_kernel<P, S, double, false, GRAD>;
}

template <bool GRAD, int S, int P = (S > 1 ? S : 1)>
bh_fn bh_pick_p(int p, bool f32, bool h)
{
    if constexpr (P > FMM_P_MAX) {
        return nullptr;
    } else {
        if (p == P) return bh_pick<GRAD, P, S>(f32, h);
        return bh_pick_p<GRAD, S, P + 1>(p, f32, h);
    }
}

// one per (field gradient, source order), each in its own generated
// translation unit (gen_bh.py)
bh_fn bh_select_f_s0(int p, bool f32, bool h);
bh_fn bh_select_f_s1(int p, bool f32, bool h);
bh_fn bh_select_f_s2(int p, bool f32, bool h);
bh_fn bh_select_f_s3(int p, bool f32, bool h);
bh_fn bh_select_g_s0(int p, bool f32, bool h);
bh_fn bh_select_g_s1(int p, bool f32, bool h);
bh_fn bh_select_g_s2(int p, bool f32, bool h);
bh_fn bh_select_g_s3(int p, bool f32, bool h);
