// GPU kernels of libfmm.so other than M2L and Barnes-Hut: particle and
// moment preparation, P2M, M2M, L2L, P2P and L2P (Pepper & Fangohr, arXiv
// 2005.12351, Section 2 and Section 3.2).
//
// All expansions on the GPU are kept in a dimensionless form:
//   M~_n(A) = M_n(A) / r_A^|n|,  L~_n(B) = L_n(B) * r_B^(|n|+1),
// with r the cell radius (half side).  Child and parent centres differ by
// exactly +-r_child per axis, so M2M and L2L become fixed rational operators
// per octant and the M2L derivative tensor depends only on the dimensionless
// pair geometry.  P2M, M2M, L2L, L2P run in FP64.
#include <cmath>
#include <mutex>
#include <type_traits>

#include "fmm_internal.h"
#include "pair_kernels.h"

// ------------------------------------------------------------------ tables
struct HalfTable {
    double v[kPTable + 2];
};
constexpr HalfTable make_half()
{
    HalfTable t{};
    double f = 1.0;
    for (int a = 0; a <= kPTable + 1; ++a) {
        if (a > 0) f = f * 0.5 / a;
        t.v[a] = f;
    }
    return t;
}
static __constant__ MITable k_mi = make_mi();
__constant__ HalfTable k_half = make_half();   // (1/2)^a / a!

__device__ __forceinline__ double cell_radius(int level, double h) { return ldexp(1.0, kMaxLevel - level) * h; }

// real centre, computed exactly as the canonical definition: lo + c * h
__device__ __forceinline__ void cell_center(const DevCell &c, const double *lo, double h, double *z)
{
    const double r = ldexp(1.0, kMaxLevel - c.level);
    z[0] = __dadd_rn(lo[0], __dmul_rn((double)(2 * c.ix + 1) * r, h));
    z[1] = __dadd_rn(lo[1], __dmul_rn((double)(2 * c.iy + 1) * r, h));
    z[2] = __dadd_rn(lo[2], __dmul_rn((double)(2 * c.iz + 1) * r, h));
}

struct Geo {
    double lo[3];
    double h;
};

// ------------------------------------------------------------------ fill
__global__ void fill_kernel(double *p, size_t n)
{
    for (size_t i = blockIdx.x * (size_t)blockDim.x + threadIdx.x; i < n; i += (size_t)gridDim.x * blockDim.x) p[i] = 0.0;
}

__global__ void zero_ints_kernel(int *p, int n)
{
    if ((int)threadIdx.x < n) p[threadIdx.x] = 0;
}

hipError_t launch_fill(double *p, size_t count, hipStream_t s)
{
    if (count == 0) return hipSuccess;
    const unsigned g = (unsigned)std::min<size_t>((count + 255) / 256, 4096);
    hipLaunchKernelGGL(fill_kernel, dim3(g), dim3(256), 0, s, p, count);
    return hipGetLastError();
}

// ------------------------------------------------------------------ particles
// sorted SoA positions
__global__ void prep_particles_kernel(int n, const double *__restrict__ pos, const int32_t *__restrict__ perm,
                                      double *__restrict__ xs)
{
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= n) return;
    const int j = perm[i];
    xs[i] = pos[3 * (size_t)j];
    xs[n + i] = pos[3 * (size_t)j + 1];
    xs[2 * (size_t)n + i] = pos[3 * (size_t)j + 2];
}

hipError_t launch_prep_positions(fmm_tree *t, const double *pos, hipStream_t s)
{
    const int n = (int)t->ht.n;
    hipLaunchKernelGGL(prep_particles_kernel, dim3((n + 255) / 256), dim3(256), 0, s, n, pos, t->d_perm, t->d_x);
    return hipGetLastError();
}

// Sorted moments of particle i (sorted order; perm maps it to the caller's
// row): FP64 (the caller's row of w values) and FP32 in the layout m32_width
// describes.  P2M writes them while it visits every particle once; the near
// field reads them.
__device__ __forceinline__ void sort_moments(size_t i, int mask, const double *__restrict__ r,
                                             double *__restrict__ m64, float *__restrict__ m32)
{
    const int w = mask_width(mask), wf = m32_width(mask);
    float v[28];
#pragma unroll
    for (int k = 0; k < 28; ++k) v[k] = 0.f;
    for (int k = 0; k < w; ++k) m64[i * w + k] = r[k];
    // the octupole block: ten components and the trace vector
    auto oct = [&](const double *o, int at) {
        for (int k = 0; k < 10; ++k) v[at + k] = (float)o[k];
        v[at + 10] = (float)(o[0] + o[3] + o[5]);
        v[at + 11] = (float)(o[1] + o[6] + o[8]);
        v[at + 12] = (float)(o[2] + o[7] + o[9]);
    };
    if (mask == 8) {
        oct(r, 0);
    } else if (mask_single(mask)) {
        for (int k = 0; k < w; ++k) v[k] = (float)r[k];
        if (w == 6) {
            v[6] = (float)(r[0] + r[3] + r[5]);
            v[7] = -1.5f * v[6];
        }
    } else {
        int off = 0;
        if (mask & 1) v[0] = (float)r[off++];
        if (mask & 2) {
            v[1] = (float)r[off];
            v[2] = (float)r[off + 1];
            v[3] = (float)r[off + 2];
            off += 3;
        }
        if (mask & 4) {
            for (int k = 0; k < 6; ++k) v[4 + k] = (float)r[off + k];
            v[10] = (float)(r[off] + r[off + 3] + r[off + 5]);
            v[11] = -1.5f * v[10];
            off += 6;
        }
        if (mask & 8) oct(r + off, 12);
    }
    float4 *o = reinterpret_cast<float4 *>(m32) + (size_t)(wf / 4) * i;
    for (int k = 0; k < wf / 4; ++k) o[k] = make_float4(v[4 * k], v[4 * k + 1], v[4 * k + 2], v[4 * k + 3]);
}

// ------------------------------------------------------------------ P2M
// M~_n = sum_j sum_k r^-k sum_{sigma <= n, |sigma| = k} zeta_j^(n-sigma)/(n-sigma)! S_sigma(j)
// with zeta = (z - x_j)/r and S_sigma = (-1)^k T_sigma / sigma! (Eq. 3, Eq. 5),
// k over the source orders present (MASK bit k), so a system with several
// orders adds each part's expansion.  One workgroup per leaf; particles are
// staged in LDS 32 at a time as per-axis tables X_a = zeta_x^a/a! (and Y, Z).
// Harmonic rows have a kernel of their own (p2m_harmonic_kernel).  Full basis:
// two kernels, chosen by the source orders:
// - p2m_coef_kernel (charges and dipoles, and any system with octupoles): a
//   thread owns one or more coefficients n and adds every particle's term,
//   1 + 3 (+ 6 + 10) products of table entries per particle;
// - p2m_kernel (any quadrupole part): the monomial factorises over the axes
//   and sigma has at most two units, so for a fixed column (ax, ay) the
//   particle's contribution to every coefficient (ax, ay, az) is
//   A0 Z_az + A1 Z_{az-1} + A2 Z_{az-2}, with
//   A0 = S_0 X0 Y0 + S_ex X1 Y0 + S_ey X0 Y1 + S_2ex X2 Y0 + S_ex+ey X1 Y1 + S_2ey X0 Y2,
//   A1 = S_ez X0 Y0 + S_ex+ez X1 Y0 + S_ey+ez X0 Y1, A2 = S_2ez X0 Y0
//   (Xk = X_{ax-k}, Yk = Y_{ay-k}).  A thread owns a block of consecutive az
//   of one column and forms A0..A2 once per particle; when the blocks fill
//   less than half the workgroup, groups of threads take every ngroups-th
//   particle and their sums are added in group order at the end (a fixed
//   order).  With quadrupoles this is 25 % faster than the per-coefficient
//   form (ten terms per coefficient and particle there); with dipoles it is
//   not, so those keep the simpler kernel.
constexpr int kP2MThreads = 128;
constexpr int kP2MStage = 32;                    // particles staged per pass
constexpr int kP2MBlk = 6;                       // longest column block
constexpr int kAxWc = FMM_P_MAX + 2;             // axis table row of the per-coefficient kernel: X_0..X_p
constexpr int kAxW = FMM_P_MAX + kP2MBlk + 4;    // of the column kernel: X_-2, X_-1 (zero), X_0..X_p, zero padding

struct InvTable {
    double v[kPTable + 2];
};
constexpr InvTable make_inv()
{
    InvTable t{};
    t.v[0] = 1.0;
    for (int a = 1; a <= kPTable + 1; ++a) t.v[a] = 1.0 / a;
    return t;
}
__constant__ InvTable k_inv = make_inv();   // 1/a

template <int MASK>
__global__ __launch_bounds__(kP2MThreads) void p2m_coef_kernel(int p, int nmp, const int32_t *__restrict__ leaves,
                                                          const DevCell *__restrict__ cells, Geo g,
                                                          const double *__restrict__ xs, int n,
                                                          const double *__restrict__ mom_user,
                                                          const int32_t *__restrict__ perm, double *__restrict__ mom64,
                                                          float *__restrict__ mom32, double *__restrict__ M,
                                                          float *__restrict__ M32)
{
    constexpr int W = mask_width(MASK);
    constexpr int S = mask_min_order(MASK);
    constexpr bool Q0 = MASK & 1, Q1 = MASK & 2, Q2 = MASK & 4, Q3 = MASK & 8;
    // source tensor slots: 0 order 0; 1..3 order 1; 4..9 order 2; 10..19
    // order 3 (index order within each order)
    __shared__ double pw[kP2MStage][3][kAxWc];
    __shared__ double sv[kP2MStage][20];
    const int c = leaves[blockIdx.x];
    const DevCell cell = cells[c];
    double z[3];
    cell_center(cell, g.lo, g.h, z);
    const double r = cell_radius(cell.level, g.h);
    const double ir = 1.0 / r;
    const int n0 = nterms(S - 1), nm = nterms(p) - n0;
    constexpr int KMAX = (nterms(FMM_P_MAX) + kP2MThreads - 1) / kP2MThreads;
    double acc[KMAX];
    int ix[KMAX], iy[KMAX], iz[KMAX];
#pragma unroll
    for (int k = 0; k < KMAX; ++k) {
        acc[k] = 0.0;
        const int i = threadIdx.x + k * kP2MThreads;
        const MultiIndex nn = k_mi.v[i < nm ? n0 + i : 0];
        ix[k] = nn.x;
        iy[k] = nn.y;
        iz[k] = nn.z;
    }
    for (int base = 0; base < cell.count; base += kP2MStage) {
        const int cnt = min(kP2MStage, cell.count - base);
        __syncthreads();
        for (int it = threadIdx.x; it < 3 * cnt; it += kP2MThreads) {
            // item -> (particle, axis): zeta^a / a! for a = 0..p
            const int t = it / 3, d = it % 3;
            const size_t j = (size_t)cell.first + base + t;
            const double zeta = (z[d] - xs[(size_t)d * n + j]) * ir;
            double f = 1.0;
            pw[t][d][0] = 1.0;
            for (int a = 1; a <= p; ++a) {
                f = f * zeta * k_inv.v[a];
                pw[t][d][a] = f;
            }
        }
        if ((int)threadIdx.x < cnt) {
            const int t = threadIdx.x;
            const size_t i = (size_t)cell.first + base + t;
            const double *m = mom_user + (size_t)perm[i] * W;
            sort_moments(i, MASK, m, mom64, mom32);
            int off = 0;
            if (Q0) sv[t][0] = m[off++];
            if (Q1) {
                sv[t][1] = -m[off] * ir;
                sv[t][2] = -m[off + 1] * ir;
                sv[t][3] = -m[off + 2] * ir;
                off += 3;
            }
            if (Q2) {
                const double ir2 = ir * ir;
                sv[t][4] = 0.5 * m[off] * ir2;       // (2,0,0)
                sv[t][5] = m[off + 1] * ir2;         // (1,1,0)
                sv[t][6] = m[off + 2] * ir2;         // (1,0,1)
                sv[t][7] = 0.5 * m[off + 3] * ir2;   // (0,2,0)
                sv[t][8] = m[off + 4] * ir2;         // (0,1,1)
                sv[t][9] = 0.5 * m[off + 5] * ir2;   // (0,0,2)
                off += 6;
            }
            if (Q3) {
                // S_m = -O_m / m!: m! = 6 for (3,0,0)-type, 2 for (2,1,0)-type,
                // 1 for (1,1,1)
                const double ir3 = ir * ir * ir;
                constexpr double kInvF[10] = {1.0 / 6, 0.5, 0.5, 0.5, 1.0, 0.5, 1.0 / 6, 0.5, 0.5, 1.0 / 6};
#pragma unroll
                for (int q = 0; q < 10; ++q) sv[t][10 + q] = -m[off + q] * kInvF[q] * ir3;
            }
        }
        __syncthreads();
#pragma unroll
        for (int k = 0; k < KMAX; ++k) {
            if ((int)threadIdx.x + k * kP2MThreads >= nm) break;
            const int ax = ix[k], ay = iy[k], az = iz[k];
            double a = acc[k];
            for (int t = 0; t < cnt; ++t) {
                // a zero table entry stands for a negative index
                const double px0 = pw[t][0][ax], py0 = pw[t][1][ay], pz0 = pw[t][2][az];
                if (Q0) a = fma(px0 * py0, pz0 * sv[t][0], a);
                if (Q1 || Q2 || Q3) {
                    const double px1 = ax >= 1 ? pw[t][0][ax - 1] : 0.0, py1 = ay >= 1 ? pw[t][1][ay - 1] : 0.0,
                                 pz1 = az >= 1 ? pw[t][2][az - 1] : 0.0;
                    if (Q1) {
                        a = fma(px1 * py0, pz0 * sv[t][1], a);
                        a = fma(px0 * py1, pz0 * sv[t][2], a);
                        a = fma(px0 * py0, pz1 * sv[t][3], a);
                    }
                    if (Q2) {
                        const double px2 = ax >= 2 ? pw[t][0][ax - 2] : 0.0, py2 = ay >= 2 ? pw[t][1][ay - 2] : 0.0,
                                     pz2 = az >= 2 ? pw[t][2][az - 2] : 0.0;
                        a = fma(px2 * py0, pz0 * sv[t][4], a);
                        a = fma(px1 * py1, pz0 * sv[t][5], a);
                        a = fma(px1 * py0, pz1 * sv[t][6], a);
                        a = fma(px0 * py2, pz0 * sv[t][7], a);
                        a = fma(px0 * py1, pz1 * sv[t][8], a);
                        a = fma(px0 * py0, pz2 * sv[t][9], a);
                    }
                    if (Q3) {
                        const double px2 = ax >= 2 ? pw[t][0][ax - 2] : 0.0, py2 = ay >= 2 ? pw[t][1][ay - 2] : 0.0,
                                     pz2 = az >= 2 ? pw[t][2][az - 2] : 0.0;
                        const double px3 = ax >= 3 ? pw[t][0][ax - 3] : 0.0, py3 = ay >= 3 ? pw[t][1][ay - 3] : 0.0,
                                     pz3 = az >= 3 ? pw[t][2][az - 3] : 0.0;
                        a = fma(px3 * py0, pz0 * sv[t][10], a);   // (3,0,0)
                        a = fma(px2 * py1, pz0 * sv[t][11], a);   // (2,1,0)
                        a = fma(px2 * py0, pz1 * sv[t][12], a);   // (2,0,1)
                        a = fma(px1 * py2, pz0 * sv[t][13], a);   // (1,2,0)
                        a = fma(px1 * py1, pz1 * sv[t][14], a);   // (1,1,1)
                        a = fma(px1 * py0, pz2 * sv[t][15], a);   // (1,0,2)
                        a = fma(px0 * py3, pz0 * sv[t][16], a);   // (0,3,0)
                        a = fma(px0 * py2, pz1 * sv[t][17], a);   // (0,2,1)
                        a = fma(px0 * py1, pz2 * sv[t][18], a);   // (0,1,2)
                        a = fma(px0 * py0, pz3 * sv[t][19], a);   // (0,0,3)
                    }
                }
            }
            acc[k] = a;
        }
    }
#pragma unroll
    for (int k = 0; k < KMAX; ++k)
        if ((int)threadIdx.x + k * kP2MThreads < nm) {
            const size_t o = (size_t)c * nmp + threadIdx.x + k * kP2MThreads;
            M[o] = acc[k];                     // the FP64 upward state
            if (M32) M32[o] = (float)acc[k];   // the copy the mixed-precision M2L reads
        }
}

// Column blocks of every (p, s), fixed at compile time: for each pair the
// block length with the fewest multiply-add steps per particle (about 10 to
// form A0..A2 plus 3 per block entry, divided by the groups of threads that
// share the particles), then the blocks in column order, (ax, ay, az0, nb).
struct P2MItem {
    int8_t ax, ay, az0, nb;
};
constexpr int kP2MPlanMax = 3 * (FMM_P_MAX + 1) * kP2MThreads;
struct P2MPlan {
    int16_t start[FMM_P_MAX + 1][3];
    int16_t nitems[FMM_P_MAX + 1][3];
    int8_t blk[FMM_P_MAX + 1][3];
    int8_t ngroups[FMM_P_MAX + 1][3];
    P2MItem items[kP2MPlanMax];
};
constexpr int p2m_count(int p, int S, int blk)
{
    int cnt = 0;
    for (int x = 0; x <= p; ++x)
        for (int y = 0; y <= p - x; ++y) {
            const int lo = S - x - y > 0 ? S - x - y : 0, hi = p - x - y;
            cnt += (hi - lo + blk) / blk;
        }
    return cnt;
}
constexpr P2MPlan make_p2m_plan()
{
    P2MPlan pl{};
    int pos = 0;
    for (int p = 0; p <= FMM_P_MAX; ++p)
        for (int S = 0; S < 3; ++S) {
            pl.start[p][S] = (int16_t)pos;
            if (S > p) continue;
            int best_b = kP2MBlk, best_n = p2m_count(p, S, kP2MBlk);
            double best = (10.0 + 3.0 * kP2MBlk) / (kP2MThreads / best_n);
            for (int bl = 2; bl < kP2MBlk; ++bl) {
                const int ni = p2m_count(p, S, bl);
                if (ni > kP2MThreads) continue;
                const double cost = (10.0 + 3.0 * bl) / (kP2MThreads / ni);
                if (cost < best) {
                    best = cost;
                    best_b = bl;
                    best_n = ni;
                }
            }
            pl.blk[p][S] = (int8_t)best_b;
            pl.nitems[p][S] = (int16_t)best_n;
            pl.ngroups[p][S] = (int8_t)(kP2MThreads / best_n);
            for (int x = 0; x <= p; ++x)
                for (int y = 0; y <= p - x; ++y) {
                    const int lo = S - x - y > 0 ? S - x - y : 0, hi = p - x - y;
                    for (int z0 = lo; z0 <= hi; z0 += best_b)
                        pl.items[pos++] = P2MItem{(int8_t)x, (int8_t)y, (int8_t)z0,
                                                  (int8_t)(hi + 1 - z0 < best_b ? hi + 1 - z0 : best_b)};
                }
        }
    return pl;
}
static __constant__ P2MPlan k_p2m = make_p2m_plan();
static constexpr P2MPlan kP2MPlanHost = make_p2m_plan();
// the longest block always fits: at p = 10, s = 0 it makes 81 blocks
static_assert(p2m_count(FMM_P_MAX, 0, kP2MBlk) <= kP2MThreads, "P2M blocks exceed the workgroup");

template <int MASK>
__global__ __launch_bounds__(kP2MThreads) void p2m_kernel(int p, int nmp, int blk, int nitems, int ngroups,
                                                          const int32_t *__restrict__ leaves,
                                                          const DevCell *__restrict__ cells, Geo g,
                                                          const double *__restrict__ xs, int n,
                                                          const double *__restrict__ mom_user,
                                                          const int32_t *__restrict__ perm, double *__restrict__ mom64,
                                                          float *__restrict__ mom32, double *__restrict__ M,
                                                          float *__restrict__ M32)
{
    constexpr int W = mask_width(MASK);
    constexpr int S = mask_min_order(MASK);
    constexpr bool Q0 = MASK & 1, Q1 = MASK & 2, Q2 = MASK & 4;
    // source tensor slots: 0 order 0; 1..3 order 1; 4..9 order 2
    __shared__ double pw[kP2MStage][3][kAxW];
    __shared__ double sv[kP2MStage][10];
    __shared__ double gsum[kP2MThreads * kP2MBlk];   // sums of groups 1.. (ngroups > 1)
    const int c = leaves[blockIdx.x];
    const DevCell cell = cells[c];
    double z[3];
    cell_center(cell, g.lo, g.h, z);
    const double r = cell_radius(cell.level, g.h);
    const double ir = 1.0 / r;
    const int n0 = nterms(S - 1);
    const int item = (int)threadIdx.x % nitems, grp = (int)threadIdx.x / nitems;
    const bool act = grp < ngroups;
    const P2MItem pi = k_p2m.items[k_p2m.start[p][S] + item];
    const int ax = pi.ax, ay = pi.ay, az0 = pi.az0, nb = pi.nb;
    double acc[kP2MBlk];
#pragma unroll
    for (int k = 0; k < kP2MBlk; ++k) acc[k] = 0.0;
    for (int base = 0; base < cell.count; base += kP2MStage) {
        const int cnt = min(kP2MStage, cell.count - base);
        __syncthreads();
        for (int it = threadIdx.x; it < 3 * cnt; it += kP2MThreads) {
            // item -> (particle, axis): two zeros, zeta^a / a! for a = 0..p, zeros
            const int t = it / 3, d = it % 3;
            const size_t j = (size_t)cell.first + base + t;
            const double zeta = (z[d] - xs[(size_t)d * n + j]) * ir;
            double *row_t = pw[t][d];
            double f = 1.0;
            row_t[0] = 0.0;
            row_t[1] = 0.0;
            row_t[2] = 1.0;
            for (int e = 1; e <= p; ++e) {
                f = f * zeta * k_inv.v[e];
                row_t[2 + e] = f;
            }
            for (int e = p + 3; e < kAxW; ++e) row_t[e] = 0.0;
        }
        if ((int)threadIdx.x < cnt) {
            const int t = threadIdx.x;
            const size_t i = (size_t)cell.first + base + t;
            const double *m = mom_user + (size_t)perm[i] * W;
            sort_moments(i, MASK, m, mom64, mom32);
            int off = 0;
            if (Q0) sv[t][0] = m[off++];
            if (Q1) {
                sv[t][1] = -m[off] * ir;
                sv[t][2] = -m[off + 1] * ir;
                sv[t][3] = -m[off + 2] * ir;
                off += 3;
            }
            if (Q2) {
                const double ir2 = ir * ir;
                sv[t][4] = 0.5 * m[off] * ir2;       // (2,0,0)
                sv[t][5] = m[off + 1] * ir2;         // (1,1,0)
                sv[t][6] = m[off + 2] * ir2;         // (1,0,1)
                sv[t][7] = 0.5 * m[off + 3] * ir2;   // (0,2,0)
                sv[t][8] = m[off + 4] * ir2;         // (0,1,1)
                sv[t][9] = 0.5 * m[off + 5] * ir2;   // (0,0,2)
            }
        }
        __syncthreads();
        if (act) {
            for (int t = grp; t < cnt; t += ngroups) {
                const double *X = pw[t][0], *Y = pw[t][1], *Z = pw[t][2] + az0;
                const double x0 = X[ax + 2], y0 = Y[ay + 2];
                const double x0y0 = x0 * y0;
                double A0 = 0.0, A1 = 0.0, A2 = 0.0;
                if (Q0) A0 = sv[t][0] * x0y0;
                if (Q1 || Q2) {
                    const double x1 = X[ax + 1], y1 = Y[ay + 1];
                    const double x1y0 = x1 * y0, x0y1 = x0 * y1;
                    if (Q1) {
                        A0 = fma(sv[t][1], x1y0, A0);
                        A0 = fma(sv[t][2], x0y1, A0);
                        A1 = sv[t][3] * x0y0;
                    }
                    if (Q2) {
                        const double x2 = X[ax], y2 = Y[ay];
                        A0 = fma(sv[t][4], x2 * y0, A0);
                        A0 = fma(sv[t][5], x1 * y1, A0);
                        A0 = fma(sv[t][7], x0 * y2, A0);
                        A1 = fma(sv[t][6], x1y0, A1);
                        A1 = fma(sv[t][8], x0y1, A1);
                        A2 = sv[t][9] * x0y0;
                    }
                }
                // Z[k + 2] = Z_{az0+k}; blocks past the column's end read
                // real or zero table entries into sums that are not written
#pragma unroll
                for (int k = 0; k < kP2MBlk; ++k) {
                    if (k >= blk) break;
                    double v = fma(A0, Z[k + 2], acc[k]);
                    if (Q1 || Q2) v = fma(A1, Z[k + 1], v);
                    if (Q2) v = fma(A2, Z[k], v);
                    acc[k] = v;
                }
            }
        }
    }
    if (ngroups > 1) {
        __syncthreads();
        if (act && grp > 0)
#pragma unroll
            for (int k = 0; k < kP2MBlk; ++k)
                if (k < blk) gsum[((grp - 1) * nitems + item) * kP2MBlk + k] = acc[k];
        __syncthreads();
        if (act && grp == 0)
            for (int q = 1; q < ngroups; ++q)
#pragma unroll
                for (int k = 0; k < kP2MBlk; ++k)
                    if (k < blk) acc[k] += gsum[((q - 1) * nitems + item) * kP2MBlk + k];
    }
    if (act && grp == 0)
#pragma unroll
        for (int k = 0; k < kP2MBlk; ++k) {
            if (k >= nb) break;
            const int i = mindex(ax, ay, az0 + k);
            const size_t o = (size_t)c * nmp + (i - n0);
            M[o] = acc[k];                     // the FP64 upward state
            if (M32) M32[o] = (float)acc[k];   // the copy the mixed-precision M2L reads
        }
}

// harmonic-basis rows written by P2M and M2M (null when unused): the FP64
// folded rows (the upward state of that basis; in FP64 precision also what
// the M2L reads) and, in MIXED, their FP32 copy the M2L reads
struct HarmOut {
    int nhp;
    float *h32;
    double *h64;
};
static HarmOut harm_out(const fmm_tree *t)
{
    HarmOut o{0, nullptr, nullptr};
    if (t->basis != FMM_M2L_HARMONIC || !t->d_Mh) return o;
    o.nhp = t->nhp;
    if (t->prec == FMM_PREC_MIXED) {
        o.h32 = (float *)t->d_Mh;
        o.h64 = t->d_Mf64;
    } else {
        o.h64 = (double *)t->d_Mh;
    }
    return o;
}

// Functions of a harmonic row: F_h(eta), h = (a, b, r) with r <= 1, the fold of
// eta^n / n!.  The fold commutes with derivatives,
//   d_x F(a,b,r) = F(a-1,b,r),  d_y F(a,b,r) = F(a,b-1,r),
//   d_z F(a,b,1) = F(a,b,0),    d_z F(a,b,0) = -F(a-2,b,1) - F(a,b-2,1),
// so the gradient of order l is entries of order l - 1, and by Euler's identity
// l F = eta . grad F gives order l.
__host__ __device__ constexpr int horder(int a, int b, int r) { return b + r == 0 ? 0 : 2 * (b + r) - 1 + r; }

// component (a, b, r) of the order held in F, zero where an index is negative
__device__ __forceinline__ double hat(const double *F, int a, int b, int r)
{
    return a < 0 || b < 0 ? 0.0 : F[horder(a, b, r)];
}

// d_z of component (a, b, r), from the entries F of one order less, and whether
// it has any term
__host__ __device__ constexpr bool hat_dz_any(int a, int b, int r)
{
    return a >= 0 && b >= 0 && (r || a >= 2 || b >= 2);
}
__device__ __forceinline__ double hat_dz(const double *F, int a, int b, int r)
{
    if (a < 0 || b < 0) return 0.0;
    if (r) return F[horder(a, b, 0)];
    if (a < 2) return -hat(F, a, b - 2, 1);
    if (b < 2) return -hat(F, a - 2, b, 1);
    return -(hat(F, a - 2, b, 1) + hat(F, a, b - 2, 1));
}

// P2M of harmonic rows.  A particle's row, G_n = sum_sigma S_sigma
// zeta^(n-sigma)/(n-sigma)! folded, has the same derivatives as F and degree
// l - k for a source of order k: (l - k) G_l = zeta . grad G_l, from G_k = the
// folded source tensor.  So every source order costs four multiply-adds a
// component, and no table of powers, full row or fold is left.  A lane owns a
// particle; the matrix unit sums the lanes: v_mfma_f64_4x4x4 adds, for its row
// i, sum_k A[i][k] B[k][j] over lanes j + 4b + 16k, and with A one in row h % 4
// and zero elsewhere component h of 16 particle groups lands in row h % 4 of
// accumulator h / 4, over all passes of a leaf; the 16 sums of a component are
// added through LDS at the end.  One wavefront per leaf.  FP64 operations bound
// it at high p.  2 x 10^6 quadrupoles, p 10: 566 -> 129 us; 10^6 dipoles, p 6: 136 ->
// 46; 100k dipoles, p 10: 45 -> 19; 400k charges in leaves of 7, p 10, where most
// lanes idle: 181 -> 148; one leaf of 1000 charges, p 10: 98 -> 35.
template <int H0, int L>
__device__ __forceinline__ void p2m_add(const double *G, const double *sel, double *acc)
{
#pragma unroll
    for (int j = 0; j <= 2 * L; ++j) {
        const int h = L * L + j - H0;
        acc[h / 4] = __builtin_amdgcn_mfma_f64_4x4x4f64(sel[h % 4], G[j], acc[h / 4], 0, 0, 0);
    }
}

// orders l.. <= p of a source of order K, F1 = order l - 1
template <int K, int H0, int PB, int l>
__device__ __forceinline__ void p2m_orders(const double *F1, double x, double y, double z, int p, const double *sel,
                                           double *acc)
{
    if constexpr (l <= PB) {
        if (l > p) return;
        const double hx = x * (1.0 / (l - K)), hy = y * (1.0 / (l - K)), hz = z * (1.0 / (l - K));
        double F0[2 * l + 1];
#pragma unroll
        for (int j = 0; j <= 2 * l; ++j) {
            const int t = (j + 1) / 2, r = j == 0 ? 0 : j - (2 * t - 1), a = l - t, b = t - r;
            double v = 0.0;
            if (a >= 1) v = hx * hat(F1, a - 1, b, r);
            if (b >= 1) v = fma(hy, hat(F1, a, b - 1, r), v);
            if (hat_dz_any(a, b, r)) v = fma(hz, hat_dz(F1, a, b, r), v);
            F0[j] = v;
        }
        p2m_add<H0, l>(F0, sel, acc);
        p2m_orders<K, H0, PB, l + 1>(F0, x, y, z, p, sel, acc);
    }
}

template <int K, int H0, int PB>
__device__ __forceinline__ void p2m_source(const double *G, double x, double y, double z, int p, const double *sel,
                                           double *acc)
{
    if constexpr (K <= PB) {
        if (K > p) return;
        p2m_add<H0, K>(G, sel, acc);
        p2m_orders<K, H0, PB, K + 1>(G, x, y, z, p, sel, acc);
    }
}

// p <= PB
template <int MASK, int PB>
__global__ __launch_bounds__(64) void p2m_harmonic_kernel(int p, const int32_t *__restrict__ leaves,
                                                          const DevCell *__restrict__ cells, Geo g,
                                                          const double *__restrict__ xs, int n,
                                                          const double *__restrict__ mom_user,
                                                          const int32_t *__restrict__ perm, double *__restrict__ mom64,
                                                          float *__restrict__ mom32, int nhp, float *__restrict__ Mh32,
                                                          double *__restrict__ Mh64)
{
    constexpr int W = mask_width(MASK), S = mask_min_order(MASK), H0 = hterms(S - 1);
    constexpr int NG = (hterms(PB) - H0 + 3) / 4;
    __shared__ double red[NG * 64];
    const int lane = threadIdx.x;
    const int c = leaves[blockIdx.x];
    const DevCell cell = cells[c];
    double z[3];
    cell_center(cell, g.lo, g.h, z);
    const double ir = 1.0 / cell_radius(cell.level, g.h);
    double sel[4], acc[NG];
#pragma unroll
    for (int k = 0; k < 4; ++k) sel[k] = (lane & 3) == k ? 1.0 : 0.0;
#pragma unroll
    for (int k = 0; k < NG; ++k) acc[k] = 0.0;
    for (int base = 0; base < cell.count; base += 64) {
        // lanes past the leaf's end add zeros
        const bool on = base + lane < cell.count;
        const size_t i = (size_t)cell.first + base + lane;
        double x = 0.0, y = 0.0, w = 0.0, m[W];
#pragma unroll
        for (int k = 0; k < W; ++k) m[k] = 0.0;
        if (on) {
            const double *src = mom_user + (size_t)perm[i] * W;
#pragma unroll
            for (int k = 0; k < W; ++k) m[k] = src[k];
            sort_moments(i, MASK, m, mom64, mom32);
            x = (z[0] - xs[i]) * ir;
            y = (z[1] - xs[(size_t)n + i]) * ir;
            w = (z[2] - xs[2 * (size_t)n + i]) * ir;
        }
        int off = 0;
        if constexpr (MASK & 1) {
            const double G[1] = {m[off++]};
            p2m_source<0, H0, PB>(G, x, y, w, p, sel, acc);
        }
        if constexpr (MASK & 2) {
            const double G[3] = {-m[off] * ir, -m[off + 1] * ir, -m[off + 2] * ir};
            off += 3;
            p2m_source<1, H0, PB>(G, x, y, w, p, sel, acc);
        }
        if constexpr (MASK & 4) {
            // S_m = Q_m / m!; (0,0,2) folds onto -(2,0,0) and -(0,2,0)
            const double ir2 = ir * ir, zz = 0.5 * m[off + 5];
            const double G[5] = {(0.5 * m[off] - zz) * ir2, m[off + 1] * ir2, m[off + 2] * ir2,
                                 (0.5 * m[off + 3] - zz) * ir2, m[off + 4] * ir2};
            off += 6;
            p2m_source<2, H0, PB>(G, x, y, w, p, sel, acc);
        }
        if constexpr (MASK & 8) {
            // S_m = -O_m / m!; (1,0,2) folds onto -(3,0,0) and -(1,2,0), (0,1,2)
            // onto -(2,1,0) and -(0,3,0), (0,0,3) onto -(2,0,1) and -(0,2,1)
            const double ir3 = -(ir * ir * ir), *o = m + off;
            const double xzz = 0.5 * o[5], yzz = 0.5 * o[8], zzz = o[9] * (1.0 / 6);
            const double G[7] = {(o[0] * (1.0 / 6) - xzz) * ir3, (0.5 * o[1] - yzz) * ir3, (0.5 * o[2] - zzz) * ir3,
                                 (0.5 * o[3] - xzz) * ir3,       o[4] * ir3,               (o[6] * (1.0 / 6) - yzz) * ir3,
                                 (0.5 * o[7] - zzz) * ir3};
            p2m_source<3, H0, PB>(G, x, y, w, p, sel, acc);
        }
    }
#pragma unroll
    for (int k = 0; k < NG; ++k) red[k * 64 + lane] = acc[k];
    __syncthreads();
    const int nh = hterms(p) - H0;
    for (int h = lane; h < nh; h += 64) {
        // component h: 16 lanes of accumulator h / 4, from another one each
        // lane so that they spread over the banks
        double v = 0.0;
#pragma unroll
        for (int k = 0; k < 16; ++k) v += red[h * 16 + ((k + h) & 15)];
        if (Mh32) Mh32[(size_t)c * nhp + h] = (float)v;
        Mh64[(size_t)c * nhp + h] = v;
    }
}

template <int MASK, int PB>
static void p2m_launch_harmonic(fmm_tree *t, const Geo &g, const HarmOut &ho, hipStream_t s)
{
    hipLaunchKernelGGL((p2m_harmonic_kernel<MASK, PB>), dim3((unsigned)t->nleaves), dim3(64), 0, s, t->p, t->d_leaves,
                       t->d_cells, g, t->d_x, (int)t->ht.n, t->mom_user, t->d_perm, t->d_mom, t->d_mom32, ho.nhp,
                       ho.h32, ho.h64);
}

template <int MASK>
static void p2m_launch(fmm_tree *t, hipStream_t s)
{
    Geo g{{t->ht.lo[0], t->ht.lo[1], t->ht.lo[2]}, t->ht.h};
    const int nmp = (nterms(t->p) - nterms(t->order - 1) + 3) / 4 * 4;
    float *m32 = t->prec == FMM_PREC_MIXED ? t->d_M32 : nullptr;
    const HarmOut ho = harm_out(t);
    if (ho.h64) {
        // registers and LDS by the highest order a kernel takes
        if (t->p <= 4) p2m_launch_harmonic<MASK, 4>(t, g, ho, s);
        else if (t->p <= 6) p2m_launch_harmonic<MASK, 6>(t, g, ho, s);
        else if (t->p <= 8) p2m_launch_harmonic<MASK, 8>(t, g, ho, s);
        else p2m_launch_harmonic<MASK, FMM_P_MAX>(t, g, ho, s);
        return;
    }
    if constexpr (!(MASK & 4) || (MASK & 8)) {
        hipLaunchKernelGGL(p2m_coef_kernel<MASK>, dim3((unsigned)t->nleaves), dim3(kP2MThreads), 0, s, t->p, nmp,
                           t->d_leaves, t->d_cells, g, t->d_x, (int)t->ht.n, t->mom_user, t->d_perm, t->d_mom,
                           t->d_mom32, t->d_M64, m32);
        return;
    }
    const int S = t->order;
    const int blk = kP2MPlanHost.blk[t->p][S], nitems = kP2MPlanHost.nitems[t->p][S];
    const int ngroups = kP2MPlanHost.ngroups[t->p][S];
    hipLaunchKernelGGL(p2m_kernel<MASK>, dim3((unsigned)t->nleaves), dim3(kP2MThreads), 0, s, t->p, nmp, blk, nitems,
                       ngroups, t->d_leaves,
                       t->d_cells, g, t->d_x, (int)t->ht.n, t->mom_user, t->d_perm, t->d_mom, t->d_mom32,
                       t->d_M64, m32);
}

hipError_t launch_p2m(fmm_tree *t, hipStream_t s)
{
    switch (t->smask) {
    case 1: p2m_launch<1>(t, s); break;
    case 2: p2m_launch<2>(t, s); break;
    case 3: p2m_launch<3>(t, s); break;
    case 4: p2m_launch<4>(t, s); break;
    case 5: p2m_launch<5>(t, s); break;
    case 6: p2m_launch<6>(t, s); break;
    case 7: p2m_launch<7>(t, s); break;
    case 8: p2m_launch<8>(t, s); break;
    case 9: p2m_launch<9>(t, s); break;
    case 10: p2m_launch<10>(t, s); break;
    case 11: p2m_launch<11>(t, s); break;
    case 12: p2m_launch<12>(t, s); break;
    case 13: p2m_launch<13>(t, s); break;
    case 14: p2m_launch<14>(t, s); break;
    case 15: p2m_launch<15>(t, s); break;
    default: return hipErrorInvalidValue;
    }
    return hipGetLastError();
}

// ------------------------------------------------------------------ M2M / L2L
// Both shifts are fixed sparse matrices whose entries change sign from octant to
// octant only by the parities x of n - m: a character of the octant, (-1)^(x.c)
// (gen_shift.py, which writes the matrices).  So a parent's children share one
// product: M2M takes for every class x the children's rows summed under its
// character, L2L sums every class once and combines the eight sums for each
// child.  Eight lanes work on one component, lane x on class x; before (M2M) or
// after (L2L) the product the same lanes stand for the octants, and the change
// between the two is an eight-point Walsh-Hadamard transform over them.
//
// A level takes as long as its chain of loads (parent, children, rows) when it
// has few parents, and its table reads when it has many.  2608 products a
// parent at p 10 in the harmonic basis (8008 with every component), against
// three passes along the axes of every child's whole row with an index
// computed for each term before.  All levels together, M2M and L2L: p 10 dipoles,
// 4096 leaves of an even tree 51 and 38 -> 24 and 21 us; 10^6 Plummer
// dipoles, p 6, nine levels 150 and 144 -> 79 and 75; 2 x 10^6 quadrupoles, p 10, 320 and
// 171 -> 80 and 62.
constexpr int kShiftThreads = 256;
#include "shift_tables.h"
static_assert(kShiftOrders == FMM_P_MAX, "the shift tables end at another order");

__device__ __forceinline__ double octant_transform(double v, int lane)
{
#pragma unroll
    for (int m = 1; m < 8; m <<= 1) {
        const double o = __shfl_xor(v, m);
        v = (lane & m) ? o - v : v + o;
    }
    return v;
}

// sum of val[e] src[idx[e] - first] over the entries [b, e)
__device__ __forceinline__ double shift_row(const uint16_t *__restrict__ idx, const double *__restrict__ val, int b,
                                            int e, const double *src, int first)
{
    double acc = 0.0;
#pragma unroll 4
    for (int i = b; i < e; ++i) acc = fma(val[i], src[idx[i] - first], acc);
    return acc;
}

// children of `P` by octant: slot[c] = the child's cell, -1 where there is none
__device__ __forceinline__ void shift_children(const DevCell *__restrict__ cells, int P, int *slot)
{
    const int tid = threadIdx.x;
    if (tid < 8) slot[tid] = -1;   // one wavefront writes both, in order
    const int nch = cells[P].nchild, kid0 = cells[P].child0;
    __builtin_amdgcn_wave_barrier();
    if (tid < nch) {
        const DevCell cc = cells[kid0 + tid];
        slot[(cc.ix & 1) << 2 | (cc.iy & 1) << 1 | (cc.iz & 1)] = kid0 + tid;
    }
}

// rows of n components from the order s on, `stride` apart; Ms: FP32 copy or null
template <bool HARM>
__global__ __launch_bounds__(kShiftThreads) void m2m_kernel(int s, int n, int stride,
                                                            const int32_t *__restrict__ parents,
                                                            const DevCell *__restrict__ cells, double *__restrict__ M,
                                                            float *__restrict__ Ms)
{
    extern __shared__ double W[];   // [8][n]
    __shared__ int slot[8];
    const int P = parents[blockIdx.x], x = threadIdx.x & 7;
    const int first = HARM ? hterms(s - 1) : nterms(s - 1);
    shift_children(cells, P, slot);
    __syncthreads();
    const int kid = slot[x];
    // eight lanes of a component leave a loop together
    for (int h = threadIdx.x >> 3; h < n; h += kShiftThreads / 8)
        W[x * n + h] = octant_transform(kid >= 0 ? M[(size_t)kid * stride + h] : 0.0, x);
    __syncthreads();
    for (int h = threadIdx.x >> 3; h < n; h += kShiftThreads / 8) {
        const uint16_t *off = HARM ? kM2MH_off[(h + first) * 8 + x] : kM2MF_off[(h + first) * 8 + x];
        double v = shift_row(HARM ? kM2MH_idx : kM2MF_idx, HARM ? kM2MH_val : kM2MF_val, off[s], off[kShiftOrders + 1],
                             W + x * n, first);
#pragma unroll
        for (int m = 1; m < 8; m <<= 1) v += __shfl_xor(v, m);
        if (x == 0) M[(size_t)P * stride + h] = v;
        if (x == 1 && Ms) Ms[(size_t)P * stride + h] = (float)v;
    }
}

hipError_t launch_m2m_level(fmm_tree *t, int level, hipStream_t s)
{
    const int a = t->level_nonleaf_ptr[level], b = t->level_nonleaf_ptr[level + 1];
    if (b <= a) return hipSuccess;
    const HarmOut ho = harm_out(t);
    if (ho.h64) {
        const int n = hterms(t->p) - hterms(t->order - 1);
        hipLaunchKernelGGL(m2m_kernel<true>, dim3(b - a), dim3(kShiftThreads), 8 * n * sizeof(double), s, t->order, n,
                           ho.nhp, t->d_nonleaf + a, t->d_cells, ho.h64, ho.h32);
    } else {
        const int n = nterms(t->p) - nterms(t->order - 1);
        hipLaunchKernelGGL(m2m_kernel<false>, dim3(b - a), dim3(kShiftThreads), 8 * n * sizeof(double), s, t->order, n,
                           (n + 3) / 4 * 4, t->d_nonleaf + a, t->d_cells, t->d_M64,
                           t->prec == FMM_PREC_MIXED ? t->d_M32 : nullptr);
    }
    return hipGetLastError();
}

// locals: rows of n components, up to the order q
template <bool HARM>
__global__ __launch_bounds__(kShiftThreads) void l2l_kernel(int q, int n, const int32_t *__restrict__ parents,
                                                            const DevCell *__restrict__ cells, double *__restrict__ L)
{
    extern __shared__ double row[];   // [n], the parent's
    __shared__ int slot[8];
    const int P = parents[blockIdx.x], x = threadIdx.x & 7;
    shift_children(cells, P, slot);
    for (int h = threadIdx.x; h < n; h += kShiftThreads) row[h] = L[(size_t)P * n + h];
    __syncthreads();
    const int kid = slot[x];
    for (int h = threadIdx.x >> 3; h < n; h += kShiftThreads / 8) {
        const double old = kid >= 0 ? L[(size_t)kid * n + h] : 0.0;
        const uint16_t *off = HARM ? kL2LH_off[h * 8 + x] : kL2LF_off[h * 8 + x];
        const double v = octant_transform(
            shift_row(HARM ? kL2LH_idx : kL2LF_idx, HARM ? kL2LH_val : kL2LF_val, off[0], off[q + 1], row, 0), x);
        if (kid >= 0) L[(size_t)kid * n + h] = old + v;
    }
}

// children at `level` receive from their parents at level - 1
hipError_t launch_l2l_level(fmm_tree *t, int level, hipStream_t s)
{
    const int a = t->level_nonleaf_ptr[level - 1], b = t->level_nonleaf_ptr[level];
    if (b <= a) return hipSuccess;
    const int q = t->p - t->order;
    const bool harm = t->basis == FMM_M2L_HARMONIC;
    const int n = harm ? hterms(q) : nterms(q);
    hipLaunchKernelGGL(harm ? l2l_kernel<true> : l2l_kernel<false>, dim3(b - a), dim3(kShiftThreads),
                       n * sizeof(double), s, q, n, t->d_nonleaf + a, t->d_cells, t->d_L64);
    return hipGetLastError();
}


#include "p2p_kernel.h"

static hipError_t launch_p2p_range(fmm_tree *t, hipStream_t s, bool grad, int first, int count,
                                   double *near_g = nullptr);

hipError_t launch_p2p(fmm_tree *t, hipStream_t s, bool grad, double *near_g)
{
    return launch_p2p_range(t, s, grad, 0, -1, near_g);
}

hipError_t launch_p2p_part(fmm_tree *t, hipStream_t s, int first, int count)
{
    return launch_p2p_range(t, s, false, first, count);
}

// Near-field gradient of the allocation-free fmm_evaluate_grad variant: every
// particle's six values are written by the gradient pass before the L2P reads
// them, so nothing needs clearing between calls.  Calls that overlap on one
// device share it and race.
static __device__ __align__(256) double scratch[(size_t)kNoAllocMaxN * 6];

hipError_t noalloc_scratch(int device, double **ptr)
{
    constexpr int kMaxDevices = 64;
    static std::mutex mu;
    static double *addr[kMaxDevices] = {};
    if (device < 0 || device >= kMaxDevices) return hipErrorInvalidDevice;
    std::lock_guard<std::mutex> lk(mu);
    if (!addr[device]) {
        // each device holds its own copy of the array; its host-side name is
        // no device address, so kernels get this one
        void *p = nullptr;
        const hipError_t e = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch));
        if (e != hipSuccess) return e;
        addr[device] = (double *)p;
    }
    *ptr = addr[device];
    return hipSuccess;
}

static hipError_t launch_p2p_range(fmm_tree *t, hipStream_t s, bool grad, int first, int count, double *near_g)
{
    if (count < 0) count = (int)t->nleaves - first;
    if (first < 0 || count < 0 || first + count > t->nleaves) return hipErrorInvalidValue;
    if (count == 0) return hipSuccess;
    P2PArgs a;
    a.leaves = t->d_leaves;
    a.ptr = t->d_p2p_ptr;
    a.src = t->d_p2p_src;
    a.cells = t->d_cells;
    for (int d = 0; d < 3; ++d) a.lo[d] = t->ht.lo[d];
    a.m32 = t->d_mom32;
    a.xs = t->d_x;
    a.m64 = t->d_mom;
    a.near = t->d_near;
    a.near_g = near_g ? near_g : t->d_near_g;
    a.n = (int)t->ht.n;
    a.h = t->ht.h;
    a.order = t->d_p2p_order + first;
    const bool f32 = t->prec == FMM_PREC_MIXED;
    if (!p2p_dispatch_lo(t->smask, f32, grad, (unsigned)count, s, a) &&
        !p2p_dispatch_oct(t->smask, f32, grad, (unsigned)count, s, a))
        return hipErrorInvalidValue;
    return hipGetLastError();
}

// ------------------------------------------------------------------ L2P
// phi = (1/r) sum_{|n|<=q} eta^n/n! L~_n, E_d = -(1/r^2) sum eta^n/n! L~_{n+e_d}
// (Eq. 9, Eq. 10 with |k| = 1), eta = (x - z)/r, plus the near field, written
// to the caller's particle order.  One wave per pack of consecutive leaves
// holding at most 64 particles together (the host packs them, so that most
// lanes work although leaves hold ~ncrit/3 particles on average).  Each
// leaf's L~ is unpacked into LDS, zero beyond the simplex, so that for fixed
// (n_x, n_y) the sums over n_z of L~_n and of its neighbours n + e_d (+ e_d')
// are unit-stride from one base each; the loop structure is the same for
// every lane.  Two layouts (COLS):
// - a dense (q+2)^3 cube: the neighbours sit at fixed offsets from the base,
//   immediates of the LDS reads;
// - packed columns: for every (n_x, n_y) with n_x + n_y <= q + 2 the entries
//   n_z = 0 .. q + 2 - n_x - n_y lie contiguously, (q+3)(q+4)(q+5)/6 values,
//   a third of the cube, but each neighbour column costs an address add.
// The columns are used when they pack more leaves into a wave than the cube
// (high orders, where one leaf's cube fills the 16 KB budget: at p - s = 9
// a cube is 10.6 KB and a wave would take one leaf of ~24 particles), or when
// the cube's LDS share limits the resident waves (1M particles and more,
// where they are about 25 % faster); the cube otherwise.  The leaves per pack
// are what a 16 KB budget of the layout allows.
// This is the kernel of the full basis (harmonic rows: l2p_harmonic_kernel).
// Compiled per q = p - s.
constexpr int kL2PMaxLeaves = 8;
constexpr int kL2PPackBudget = 16384;   // bytes of (q+2)^3 cubes that fix the leaves per pack

// values of one leaf's columns, and the start of column (x, y) (K = q + 3:
// column (x', y') holds K - x' - y' values)
__host__ __device__ constexpr int l2p_cols(int q) { return (q + 3) * (q + 4) * (q + 5) / 6; }
__host__ __device__ constexpr int l2p_col(int q, int x, int y)
{
    const int K = q + 3, kx = K - x;
    return K * (K + 1) * (K + 2) / 6 - kx * (kx + 1) * (kx + 2) / 6 + y * kx - y * (y - 1) / 2;
}
__host__ __device__ constexpr int l2p_cube(int q) { return (q + 2) * (q + 2) * (q + 2); }
int l2p_pack_limit(int q, bool cols)
{
    return std::max(1, std::min(kL2PMaxLeaves, kL2PPackBudget / (8 * (cols ? l2p_cols(q) : l2p_cube(q)))));
}
int l2p_harmonic_leaves() { return kL2PMaxLeaves; }
constexpr int kLdsPerCU = 160 * 1024;
bool l2p_columns_pay(int q, int npacks, int ncu)
{
    const int cube_bytes = l2p_pack_limit(q, false) * l2p_cube(q) * 8;
    return (int64_t)npacks > (int64_t)ncu * std::max(1, kLdsPerCU / cube_bytes);
}

// GRAD: also the field gradient, -(1/r^3) sum_{|n|<=q-2} eta^n/n! L~_{n+e_i+e_j}
// (the second derivatives of the expansion, the general-k form of Eq. 10),
// plus the near field's gradient; its sums read the same cube (indices stay
// inside the simplex, so no larger edge is needed)
template <int Q, bool GRAD, bool COLS>
__global__ __launch_bounds__(64) void l2p_kernel(int outputs, const int32_t *__restrict__ pack,
                                                 const int32_t *__restrict__ leaves, const DevCell *__restrict__ cells,
                                                 Geo g, const double *__restrict__ xs, int n,
                                                 const double *__restrict__ L, const double *__restrict__ near, const int32_t *__restrict__ perm,
                                                 double *__restrict__ phi, double *__restrict__ field,
                                                 const double *__restrict__ near_g, double *__restrict__ grad)
{
    constexpr int NL = nterms(Q);
    constexpr int E = Q + 2;                     // cube edge: room for n + e_d
    constexpr int NC = COLS ? l2p_cols(Q) : E * E * E;   // values per leaf
    // start of the n_z run of (x, y)
    auto at = [](int x, int y) { return COLS ? l2p_col(Q, x, y) : (x * E + y) * E; };
    extern __shared__ double cubes[];            // one cube or set of columns per leaf of the pack
    __shared__ int lfirst[kL2PMaxLeaves], lstart[kL2PMaxLeaves + 1];
    __shared__ double lgeo[kL2PMaxLeaves][4];    // centre, 1 / radius
    const int p0 = pack[blockIdx.x], nlv = pack[blockIdx.x + 1] - p0;
    for (int i = threadIdx.x; i < nlv * NC; i += blockDim.x) cubes[i] = 0.0;
    if ((int)threadIdx.x < nlv) {
        const DevCell c = cells[leaves[p0 + threadIdx.x]];
        double z[3];
        cell_center(c, g.lo, g.h, z);
        lfirst[threadIdx.x] = c.first;
        lstart[threadIdx.x + 1] = c.count;
        lgeo[threadIdx.x][0] = z[0];
        lgeo[threadIdx.x][1] = z[1];
        lgeo[threadIdx.x][2] = z[2];
        lgeo[threadIdx.x][3] = 1.0 / cell_radius(c.level, g.h);
    }
    __syncthreads();
    if (threadIdx.x == 0) {
        lstart[0] = 0;
        for (int q = 0; q < nlv; ++q) lstart[q + 1] += lstart[q];
    }
    for (int q = 0; q < nlv; ++q) {
        const size_t c = (size_t)leaves[p0 + q];
        for (int i = threadIdx.x; i < NL; i += blockDim.x) {
            const MultiIndex nn = k_mi.v[i];
            cubes[q * NC + at(nn.x, nn.y) + nn.z] = L[c * NL + i];
        }
    }
    __syncthreads();
    const int tot = lstart[nlv];
    for (int k = threadIdx.x; k < tot; k += blockDim.x) {
        int q = 0;
        while (q + 1 < nlv && k >= lstart[q + 1]) ++q;
        const int i = lfirst[q] + (k - lstart[q]);
        const double *cube = cubes + q * NC;
        const double ir = lgeo[q][3];
        const double ex = (xs[i] - lgeo[q][0]) * ir, ey = (xs[n + i] - lgeo[q][1]) * ir,
                     ez = (xs[2 * (size_t)n + i] - lgeo[q][2]) * ir;
        double pz[Q + 1];
        pz[0] = 1.0;
#pragma unroll
        for (int a = 1; a <= Q; ++a) pz[a] = pz[a - 1] * ez * (1.0 / a);
        double ph = 0.0, fx = 0.0, fy = 0.0, fz = 0.0;
        double G[6] = {0.0, 0.0, 0.0, 0.0, 0.0, 0.0};   // xx, xy, xz, yy, yz, zz
        double px = 1.0;
#pragma unroll 1
        for (int nx = 0; nx <= Q; ++nx) {
            if (nx) px *= ex * k_inv.v[nx];
            double py = px;
#pragma unroll 1
            for (int ny = 0; ny <= Q - nx; ++ny) {
                if (ny) py *= ey * k_inv.v[ny];
                // columns (nx, ny), (nx+1, ny), (nx, ny+1) and, for the
                // gradient, (nx+2, ny), (nx+1, ny+1), (nx, ny+2)
                const double *b = cube + at(nx, ny);
                const double *bx = cube + at(nx + 1, ny), *by = cube + at(nx, ny + 1);
                const int lim = Q - nx - ny;
                // entries beyond the simplex are zero, so the field sums may
                // run to the same bound as the potential sum
                double tp = 0.0, tx = 0.0, ty = 0.0, tz = 0.0;
#pragma unroll
                for (int nz = 0; nz <= Q; ++nz) {
                    if (nz > lim) break;
                    tp = fma(pz[nz], b[nz], tp);
                    tx = fma(pz[nz], bx[nz], tx);
                    ty = fma(pz[nz], by[nz], ty);
                    tz = fma(pz[nz], b[nz + 1], tz);
                }
                ph = fma(py, tp, ph);
                fx = fma(py, tx, fx);
                fy = fma(py, ty, fy);
                fz = fma(py, tz, fz);
                if constexpr (GRAD) {
                    double tg[6] = {0.0, 0.0, 0.0, 0.0, 0.0, 0.0};
                    const double *bxx = cube + at(nx + 2, ny), *bxy = cube + at(nx + 1, ny + 1),
                                 *byy = cube + at(nx, ny + 2);
#pragma unroll
                    for (int nz = 0; nz + 2 <= Q; ++nz) {
                        if (nz > lim - 2) break;
                        tg[0] = fma(pz[nz], bxx[nz], tg[0]);
                        tg[1] = fma(pz[nz], bxy[nz], tg[1]);
                        tg[2] = fma(pz[nz], bx[nz + 1], tg[2]);
                        tg[3] = fma(pz[nz], byy[nz], tg[3]);
                        tg[4] = fma(pz[nz], by[nz + 1], tg[4]);
                        tg[5] = fma(pz[nz], b[nz + 2], tg[5]);
                    }
#pragma unroll
                    for (int c = 0; c < 6; ++c) G[c] = fma(py, tg[c], G[c]);
                }
            }
        }
        const double *nr = near + 4 * (size_t)i;
        const size_t o = (size_t)perm[i];
        if (outputs & FMM_POT) phi[o] = ph * ir + nr[0];
        if (outputs & FMM_FIELD) {
            const double ir2 = ir * ir;
            field[3 * o] = -fx * ir2 + nr[1];
            field[3 * o + 1] = -fy * ir2 + nr[2];
            field[3 * o + 2] = -fz * ir2 + nr[3];
        }
        if constexpr (GRAD) {
            const double ir3 = ir * ir * ir;
            const double *ng = near_g + 6 * (size_t)i;
#pragma unroll
            for (int c = 0; c < 6; ++c) grad[6 * o + c] = -G[c] * ir3 + ng[c];
        }
    }
}

// Harmonic basis: the expansion is sum_h L~_h F_h (the functions of a harmonic
// row, above P2M), the gradient of order l is entries of order l - 1, and Euler's
// identity gives the next order, and the potential of each order from its field.
// One pass over the row then reads every coefficient once and has nothing to
// rebuild; the second derivatives come from order l - 2, and
// zz = -xx - yy.  The sums over monomials read each coefficient four times from
// LDS, which bound them: 2 x 10^6 targets, q 8: 475 -> 102 us; 10^6, q 5: 74 -> 33;
// 100k, q 9: 59 -> 14.  With the gradient, 400k targets: q 4 48 -> 30 us, q 8 200 ->
// 71, q 10 332 -> 148 (there the orders no longer fit the registers).  What bounds
// it now: the FP64 operations at high q, the targets' own traffic at low q.
struct L2PSums {
    double ph, fx, fy, fz, gxx, gxy, gxz, gyy, gyz;
};

// orders l.. of the row: F1, F2 hold the orders l - 1 and l - 2 (one array an
// order, so that all stay in registers)
template <int Q, bool GRAD, int l>
__device__ __forceinline__ void l2p_orders(const double *row, const double *F1, const double *F2, double ex, double ey,
                                           double ez, L2PSums &o)
{
    if constexpr (l <= Q) {
        const double hx = ex * (1.0 / l), hy = ey * (1.0 / l), hz = ez * (1.0 / l);
        double sx = 0.0, sy = 0.0, sz = 0.0;
        double F0[2 * l + 1];
#pragma unroll
        for (int j = 0; j <= 2 * l; ++j) {
            const int t = (j + 1) / 2, r = j == 0 ? 0 : j - (2 * t - 1), a = l - t, b = t - r;
            const double c = row[l * l + j];
            const double dx = hat(F1, a - 1, b, r), dy = hat(F1, a, b - 1, r), dz = hat_dz(F1, a, b, r);
            // terms that are zero by their indices are left out
            const bool zx = a >= 1, zy = b >= 1, zz = hat_dz_any(a, b, r);
            if (l < Q) {
                double v = 0.0;
                if (zx) v = hx * dx;
                if (zy) v = fma(hy, dy, v);
                if (zz) v = fma(hz, dz, v);
                F0[j] = v;
            }
            if (zx) sx = fma(c, dx, sx);
            if (zy) sy = fma(c, dy, sy);
            if (zz) sz = fma(c, dz, sz);
            if constexpr (GRAD && l >= 2) {
                if (a >= 2) o.gxx = fma(c, hat(F2, a - 2, b, r), o.gxx);
                if (zx && zy) o.gxy = fma(c, hat(F2, a - 1, b - 1, r), o.gxy);
                if (b >= 2) o.gyy = fma(c, hat(F2, a, b - 2, r), o.gyy);
                if (hat_dz_any(a - 1, b, r)) o.gxz = fma(c, hat_dz(F2, a - 1, b, r), o.gxz);
                if (hat_dz_any(a, b - 1, r)) o.gyz = fma(c, hat_dz(F2, a, b - 1, r), o.gyz);
            }
        }
        o.fx += sx;
        o.fy += sy;
        o.fz += sz;
        o.ph = fma(hx, sx, fma(hy, sy, fma(hz, sz, o.ph)));
        l2p_orders<Q, GRAD, l + 1>(row, F0, F1, ex, ey, ez, o);
    }
}

template <int Q, bool GRAD>
__global__ __launch_bounds__(64) void l2p_harmonic_kernel(int outputs, const int32_t *__restrict__ pack,
                                                          const int32_t *__restrict__ leaves,
                                                          const DevCell *__restrict__ cells, Geo g,
                                                          const double *__restrict__ xs, int n,
                                                          const double *__restrict__ L, const double *__restrict__ near,
                                                          const int32_t *__restrict__ perm, double *__restrict__ phi,
                                                          double *__restrict__ field, const double *__restrict__ near_g,
                                                          double *__restrict__ grad)
{
    constexpr int NH = hterms(Q);
    __shared__ double rows[kL2PMaxLeaves * NH];
    __shared__ int lfirst[kL2PMaxLeaves], lstart[kL2PMaxLeaves + 1];
    __shared__ double lgeo[kL2PMaxLeaves][4];    // centre, 1 / radius
    const int p0 = pack[blockIdx.x], nlv = pack[blockIdx.x + 1] - p0;
    if ((int)threadIdx.x < nlv) {
        const DevCell c = cells[leaves[p0 + threadIdx.x]];
        double z[3];
        cell_center(c, g.lo, g.h, z);
        lfirst[threadIdx.x] = c.first;
        lstart[threadIdx.x + 1] = c.count;
        lgeo[threadIdx.x][0] = z[0];
        lgeo[threadIdx.x][1] = z[1];
        lgeo[threadIdx.x][2] = z[2];
        lgeo[threadIdx.x][3] = 1.0 / cell_radius(c.level, g.h);
    }
    for (int q = 0; q < nlv; ++q) {
        const size_t c = (size_t)leaves[p0 + q];
        for (int h = threadIdx.x; h < NH; h += 64) rows[q * NH + h] = L[c * NH + h];
    }
    __syncthreads();
    if (threadIdx.x == 0) {
        lstart[0] = 0;
        for (int q = 0; q < nlv; ++q) lstart[q + 1] += lstart[q];
    }
    __syncthreads();
    const int tot = lstart[nlv];
    for (int k = threadIdx.x; k < tot; k += 64) {
        int q = 0;
        while (q + 1 < nlv && k >= lstart[q + 1]) ++q;
        const int i = lfirst[q] + (k - lstart[q]);
        const double *row = rows + q * NH;
        const double ir = lgeo[q][3];
        const double ex = (xs[i] - lgeo[q][0]) * ir, ey = (xs[n + i] - lgeo[q][1]) * ir,
                     ez = (xs[2 * (size_t)n + i] - lgeo[q][2]) * ir;
        L2PSums v{row[0], 0.0, 0.0, 0.0, 0.0, 0.0, 0.0, 0.0, 0.0};
        const double one[1] = {1.0};
        l2p_orders<Q, GRAD, 1>(row, one, one, ex, ey, ez, v);
        const double *nr = near + 4 * (size_t)i;
        const size_t o = (size_t)perm[i];
        if (outputs & FMM_POT) phi[o] = v.ph * ir + nr[0];
        if (outputs & FMM_FIELD) {
            const double ir2 = ir * ir;
            field[3 * o] = -v.fx * ir2 + nr[1];
            field[3 * o + 1] = -v.fy * ir2 + nr[2];
            field[3 * o + 2] = -v.fz * ir2 + nr[3];
        }
        if constexpr (GRAD) {
            const double ir3 = ir * ir * ir;
            const double *ng = near_g + 6 * (size_t)i;
            const double G[6] = {v.gxx, v.gxy, v.gxz, v.gyy, v.gyz, -(v.gxx + v.gyy)};
#pragma unroll
            for (int c = 0; c < 6; ++c) grad[6 * o + c] = -G[c] * ir3 + ng[c];
        }
    }
}

template <int Q, bool COLS>
static void l2p_launch_layout(fmm_tree *t, int outputs, double *phi, double *field, double *grad, hipStream_t s,
                              const double *near_g)
{
    Geo g{{t->ht.lo[0], t->ht.lo[1], t->ht.lo[2]}, t->ht.h};
    const size_t lds = (size_t)l2p_pack_limit(Q, COLS) * (COLS ? l2p_cols(Q) : l2p_cube(Q)) * sizeof(double);
    if constexpr (Q >= 2) {
        if (outputs & FMM_GRAD) {
            hipLaunchKernelGGL((l2p_kernel<Q, true, COLS>), dim3((unsigned)t->l2p_npacks), dim3(64), lds, s, outputs,
                               t->d_l2p_pack, t->d_leaves, t->d_cells, g, t->d_x, (int)t->ht.n, t->d_L64,
                               t->d_near, t->d_perm, phi, field, near_g, grad);
            return;
        }
    }
    hipLaunchKernelGGL((l2p_kernel<Q, false, COLS>), dim3((unsigned)t->l2p_npacks), dim3(64), lds, s, outputs,
                       t->d_l2p_pack, t->d_leaves, t->d_cells, g, t->d_x, (int)t->ht.n, t->d_L64, t->d_near,
                       t->d_perm, phi, field, nullptr, nullptr);
}

template <int Q>
static void l2p_launch(fmm_tree *t, int outputs, double *phi, double *field, double *grad, hipStream_t s,
                       const double *near_g)
{
    if (t->basis == FMM_M2L_HARMONIC) {
        Geo g{{t->ht.lo[0], t->ht.lo[1], t->ht.lo[2]}, t->ht.h};
        auto kernel = l2p_harmonic_kernel<Q, false>;
        if constexpr (Q >= 2)
            if (outputs & FMM_GRAD) kernel = l2p_harmonic_kernel<Q, true>;
        hipLaunchKernelGGL(kernel, dim3((unsigned)t->l2p_npacks), dim3(64), 0, s, outputs, t->d_l2p_pack, t->d_leaves,
                           t->d_cells, g, t->d_x, (int)t->ht.n, t->d_L64, t->d_near, t->d_perm, phi, field, near_g,
                           grad);
    } else if (t->l2p_columns) l2p_launch_layout<Q, true>(t, outputs, phi, field, grad, s, near_g);
    else l2p_launch_layout<Q, false>(t, outputs, phi, field, grad, s, near_g);
}

hipError_t launch_l2p_final(fmm_tree *t, int outputs, double *phi, double *field, double *grad, hipStream_t s,
                            const double *near_g)
{
    if ((outputs & FMM_GRAD) && t->p - t->order < 2) return hipErrorInvalidValue;
    if (!near_g) near_g = t->d_near_g;
    switch (t->p - t->order) {
    case 0: l2p_launch<0>(t, outputs, phi, field, grad, s, near_g); break;
    case 1: l2p_launch<1>(t, outputs, phi, field, grad, s, near_g); break;
    case 2: l2p_launch<2>(t, outputs, phi, field, grad, s, near_g); break;
    case 3: l2p_launch<3>(t, outputs, phi, field, grad, s, near_g); break;
    case 4: l2p_launch<4>(t, outputs, phi, field, grad, s, near_g); break;
    case 5: l2p_launch<5>(t, outputs, phi, field, grad, s, near_g); break;
    case 6: l2p_launch<6>(t, outputs, phi, field, grad, s, near_g); break;
    case 7: l2p_launch<7>(t, outputs, phi, field, grad, s, near_g); break;
    case 8: l2p_launch<8>(t, outputs, phi, field, grad, s, near_g); break;
    case 9: l2p_launch<9>(t, outputs, phi, field, grad, s, near_g); break;
    case 10: l2p_launch<10>(t, outputs, phi, field, grad, s, near_g); break;
    default: return hipErrorInvalidValue;
    }
    return hipGetLastError();
}

