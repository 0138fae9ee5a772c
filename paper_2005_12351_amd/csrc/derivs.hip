// Derivatives of the potential of order K = 1..3 at every particle (Pepper &
// Fangohr, arXiv 2005.12351, Section 2: the derivatives of the potential of
// order |k| follow from the local expansion, Eq. 10; the near field adds the
// same derivatives of the pair potentials).  For each multi-index k with
// |k| = K, in the index order of that order:
//   FMM far:  d^k phi = r^-(K+1) sum_{|n| <= q-K} eta^n/n! L~_{n+k},
//             eta = (x - z)/r, q = p - s, L~ the normalised local of the leaf;
//   BH far:   d^k phi = r^-(K+1) sum_{s <= |n| <= p} M~_n D_{n+k}(u),
//             u = (x - z_A)/r, for every cell the particle accepts (Eq. 6
//             differentiated K times, the traversal of Eq. 12);
//   near:     d^k phi = sum_j sum_{|m|=s} S_m D_{m+k}(x - x_j), S the source
//             tensor S_m = (-1)^|m| T_m / m! of the physical moment T, D the
//             derivatives of 1/r (Eq. 6 applied to a point source's own
//             expansion).
// FP64 throughout, from the tree's FP64 expansions and sorted FP64 moments,
// in both precisions of the tree.  FMM: one workgroup per leaf, its threads a
// (target, slice) grid as in the near-field kernels: the sources of the leaf's
// P2P list staged in LDS with their source tensors formed, each slice taking
// every ns-th of them, the pair's derivative tensor written out at compile
// time; the leaf's local row in LDS, the slices sharing out its terms.
// Barnes-Hut: one wavefront per particle; the wave walks the
// particle's traversal, builds an accepted cell's derivative tensor in LDS
// (one component per lane) and contracts it with the cell's multipole row
// (one term per lane), and splits an unaccepted leaf's sources over lanes.
#include <utility>

#include "fmm_internal.h"
#include "p2p_kernel.h"

namespace {

struct DerivArgs {
    P2PArgs near;          // leaves, P2P lists, dispatch order, cells, positions, moments, root geometry
    const int32_t *perm;
    const double *L;       // normalised locals, nl per cell (harmonic basis: nlh, the n_z <= 1 part)
    double *out;           // nk per particle, caller order
    int nl, nlh, q, w, smask;
};

// D_k(r) = d^k (1/|r|) by the Hermite form of the derivatives of f(r^2/2),
// f(u) = (2u)^-1/2:  d^k f = sum_{a <= k/2} prod_d c(k_d, a_d) x_d^(k_d-2a_d)
// f^(|k|-|a|)(u),  c(n, a) = n! / (2^a a! (n-2a)!),
// f^(j) = (-1)^j (2j-1)!! r^-(2j+1)
// c(n, a) for n <= FMM_P_MAX + 3 = 13, a <= 6
constexpr int kQMax = FMM_P_MAX + 3;
__constant__ double kHc[kQMax + 1][kQMax / 2 + 1] = {
    {1, 0, 0, 0, 0, 0, 0},           {1, 0, 0, 0, 0, 0, 0},
    {1, 1, 0, 0, 0, 0, 0},           {1, 3, 0, 0, 0, 0, 0},
    {1, 6, 3, 0, 0, 0, 0},           {1, 10, 15, 0, 0, 0, 0},
    {1, 15, 45, 15, 0, 0, 0},        {1, 21, 105, 105, 0, 0, 0},
    {1, 28, 210, 420, 105, 0, 0},    {1, 36, 378, 1260, 945, 0, 0},
    {1, 45, 630, 3150, 4725, 945, 0},  {1, 55, 990, 6930, 17325, 10395, 0},
    {1, 66, 1485, 13860, 51975, 62370, 10395},  {1, 78, 2145, 25740, 135135, 270270, 135135}};

__device__ __forceinline__ double hcoef(int n, int a) { return kHc[n][a]; }

template <int Q>
__device__ __forceinline__ double dtensor_k(int kx, int ky, int kz, const double (&px)[Q + 1],
                                            const double (&py)[Q + 1], const double (&pz)[Q + 1],
                                            const double (&F)[Q + 1])
{
    double acc = 0.0;
    const int kk = kx + ky + kz;
    for (int ax = 0; 2 * ax <= kx; ++ax)
        for (int ay = 0; 2 * ay <= ky; ++ay)
            for (int az = 0; 2 * az <= kz; ++az)
                acc += hcoef(kx, ax) * hcoef(ky, ay) * hcoef(kz, az) * px[kx - 2 * ax] * py[ky - 2 * ay] *
                       pz[kz - 2 * az] * F[kk - ax - ay - az];
    return acc;
}

// the source tensor of one order from its physical moments (S_0 = q,
// S_{e_i} = -mu_i, S_{e_i+e_j} = Q_ij / (e_i+e_j)!, S_m = -O_m / m! for an
// octupole), in the index order of that order
__device__ __forceinline__ void source_of(int s, const double *t, double (&S)[10])
{
    if (s == 3) {
        constexpr double kInvF[10] = {1.0 / 6, 0.5, 0.5, 0.5, 1.0, 0.5, 1.0 / 6, 0.5, 0.5, 1.0 / 6};
#pragma unroll
        for (int q = 0; q < 10; ++q) S[q] = -t[q] * kInvF[q];
    } else if (s == 0) {
        S[0] = t[0];
    } else if (s == 1) {
        S[0] = -t[0];
        S[1] = -t[1];
        S[2] = -t[2];
    } else {   // (2,0,0) (1,1,0) (1,0,1) (0,2,0) (0,1,1) (0,0,2)
        S[0] = 0.5 * t[0];
        S[1] = t[1];
        S[2] = t[2];
        S[3] = 0.5 * t[3];
        S[4] = t[4];
        S[5] = 0.5 * t[5];
    }
}

// multi-index number c of order K in the index order (n_x descending, then n_y)
__device__ __forceinline__ void mi_of(int K, int c, int &nx, int &ny, int &nz)
{
    nx = K;
    int left = c;
    while (left > K - nx) {
        left -= K - nx + 1;
        --nx;
    }
    ny = K - nx - left;
    nz = K - nx - ny;
}

// multi-index of position idx in the ordering by total order
__device__ __forceinline__ void mi_at(int idx, int &nx, int &ny, int &nz)
{
    int o = 0;
    while (nterms(o) <= idx) ++o;
    mi_of(o, idx - nterms(o - 1), nx, ny, nz);
}

// the K-th derivatives of the pair potentials of one source (every order
// its mask holds) at displacement (rx, ry, rz), added to acc
template <int K>
__device__ __forceinline__ void pair_derivs_add(double rx, double ry, double rz, const double *mj, int smask,
                                                const int (&kidx)[(K + 1) * (K + 2) / 2][3],
                                                double (&acc)[(K + 1) * (K + 2) / 2])
{
    constexpr int NK = (K + 1) * (K + 2) / 2;
    constexpr int Q = K + 3;                 // highest derivative order a pair needs (octupoles)
    const double r2 = rx * rx + ry * ry + rz * rz;
    const double ir = 1.0 / sqrt(r2), ir2 = ir * ir;
    double px[Q + 1], py[Q + 1], pz[Q + 1], F[Q + 1];
    px[0] = py[0] = pz[0] = 1.0;
    F[0] = ir;
#pragma unroll
    for (int d = 1; d <= Q; ++d) {
        px[d] = px[d - 1] * rx;
        py[d] = py[d - 1] * ry;
        pz[d] = pz[d - 1] * rz;
        F[d] = -F[d - 1] * (2.0 * d - 1.0) * ir2;
    }
    int off = 0;
    for (int s = 0; s < 4; ++s) {
        if (!(smask & (1 << s))) continue;
        double S[10];
        source_of(s, mj + off, S);
        off += (s + 1) * (s + 2) / 2;
        const int nm = (s + 1) * (s + 2) / 2;
        for (int mi = 0; mi < nm; ++mi) {
            int mx, my, mz;
            mi_of(s, mi, mx, my, mz);
#pragma unroll
            for (int c = 0; c < NK; ++c)
                acc[c] = fma(S[mi], dtensor_k<Q>(mx + kidx[c][0], my + kidx[c][1], mz + kidx[c][2], px, py, pz, F),
                             acc[c]);
        }
    }
}

// f(integral_constant<int, 0>) ... f(integral_constant<int, N - 1>)
template <typename F, int... I>
__device__ __forceinline__ void unrolled(F &&f, std::integer_sequence<int, I...>)
{
    (f(std::integral_constant<int, I>{}), ...);
}
template <int N, typename F>
__device__ __forceinline__ void unrolled(F &&f)
{
    unrolled(f, std::make_integer_sequence<int, N>{});
}

// multi-index number c of order k, at compile time
struct MI3 {
    int x, y, z;
};
constexpr MI3 mi_const(int k, int c)
{
    int x = k, left = c;
    while (left > k - x) {
        left -= k - x + 1;
        --x;
    }
    const int y = k - x - left;
    return MI3{x, y, k - x - y};
}
// c(n, a) = n! / (2^a a! (n - 2a)!) of the Hermite form
constexpr double hermite_const(int n, int a)
{
    double v = 1.0;
    for (int i = n; i > n - 2 * a; --i) v *= i;
    for (int i = 1; i <= a; ++i) v /= 2.0 * i;
    return v;
}

// acc[c] += sum_{|m|=S} T_m D_{m+k_c}(r), |k_c| = K: the K-th derivatives of
// the potential of one source of order S with source tensor T(m).  Only the
// derivative components of order S + K are formed, each as its Hermite sum
// with every index and coefficient a constant.
template <int K, int S, typename TF>
__device__ __forceinline__ void pair_derivs_const(double rx, double ry, double rz, double ir, TF &&T,
                                                  double (&acc)[(K + 1) * (K + 2) / 2])
{
    constexpr int Q = K + S, NQ = (Q + 1) * (Q + 2) / 2, NM = (S + 1) * (S + 2) / 2, NK = (K + 1) * (K + 2) / 2;
    const double ir2 = ir * ir;
    double px[Q + 1], py[Q + 1], pz[Q + 1], F[Q + 1], D[NQ];
    px[0] = py[0] = pz[0] = 1.0;
    F[0] = ir;
    unrolled<Q>([&](auto d_) {
        constexpr int d = decltype(d_)::value + 1;
        px[d] = d == 1 ? rx : px[d - 1] * rx;
        py[d] = d == 1 ? ry : py[d - 1] * ry;
        pz[d] = d == 1 ? rz : pz[d - 1] * rz;
        F[d] = F[d - 1] * (ir2 * -(2.0 * d - 1.0));
    });
    unrolled<NQ>([&](auto i_) {
        constexpr MI3 k = mi_const(Q, decltype(i_)::value);
        double v = 0.0;
        unrolled<(k.x / 2 + 1) * (k.y / 2 + 1) * (k.z / 2 + 1)>([&](auto t_) {
            constexpr int t = decltype(t_)::value;
            constexpr int az = t % (k.z / 2 + 1), ay = t / (k.z / 2 + 1) % (k.y / 2 + 1),
                          ax = t / (k.z / 2 + 1) / (k.y / 2 + 1);
            constexpr double c = hermite_const(k.x, ax) * hermite_const(k.y, ay) * hermite_const(k.z, az);
            v = fma(c * F[Q - ax - ay - az], px[k.x - 2 * ax] * py[k.y - 2 * ay] * pz[k.z - 2 * az], v);
        });
        D[decltype(i_)::value] = v;
    });
    unrolled<NM>([&](auto m_) {
        constexpr MI3 m = mi_const(S, decltype(m_)::value);
        const double t = T(decltype(m_)::value);
        unrolled<NK>([&](auto c_) {
            constexpr MI3 k = mi_const(K, decltype(c_)::value);
            acc[decltype(c_)::value] =
                fma(t, D[mindex(m.x + k.x, m.y + k.y, m.z + k.z) - nterms(Q - 1)], acc[decltype(c_)::value]);
        });
    });
}

// The derivatives of order K at every particle of a leaf.  What bounds it is
// FP64 issue: per pair about 100 operations for dipoles at K = 2.  The grid of
// 256 threads is (target, slice) with floor(256 / targets) slices, as in the
// near-field kernels, so leaves of 10 to 60 particles fill the workgroup.
// ONE >= 0: the only source order present; -1: any mask, told at run time.
// (An earlier form, one wave a leaf with run-time multi-indices, spent its
// time in index arithmetic and scratch memory: 9.44 ms for 20 011 dipoles at
// K = 2, ncrit 64, against 0.106 ms for this one.)
constexpr int kDT = kPT;      // threads per leaf
constexpr int kDChunk = 128;  // staged sources
template <int K, int ONE>
__global__ __launch_bounds__(kDT) void derivs_kernel(DerivArgs d)
{
    constexpr int NK = (K + 1) * (K + 2) / 2;
    constexpr int W = ONE < 0 ? 20 : (ONE + 1) * (ONE + 2) / 2;   // source tensor components staged
    constexpr int EMAX = FMM_P_MAX + 1;
    constexpr int kCube = EMAX * EMAX * EMAX;
    // one area for the leaf's local (a cube of edge q + 1 indexed by
    // multi-index), then the staged sources, then the slices' sums
    constexpr int kStage = (3 + W) * kDChunk, kRed = NK * kDT;
    constexpr int kArea = kCube > kStage ? (kCube > kRed ? kCube : kRed) : (kStage > kRed ? kStage : kRed);
    __shared__ double area[kArea];
    __shared__ int wstart[kPList], wfirst[kPList];
    __shared__ int sh[kPT / 64];
    __shared__ int wself;
    const P2PArgs &a = d.near;
    const int tid = threadIdx.x;
    const int lk = a.order[blockIdx.x];
    const int b = a.leaves[lk];
    const DevCell cb = a.cells[b];
    const int e0 = a.ptr[lk], e1 = a.ptr[lk + 1];
    const double r = ldexp(1.0, kMaxLevel - cb.level) * a.h;
    const double zb[3] = {a.lo[0] + (double)(2 * cb.ix + 1) * r, a.lo[1] + (double)(2 * cb.iy + 1) * r,
                          a.lo[2] + (double)(2 * cb.iz + 1) * r};
    const size_t n = a.n;
    const int E = d.q + 1;
    for (int tg0 = 0; tg0 < cb.count; tg0 += kDT) {
        const int cs = min(kDT, cb.count - tg0);
        const int ns = kDT / cs;
        const int t = tid % cs, sl = tid / cs;
        const bool act = sl < ns;
        const int i = cb.first + tg0 + t;
        const double x = a.xs[i], y = a.xs[n + i], z = a.xs[2 * n + i];
        double acc[NK];
#pragma unroll
        for (int c = 0; c < NK; ++c) acc[c] = 0.0;
        __syncthreads();
        // far field: Eq. 10 on the normalised local, the slices taking every
        // ns-th n_x
        for (int it = tid; it < d.nl; it += kDT) {
            int nx, ny, nz;
            mi_at(it, nx, ny, nz);
            double v;
            if (d.nlh > 0) {
                // harmonic basis: the row is rebuilt from its n_z <= 1 components,
                // (a, b, 2j + r) = (-1)^j sum_i C(j, i) (a + 2i, b + 2(j - i), r)
                const double *R = d.L + (size_t)b * d.nlh;
                const int j = nz >> 1, rr = nz & 1;
                double w = 1.0;
                v = 0.0;
                for (int k = 0; k <= j; ++k) {
                    v = fma(w, R[hindex(nx + 2 * k, ny + 2 * (j - k), rr)], v);
                    w = w * (j - k) / (k + 1);
                }
                if (j & 1) v = -v;
            } else {
                v = d.L[(size_t)b * d.nl + it];
            }
            area[(nx * E + ny) * E + nz] = v;
        }
        __syncthreads();
        if (act) {
            const double e[3] = {(x - zb[0]) / r, (y - zb[1]) / r, (z - zb[2]) / r};
            const int qk = d.q - K;
            int off[NK];
            unrolled<NK>([&](auto c_) {
                constexpr MI3 k = mi_const(K, decltype(c_)::value);
                off[decltype(c_)::value] = (k.x * E + k.y) * E + k.z;
            });
            double ax = 1.0;
            int done = 0;   // ax = e_x^done / done!
            for (int nx = sl; nx <= qk; nx += ns) {
                for (; done < nx; ++done) ax *= e[0] / (done + 1);
                double ay = ax;
                for (int ny = 0; nx + ny <= qk; ++ny) {
                    double az = ay;
                    for (int nz = 0; nx + ny + nz <= qk; ++nz) {
                        const double *c0 = area + (nx * E + ny) * E + nz;
#pragma unroll
                        for (int c = 0; c < NK; ++c) acc[c] = fma(az, c0[off[c]], acc[c]);
                        az *= e[2] / (nz + 1);
                    }
                    ay *= e[1] / (ny + 1);
                }
            }
            double sc = 1.0 / r;
            const double ir = sc;
#pragma unroll
            for (int k = 0; k < K; ++k) sc *= ir;
#pragma unroll
            for (int c = 0; c < NK; ++c) acc[c] *= sc;
        }
        // near field: every source of the leaf's P2P list but the target
        for (int w0 = e0; w0 < e1; w0 += kPList) {
            const int nw = min(kPList, e1 - w0);
            __syncthreads();
            if (tid == 0) wself = -1;
            __syncthreads();
            const int nsw = p2p_window(a, b, w0, nw, wstart, wfirst, &wself, sh);
            for (int c0 = 0; c0 < nsw; c0 += kDChunk) {
                const int nc = min(kDChunk, nsw - c0);
                __syncthreads();
                // record j: x, y, z and the source tensors of the orders present
                for (int j = tid; j < nc; j += kDT) {
                    const int q = p2p_entry(wstart, nw, c0 + j);
                    const size_t pj = (size_t)wfirst[q] + (c0 + j - wstart[q]);
                    double *o = area + (3 + W) * j;
                    o[0] = a.xs[pj];
                    o[1] = a.xs[n + pj];
                    o[2] = a.xs[2 * n + pj];
                    int at = 0;
                    for (int s = 0; s < 4; ++s) {
                        if (ONE >= 0 ? s != ONE : !(d.smask & (1 << s))) continue;
                        double S[10];
                        source_of(s, a.m64 + pj * d.w + at, S);
                        const int nm = (s + 1) * (s + 2) / 2;
#pragma unroll
                        for (int c = 0; c < 10; ++c)
                            if (c < nm) o[3 + at + c] = S[c];
                        at += nm;
                    }
                }
                __syncthreads();
                if (act) {
                    const int jself = wself >= 0 ? wself + tg0 + t - c0 : -1;
                    for (int j = sl; j < nc; j += ns) {
                        if (j == jself) continue;
                        const double *o = area + (3 + W) * j;
                        const double rx = x - o[0], ry = y - o[1], rz = z - o[2];
                        const double ir = rsq_f64(rx * rx + ry * ry + rz * rz);
                        const double *m = o + 3;
                        auto T = [&](int c) { return m[c]; };
                        if constexpr (ONE >= 0) {
                            pair_derivs_const<K, ONE>(rx, ry, rz, ir, T, acc);
                        } else {
                            if (d.smask & 1) {
                                pair_derivs_const<K, 0>(rx, ry, rz, ir, T, acc);
                                m += 1;
                            }
                            if (d.smask & 2) {
                                pair_derivs_const<K, 1>(rx, ry, rz, ir, T, acc);
                                m += 3;
                            }
                            if (d.smask & 4) {
                                pair_derivs_const<K, 2>(rx, ry, rz, ir, T, acc);
                                m += 6;
                            }
                            if (d.smask & 8) pair_derivs_const<K, 3>(rx, ry, rz, ir, T, acc);
                        }
                    }
                }
            }
        }
        // the slices' sums, in slice order
        __syncthreads();
#pragma unroll
        for (int c = 0; c < NK; ++c) area[c * kDT + tid] = act ? acc[c] : 0.0;
        __syncthreads();
        if (tid < cs) {
            double v[NK];
#pragma unroll
            for (int c = 0; c < NK; ++c) v[c] = 0.0;
            for (int k = 0; k < ns; ++k)
#pragma unroll
                for (int c = 0; c < NK; ++c) v[c] += area[c * kDT + tid + k * cs];
            double *o = d.out + (size_t)NK * d.perm[i];
#pragma unroll
            for (int c = 0; c < NK; ++c) o[c] = v[c];
        }
    }
}

template <int K>
void derivs_launch(const DerivArgs &a, unsigned nleaves, hipStream_t s)
{
    const dim3 g(nleaves), bl(kDT);
    switch (a.smask) {
    case 1: hipLaunchKernelGGL((derivs_kernel<K, 0>), g, bl, 0, s, a); break;
    case 2: hipLaunchKernelGGL((derivs_kernel<K, 1>), g, bl, 0, s, a); break;
    case 4: hipLaunchKernelGGL((derivs_kernel<K, 2>), g, bl, 0, s, a); break;
    case 8: hipLaunchKernelGGL((derivs_kernel<K, 3>), g, bl, 0, s, a); break;
    default: hipLaunchKernelGGL((derivs_kernel<K, -1>), g, bl, 0, s, a); break;
    }
}

constexpr int kBW = 4;                                  // wavefronts (particles) per workgroup
constexpr int kDMax = nterms(kQMax);                    // derivative tensor to order p + K
constexpr int kBStack = 8 * (kMaxLevel + 3);

struct BHDerivArgs {
    const DevCell *cells;
    const double *xs;      // sorted positions, SoA
    const double *mom;     // sorted moments, w per particle
    const double *M;       // normalised multipoles, rows of nmp from order s (folded: harmonic order)
    const int32_t *perm;
    double *out;           // nk per particle, caller order
    int n, p, s, nmp, w, smask, folded;
    double theta2, h, lo[3];
};

__device__ __forceinline__ void wave_sync_d()
{
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}


template <int K>
__global__ __launch_bounds__(64 * kBW) void bh_derivs_kernel(BHDerivArgs a)
{
    constexpr int NK = (K + 1) * (K + 2) / 2;
    __shared__ double sD[kBW][kDMax];
    __shared__ double sPow[kBW][4][kQMax + 1];   // u_x^e, u_y^e, u_z^e and f^(e) at |u|
    __shared__ int stk[kBW][kBStack];
    const int wv = threadIdx.x / 64, lane = threadIdx.x % 64;
    const int i = blockIdx.x * kBW + wv;
    if (i >= a.n) return;   // the whole wavefront: it synchronises only with itself
    const size_t n = a.n;
    const double xi = a.xs[i], yi = a.xs[n + i], zi = a.xs[2 * n + i];
    int kidx[NK][3];
#pragma unroll
    for (int c = 0; c < NK; ++c) mi_of(K, c, kidx[c][0], kidx[c][1], kidx[c][2]);
    double acc[NK];
#pragma unroll
    for (int c = 0; c < NK; ++c) acc[c] = 0.0;
    const int Q = a.p + K;
    const int d0 = nterms(a.s + K - 1), d1 = nterms(Q);   // the derivative orders a contraction reads
    const int n0 = nterms(a.s - 1), n1 = nterms(a.p);
    double *D = sD[wv];
    if (lane == 0) stk[wv][0] = 0;
    int sp = 1;
    wave_sync_d();
    while (sp > 0) {
        --sp;
        const int c = stk[wv][sp];
        wave_sync_d();
        const DevCell cell = a.cells[c];
        // the acceptance test of Eq. 12 in the rounding sequence of the
        // Barnes-Hut evaluation kernel, so both accept the same cells
        const double rc = ldexp(1.0, kMaxLevel - cell.level);
        const double zx = __dadd_rn(a.lo[0], __dmul_rn((double)(2 * cell.ix + 1) * rc, a.h));
        const double zy = __dadd_rn(a.lo[1], __dmul_rn((double)(2 * cell.iy + 1) * rc, a.h));
        const double zz = __dadd_rn(a.lo[2], __dmul_rn((double)(2 * cell.iz + 1) * rc, a.h));
        const double r = __dmul_rn(rc, a.h);
        const double dx = __dsub_rn(xi, zx), dy = __dsub_rn(yi, zy), dz = __dsub_rn(zi, zz);
        const double d2 = __dadd_rn(__dadd_rn(__dmul_rn(dx, dx), __dmul_rn(dy, dy)), __dmul_rn(dz, dz));
        const bool inside = i >= cell.first && i < cell.first + cell.count;
        if (!inside && (__dmul_rn(r, r) < __dmul_rn(a.theta2, d2))) {
            const double ir = 1.0 / r;
            const double ux = dx * ir, uy = dy * ir, uz = dz * ir;
            if (lane <= Q) {
                const double iu2 = 1.0 / (ux * ux + uy * uy + uz * uz);
                double px = 1.0, py = 1.0, pz = 1.0, F = sqrt(iu2);
                for (int e = 1; e <= lane; ++e) {
                    px *= ux;
                    py *= uy;
                    pz *= uz;
                    F *= -(2.0 * e - 1.0) * iu2;
                }
                sPow[wv][0][lane] = px;
                sPow[wv][1][lane] = py;
                sPow[wv][2][lane] = pz;
                sPow[wv][3][lane] = F;
            }
            wave_sync_d();
            const double *PX = sPow[wv][0], *PY = sPow[wv][1], *PZ = sPow[wv][2], *FF = sPow[wv][3];
            for (int idx = d0 + lane; idx < d1; idx += 64) {
                int kx, ky, kz;
                mi_at(idx, kx, ky, kz);
                const int kk = kx + ky + kz;
                double v = 0.0;
                for (int ax = 0; 2 * ax <= kx; ++ax) {
                    const double cx = kHc[kx][ax] * PX[kx - 2 * ax];
                    for (int ay = 0; 2 * ay <= ky; ++ay) {
                        const double cxy = cx * kHc[ky][ay] * PY[ky - 2 * ay];
                        for (int az = 0; 2 * az <= kz; ++az)
                            v = fma(cxy * kHc[kz][az] * PZ[kz - 2 * az], FF[kk - ax - ay - az], v);
                    }
                }
                D[idx] = v;
            }
            wave_sync_d();
            double tq[NK];
#pragma unroll
            for (int q = 0; q < NK; ++q) tq[q] = 0.0;
            // a folded row holds the m_z <= 1 components: D_{.+k} is
            // harmonic, so contracting them gives the same sums
            const int j0 = a.folded ? hterms(a.s - 1) : n0, j1 = a.folded ? hterms(a.p) : n1;
            const double *Mc = a.M + (size_t)c * a.nmp - j0;
            for (int j = j0 + lane; j < j1; j += 64) {
                int mx, my, mz;
                if (a.folded) hmulti(j, mx, my, mz);
                else mi_at(j, mx, my, mz);
                const double mv = Mc[j];
#pragma unroll
                for (int q = 0; q < NK; ++q)
                    tq[q] = fma(mv, D[mindex(mx + kidx[q][0], my + kidx[q][1], mz + kidx[q][2])], tq[q]);
            }
            double sc = ir;
#pragma unroll
            for (int e = 0; e < K; ++e) sc *= ir;
#pragma unroll
            for (int q = 0; q < NK; ++q) acc[q] = fma(tq[q], sc, acc[q]);
            wave_sync_d();   // D and sPow are rewritten by the next accepted cell
        } else if (cell.nchild == 0) {
            for (int j = cell.first + lane; j < cell.first + cell.count; j += 64) {
                if (j == i) continue;
                pair_derivs_add<K>(xi - a.xs[j], yi - a.xs[n + j], zi - a.xs[2 * n + j], a.mom + (size_t)a.w * j,
                                   a.smask, kidx, acc);
            }
        } else {
            // children in reverse, so that they are visited in octant order
            if (lane == 0)
                for (int k = cell.nchild - 1; k >= 0; --k) stk[wv][sp + (cell.nchild - 1 - k)] = cell.child0 + k;
            sp += cell.nchild;
            wave_sync_d();
        }
    }
#pragma unroll
    for (int q = 0; q < NK; ++q)
        for (int o = 32; o > 0; o >>= 1) acc[q] += __shfl_down(acc[q], o, 64);
    if (lane == 0) {
        double *o = a.out + (size_t)NK * a.perm[i];
#pragma unroll
        for (int q = 0; q < NK; ++q) o[q] = acc[q];
    }
}

}  // namespace

hipError_t launch_derivs(fmm_tree *t, int K, double *out, hipStream_t s)
{
    if (t->nleaves == 0) return hipSuccess;
    DerivArgs a;
    a.near = P2PArgs{};
    a.near.leaves = t->d_leaves;
    a.near.ptr = t->d_p2p_ptr;
    a.near.src = t->d_p2p_src;
    a.near.order = t->d_p2p_order;
    a.near.cells = t->d_cells;
    a.near.xs = t->d_x;
    a.near.m64 = t->d_mom;
    a.near.n = (int)t->ht.n;
    a.near.h = t->ht.h;
    for (int d = 0; d < 3; ++d) a.near.lo[d] = t->ht.lo[d];
    a.perm = t->d_perm;
    a.L = t->d_L64;
    a.out = out;
    a.q = t->p - t->order;
    a.nl = nterms(a.q);
    a.nlh = t->basis == FMM_M2L_HARMONIC ? hterms(a.q) : 0;
    a.w = mask_width(t->smask);
    a.smask = t->smask;
    switch (K) {
    case 1: derivs_launch<1>(a, (unsigned)t->nleaves, s); break;
    case 2: derivs_launch<2>(a, (unsigned)t->nleaves, s); break;
    case 3: derivs_launch<3>(a, (unsigned)t->nleaves, s); break;
    default: return hipErrorInvalidValue;
    }
    return hipGetLastError();
}

hipError_t launch_bh_derivs(fmm_tree *t, int K, double *out, hipStream_t s)
{
    if (t->ht.n == 0) return hipSuccess;
    BHDerivArgs a;
    a.cells = t->d_cells;
    a.xs = t->d_x;
    a.mom = t->d_mom;
    a.folded = t->basis == FMM_M2L_HARMONIC;
    // the FP64 upward state: full rows, or folded ones in the harmonic basis
    a.M = a.folded ? (t->prec == FMM_PREC_MIXED ? t->d_Mf64 : (const double *)t->d_Mh) : t->d_M64;
    a.perm = t->d_perm;
    a.out = out;
    a.n = (int)t->ht.n;
    a.p = t->p;
    a.s = t->order;
    a.nmp = a.folded ? t->nhp : (nterms(t->p) - nterms(t->order - 1) + 3) / 4 * 4;
    a.w = mask_width(t->smask);
    a.smask = t->smask;
    a.theta2 = t->theta * t->theta;
    a.h = t->ht.h;
    for (int d = 0; d < 3; ++d) a.lo[d] = t->ht.lo[d];
    const dim3 g((unsigned)((t->ht.n + kBW - 1) / kBW)), bl(64 * kBW);
    switch (K) {
    case 1: hipLaunchKernelGGL(bh_derivs_kernel<1>, g, bl, 0, s, a); break;
    case 2: hipLaunchKernelGGL(bh_derivs_kernel<2>, g, bl, 0, s, a); break;
    case 3: hipLaunchKernelGGL(bh_derivs_kernel<3>, g, bl, 0, s, a); break;
    default: return hipErrorInvalidValue;
    }
    return hipGetLastError();
}
