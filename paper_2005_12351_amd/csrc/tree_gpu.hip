// Octree construction and dual-tree interaction lists on the GPU (Pepper &
// Fangohr, arXiv 2005.12351, Section 3.2): root box, 21-bit quantisation,
// Morton keys, stable sort, adaptive octree (split while a cell holds more
// than ncrit particles, depth cap 21), and the dual traversal with the FMM
// acceptance criterion (Eq. 13), which yields the M2L and P2P lists.
//
// Canonical definitions (the same as the test oracle's, shared by
// specification only): root cube of side W = largest extent at the
// componentwise minimum; q = floor((x - lo) * 2^21 / W) clamped to 2^21 - 1;
// key = bit interleave with x most significant in every octal digit; stable
// sort by key; cells level-major in ascending key order, children in octant
// order, empty children not created; geometry in units of h = W 2^-22 with
// centre (2i+1) 2^(21-l) and radius (half side) 2^(21-l); acceptance
// (rA + rB)^2 < theta^2 d^2 evaluated in FP64 on exact integers; when a pair
// is neither accepted nor a leaf pair the larger cell is split (both on a
// tie; a leaf is never split).  Each target's lists are sorted by source.
//
// Layout of the work.  A build is bound by its launches and read-backs, not by
// bytes, so it takes few of both: the sorted keys alone give every cell of
// every level at once (cell_depth / cells_emit), each target cell finds its
// lists from its parent's open pairs in one workgroup (lists_count, a launch
// per level; lists_emit, one for all cells), and the M2L schedule follows in
// four kernels (launch_tiling).  The host waits for the number of cells, the
// list lengths and the schedule's sizes, and uses the first wait's cells
// while the lists are made.  Every pass is deterministic: counts come from
// ballots and scans, and where atomics hand out space the result does not
// depend on their order.  Build, upward pass and evaluation, against a launch
// and a scan per level and traversal step and sorts of the lists (about 130
// launches and ten waits): 100k dipoles, theta 0.5, p 8: 1465 -> 845 us; 3001
// Plummer quadrupoles, p 4: 1065 -> 707 us.
#include <algorithm>
#include <chrono>
#include <climits>
#include <cmath>
#include <vector>

#include "fmm_internal.h"

namespace {

constexpr int kScanT = 256;           // threads per scan block
constexpr int kScanI = 4;             // items per thread
constexpr int kScanTile = kScanT * kScanI;

// ---------------------------------------------------------------- scans
__device__ __forceinline__ int wave_incl_scan(int v)
{
    const int lane = threadIdx.x & 63;
#pragma unroll
    for (int o = 1; o < 64; o <<= 1) {
        const int u = __shfl_up(v, o, 64);
        if (lane >= o) v += u;
    }
    return v;
}

// exclusive prefix over the threads of a block of NT threads; returns the
// block total through *tot
template <int NT>
__device__ int block_excl_scan(int v, int *sh, int *tot)
{
    const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
    const int inc = wave_incl_scan(v);
    if (lane == 63) sh[w] = inc;
    __syncthreads();
    int base = 0, all = 0;
    for (int k = 0; k < NT / 64; ++k) {
        if (k < w) base += sh[k];
        all += sh[k];
    }
    __syncthreads();
    *tot = all;
    return base + inc - v;
}

// one block of 1024 threads: exclusive scan of up to kSmallScan values,
// 64-bit total to *total
constexpr int kSmallT = 1024;
constexpr int kSmallScan = 1 << 16;
__device__ __forceinline__ void scan_small_body(const int32_t *__restrict__ in, int32_t *__restrict__ out, int n,
                                                int64_t *__restrict__ total);
__global__ __launch_bounds__(kSmallT) void scan_small_kernel(const int32_t *__restrict__ in, int32_t *__restrict__ out,
                                                             int n, int64_t *__restrict__ total)
{
    scan_small_body(in, out, n, total);
}

// two independent small scans of n values in one launch, one block each; the
// total also follows the scanned values (out[n])
struct Scan2 {
    const int32_t *in[2];
    int32_t *out[2];
    int64_t *total[2];
};
__global__ __launch_bounds__(kSmallT) void scan_small2_kernel(Scan2 a, int n)
{
    const int k = blockIdx.x;
    scan_small_body(a.in[k], a.out[k], n, a.total[k]);
    if (threadIdx.x == 0) a.out[k][n] = (int32_t)*a.total[k];
}

__device__ __forceinline__ void scan_small_body(const int32_t *__restrict__ in, int32_t *__restrict__ out, int n,
                                                int64_t *__restrict__ total)
{
    __shared__ int sh[kSmallT / 64];
    __shared__ long long t64[kSmallT / 64];
    const int per = (n + kSmallT - 1) / kSmallT;
    const int b0 = threadIdx.x * per, b1 = min(n, b0 + per);
    int s = 0;
    for (int b = b0; b < b1; ++b) s += in[b];
    int tot;
    int run = block_excl_scan<kSmallT>(s, sh, &tot);
    for (int b = b0; b < b1; ++b) {
        const int v = in[b];
        out[b] = run;
        run += v;
    }
    // 64-bit total: per-wave sums of the per-thread sums
    long long w64 = s;
    for (int o = 32; o > 0; o >>= 1) w64 += __shfl_down(w64, o, 64);
    if ((threadIdx.x & 63) == 0) t64[threadIdx.x >> 6] = w64;
    __syncthreads();
    if (threadIdx.x == 0) {
        long long a = 0;
        for (int k = 0; k < kSmallT / 64; ++k) a += t64[k];
        *total = a;
    }
}

// per block: exclusive scan of its tile, block total to sums[b]
__global__ __launch_bounds__(kScanT) void scan_tile_kernel(const int32_t *__restrict__ in, int32_t *__restrict__ out,
                                                           int n, int32_t *__restrict__ sums)
{
    __shared__ int sh[kScanT / 64];
    const int64_t base = (int64_t)blockIdx.x * kScanTile + (int64_t)threadIdx.x * kScanI;
    int v[kScanI], s = 0;
#pragma unroll
    for (int j = 0; j < kScanI; ++j) {
        v[j] = base + j < n ? in[base + j] : 0;
        s += v[j];
    }
    int tot;
    int run = block_excl_scan<kScanT>(s, sh, &tot);
#pragma unroll
    for (int j = 0; j < kScanI; ++j) {
        if (base + j < n) out[base + j] = run;
        run += v[j];
    }
    if (threadIdx.x == 0) sums[blockIdx.x] = tot;
}

// one block: exclusive scan of the block sums in place; grand total (64-bit)
// to *total
__global__ __launch_bounds__(kScanT) void scan_sums_kernel(int32_t *__restrict__ sums, int nb, int64_t *__restrict__ total)
{
    __shared__ int sh[kScanT / 64];
    const int per = (nb + kScanT - 1) / kScanT;
    const int b0 = threadIdx.x * per, b1 = min(nb, b0 + per);
    int s = 0;
    long long s64 = 0;
    for (int b = b0; b < b1; ++b) {
        s += sums[b];
        s64 += sums[b];
    }
    int tot;
    int run = block_excl_scan<kScanT>(s, sh, &tot);
    for (int b = b0; b < b1; ++b) {
        const int v = sums[b];
        sums[b] = run;
        run += v;
    }
    // 64-bit total, in case the 32-bit prefix overflowed (checked by the host)
    __shared__ long long t64[kScanT];
    t64[threadIdx.x] = s64;
    __syncthreads();
    if (threadIdx.x == 0) {
        long long a = 0;
        for (int k = 0; k < kScanT; ++k) a += t64[k];
        *total = a;
    }
}

__global__ __launch_bounds__(kScanT) void scan_add_kernel(int32_t *__restrict__ out, int n, const int32_t *__restrict__ sums)
{
    const int64_t base = (int64_t)blockIdx.x * kScanTile + (int64_t)threadIdx.x * kScanI;
    const int add = sums[blockIdx.x];
#pragma unroll
    for (int j = 0; j < kScanI; ++j)
        if (base + j < n) out[base + j] += add;
}

// ---------------------------------------------------------------- small sort
// one workgroup, in place: the order of the stable sort on (key & mask) for
// n <= kSmallSort items, as a bitonic sort of (masked key, position) in LDS;
// keys and values are then gathered by position
constexpr int kSmallSort = 2048;
constexpr int kSmallSortT = 1024;
__global__ __launch_bounds__(kSmallSortT) void small_sort_kernel(uint64_t *__restrict__ k, int32_t *__restrict__ v, int n,
                                                                 uint64_t mask)
{
    __shared__ uint64_t sk[kSmallSort];
    __shared__ uint16_t sp[kSmallSort];
    int np = 1;
    while (np < n) np <<= 1;
    for (int i = threadIdx.x; i < np; i += kSmallSortT) {
        sk[i] = i < n ? (k[i] & mask) : mask;   // padding sorts last: its position is >= n
        sp[i] = (uint16_t)i;
    }
    __syncthreads();
    for (int size = 2; size <= np; size <<= 1)
        for (int j = size >> 1; j > 0; j >>= 1) {
            for (int i = threadIdx.x; i < np; i += kSmallSortT) {
                const int l = i ^ j;
                if (l > i) {
                    const uint64_t a = sk[i], b = sk[l];
                    const uint16_t pa = sp[i], pb = sp[l];
                    const bool gt = a > b || (a == b && pa > pb);
                    if (gt == ((i & size) == 0)) {
                        sk[i] = b;
                        sk[l] = a;
                        sp[i] = pb;
                        sp[l] = pa;
                    }
                }
            }
            __syncthreads();
        }
    constexpr int kPer = kSmallSort / kSmallSortT;
    uint64_t kk[kPer];
    int32_t vv[kPer];
#pragma unroll
    for (int q = 0; q < kPer; ++q) {
        const int i = threadIdx.x + q * kSmallSortT;
        if (i < n) {
            kk[q] = k[sp[i]];
            vv[q] = v[sp[i]];
        }
    }
    __syncthreads();
#pragma unroll
    for (int q = 0; q < kPer; ++q) {
        const int i = threadIdx.x + q * kSmallSortT;
        if (i < n) {
            k[i] = kk[q];
            v[i] = vv[q];
        }
    }
}

// ---------------------------------------------------------------- keys
// Words the host reads back (whole 8-byte words).
struct BuildState {
    double box[8];                       // minima, maxima, non-finite flag, key scale
    int32_t totals[kMaxLevel + 3];       // cells of every level
    int64_t nm2l, np2p;                  // list lengths
    unsigned long long down;             // open-pair entries asked for
    unsigned long long info[6];          // schedule: targets, flags, entries, classes, shallowest target, source
    unsigned long long longs;            // lists left unsorted: number << 40 | entries
    int32_t cursor, pad;                 // schedule: geometries of all tiles so far
};

// per block: componentwise min and max, and 1 if any coordinate is not finite
__global__ void bbox_partial_kernel(const double *__restrict__ pos, int64_t n, double *__restrict__ part)
{
    __shared__ double sh[7][256];
    double lo[3] = {INFINITY, INFINITY, INFINITY}, hi[3] = {-INFINITY, -INFINITY, -INFINITY};
    double bad = 0.0;
    for (int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; i < n; i += (int64_t)gridDim.x * blockDim.x)
        for (int d = 0; d < 3; ++d) {
            const double x = pos[3 * i + d];
            if (!isfinite(x)) bad = 1.0;
            lo[d] = fmin(lo[d], x);
            hi[d] = fmax(hi[d], x);
        }
    for (int d = 0; d < 3; ++d) {
        sh[d][threadIdx.x] = lo[d];
        sh[3 + d][threadIdx.x] = hi[d];
    }
    sh[6][threadIdx.x] = bad;
    __syncthreads();
    for (int s = blockDim.x / 2; s > 0; s >>= 1) {
        if ((int)threadIdx.x < s) {
            for (int d = 0; d < 3; ++d) {
                sh[d][threadIdx.x] = fmin(sh[d][threadIdx.x], sh[d][threadIdx.x + s]);
                sh[3 + d][threadIdx.x] = fmax(sh[3 + d][threadIdx.x], sh[3 + d][threadIdx.x + s]);
            }
            sh[6][threadIdx.x] = fmax(sh[6][threadIdx.x], sh[6][threadIdx.x + s]);
        }
        __syncthreads();
    }
    if (threadIdx.x < 7) part[7 * blockIdx.x + threadIdx.x] = sh[threadIdx.x][0];
}

// one block of 256: the 7 components (3 minima, 3 maxima, the non-finite
// flag) over the nb partial results, strided over the threads, then an LDS
// tree; min and max are exact, so the order does not matter.  The rest of the
// state starts here too.
__global__ __launch_bounds__(256) void bbox_final_kernel(const double *__restrict__ part, int nb, BuildState *bs)
{
    __shared__ double sh[7][256];
    double *out = bs->box;
    if (threadIdx.x < kMaxLevel + 3) bs->totals[threadIdx.x] = 0;
    if (threadIdx.x < 6) bs->info[threadIdx.x] = threadIdx.x < 4 ? 0ull : ~0ull;
    if (threadIdx.x == 0) {
        bs->nm2l = bs->np2p = 0;
        bs->down = 0;
        bs->longs = 0;
        bs->cursor = 0;
    }
    double v[7];
    for (int k = 0; k < 7; ++k) v[k] = k < 3 ? INFINITY : -INFINITY;
    for (int b = threadIdx.x; b < nb; b += 256)
        for (int k = 0; k < 7; ++k) v[k] = k < 3 ? fmin(v[k], part[7 * b + k]) : fmax(v[k], part[7 * b + k]);
    for (int k = 0; k < 7; ++k) sh[k][threadIdx.x] = v[k];
    __syncthreads();
    for (int w = 128; w > 0; w >>= 1) {
        if (threadIdx.x < w)
            for (int k = 0; k < 7; ++k)
                sh[k][threadIdx.x] = k < 3 ? fmin(sh[k][threadIdx.x], sh[k][threadIdx.x + w])
                                           : fmax(sh[k][threadIdx.x], sh[k][threadIdx.x + w]);
        __syncthreads();
    }
    if (threadIdx.x < 7) out[threadIdx.x] = sh[threadIdx.x][0];
    if (threadIdx.x == 0) {   // out[7]: the key scale 2^21 / W, W the largest extent (1 if all coincide)
        const double e0 = sh[3][0] - sh[0][0], e1 = sh[4][0] - sh[1][0], e2 = sh[5][0] - sh[2][0];
        const double m12 = e1 < e2 ? e2 : e1;
        double W = e0 < m12 ? m12 : e0;
        if (W == 0.0) W = 1.0;
        out[7] = ldexp(1.0, kMaxLevel) / W;
    }
}

__device__ __forceinline__ uint64_t spread3(uint64_t v)
{
    v &= 0x1fffffULL;
    v = (v | (v << 32)) & 0x1f00000000ffffULL;
    v = (v | (v << 16)) & 0x1f0000ff0000ffULL;
    v = (v | (v << 8)) & 0x100f00f00f00f00fULL;
    v = (v | (v << 4)) & 0x10c30c30c30c30c3ULL;
    v = (v | (v << 2)) & 0x1249249249249249ULL;
    return v;
}

// box: the componentwise minima, maxima, the non-finite flag and the key
// scale (bbox_final_kernel); with a non-finite position every key is 0 (the
// host rejects the build at its first read-back)
__global__ void keys_kernel(const double *__restrict__ pos, int n, const double *__restrict__ box,
                            uint64_t *__restrict__ key, int32_t *__restrict__ idx)
{
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= n) return;
    idx[i] = i;
    if (box[6] != 0.0) {
        key[i] = 0;
        return;
    }
    const double scale = box[7];
    const int64_t qmax = (int64_t(1) << kMaxLevel) - 1;
    uint64_t q[3];
    for (int d = 0; d < 3; ++d) {
        const double v = __dmul_rn(__dsub_rn(pos[3 * (size_t)i + d], box[d]), scale);
        const int64_t qi = (int64_t)floor(v);
        q[d] = (uint64_t)min(max(qi, (int64_t)0), qmax);
    }
    key[i] = (spread3(q[0]) << 2) | (spread3(q[1]) << 1) | spread3(q[2]);
}

// ---------------------------------------------------------------- tree
// octal digits two 63-bit keys have in common, from the top
__device__ __forceinline__ int common_digits(uint64_t a, uint64_t b)
{
    return a == b ? kMaxLevel : (__clzll((long long)(a ^ b)) - 1) / 3;
}

// Every cell of the tree from the sorted keys.  With d_i the digits particle i
// shares with its predecessor, a cell of level l starts at i iff d_i < l; it
// exists iff its parent splits, and a cell of level l around i holds more
// than ncrit particles iff some window of ncrit + 1 consecutive particles
// around i agrees in l digits.  So with D_i the largest m_j = digits that
// particles j and j + ncrit share, over j in [i - ncrit, i] (at most 20: cells
// of level 21 do not split), the cells that start at i are those of the
// levels d_i + 1 .. D_i + 1 (level 0 at i = 0).
// One workgroup takes kCellT particles; the window maximum by doubling in LDS
// for ncrit <= kWinMax, else from wide (window_max_kernel).  Writes the level
// range of every particle and the workgroup's cells per level.
constexpr int kCellT = 256;              // particles per workgroup, one a thread
constexpr int kWinMax = 3840;
constexpr int kLevels = kMaxLevel + 1;
__device__ __forceinline__ int8_t window_digits(const uint64_t *key, int64_t j, int64_t n, int ncrit)
{
    if (j < 0 || j + ncrit >= n) return -1;
    return (int8_t)min(kMaxLevel - 1, common_digits(key[j], key[j + ncrit]));
}

__global__ __launch_bounds__(256) void cell_depth_kernel(const uint64_t *__restrict__ key, int n, int ncrit,
                                                         const int8_t *__restrict__ wide, uchar2 *__restrict__ range,
                                                         int32_t *__restrict__ cnt)
{
    __shared__ int8_t buf[2][kCellT + kWinMax];
    __shared__ int hist[kLevels + 2];
    const int base = blockIdx.x * kCellT;
    if (threadIdx.x < kLevels + 2) hist[threadIdx.x] = 0;
    int8_t *w = buf[0], *w2 = buf[1];
    int half = 1;                        // w[x]: maximum over the last `half` windows up to x
    const int W = ncrit + 1;
    if (!wide) {
        const int m = kCellT + ncrit;
        for (int x = threadIdx.x; x < m; x += 256) w[x] = window_digits(key, (int64_t)base - ncrit + x, n, ncrit);
        __syncthreads();
        while (2 * half <= W) {
            for (int x = threadIdx.x; x < m; x += 256) w2[x] = x >= half ? max(w[x], w[x - half]) : w[x];
            __syncthreads();
            int8_t *t = w;
            w = w2;
            w2 = t;
            half *= 2;
        }
    } else {
        __syncthreads();
    }
    const int i = base + threadIdx.x;
    if (i < n) {
        int D;
        if (wide) {
            D = wide[i];
        } else {
            const int x = i - base + ncrit;
            D = max(w[x], w[x - (W - half)]);
        }
        const int lo = i == 0 ? 0 : common_digits(key[i - 1], key[i]) + 1, hi = D + 1;
        range[i] = make_uchar2((uint8_t)lo, (uint8_t)hi);
        if (lo <= hi) {
            atomicAdd(&hist[lo], 1);
            atomicAdd(&hist[hi + 1], -1);
        }
    }
    __syncthreads();
    if (threadIdx.x < kLevels) {
        int c = 0;
        for (int l = 0; l <= (int)threadIdx.x; ++l) c += hist[l];
        cnt[(size_t)threadIdx.x * gridDim.x + blockIdx.x] = c;
    }
}

// the window maximum for ncrit > kWinMax: out[i] = max(in[i], in[i - back]);
// first: in is the digits themselves
__global__ void window_max_kernel(const uint64_t *__restrict__ key, int n, int ncrit, int first, int back,
                                  const int8_t *__restrict__ in, int8_t *__restrict__ out)
{
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= n) return;
    if (first) out[i] = window_digits(key, i, n, ncrit);
    else out[i] = i >= back ? max(in[i], in[i - back]) : in[i];
}

// one block per level: its workgroups' cell counts to exclusive offsets
__global__ __launch_bounds__(kSmallT) void level_offsets_kernel(int32_t *__restrict__ cnt, int nblk, BuildState *bs)
{
    __shared__ int64_t tot;
    int32_t *row = cnt + (size_t)blockIdx.x * nblk;
    scan_small_body(row, row, nblk, &tot);
    if (threadIdx.x == 0) bs->totals[blockIdx.x] = (int32_t)tot;
}

struct LevelPtr {
    int32_t v[kLevels + 1];
};

__device__ __forceinline__ int compact_axis(uint64_t key, int axis, int level)
{
    // the axis's bit of each of the key's first `level` octal digits
    uint64_t v = (key >> (3 * (kMaxLevel - level))) >> (2 - axis);
    v &= 0x1249249249249249ULL;
    v = (v | (v >> 2)) & 0x10c30c30c30c30c3ULL;
    v = (v | (v >> 4)) & 0x100f00f00f00f00fULL;
    v = (v | (v >> 8)) & 0x1f0000ff0000ffULL;
    v = (v | (v >> 16)) & 0x1f00000000ffffULL;
    return (int)((v | (v >> 32)) & 0x1fffffULL);
}

// The cells of kCellT particles, level-major.  A particle writes the cells that
// start at it, and where those of its predecessor end and their children end
// (pad0, pad1; cells_finish_kernel turns them into counts).
__global__ __launch_bounds__(kCellT) void cells_emit_kernel(const uint64_t *__restrict__ key, int n,
                                                            const uchar2 *__restrict__ range,
                                                            const int32_t *__restrict__ cnt, LevelPtr lp, int nlev,
                                                            DevCell *__restrict__ cells)
{
    constexpr int kWaves = kCellT / 64;
    __shared__ int off[kWaves][kLevels + 1];   // cells of the level before the wave's first particle
    const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
    const int i = blockIdx.x * kCellT + threadIdx.x;
    int lo = 1, hi = 0, hp = -1;               // levels that start here; deepest level of the predecessor
    uint64_t k = 0;
    if (i < n) {
        const uchar2 v = range[i];
        lo = v.x;
        hi = v.y;
        if (i > 0) hp = range[i - 1].y;
        k = key[i];
    }
    for (int l = 0; l < nlev; ++l) {
        const unsigned long long m = __ballot(lo <= l && l <= hi);
        if (lane == 0) off[wv][l] = __popcll(m);
    }
    __syncthreads();
    if ((int)threadIdx.x < nlev) {
        int run = cnt[(size_t)threadIdx.x * gridDim.x + blockIdx.x];
        for (int c = 0; c < kWaves; ++c) {
            const int v = off[c][threadIdx.x];
            off[c][threadIdx.x] = run;
            run += v;
        }
    }
    __syncthreads();
    const unsigned long long before = (1ull << lane) - 1;
    // from the deepest level up: the index of the level's first cell at or
    // after i, at this level, the one below and the one above
    auto at = [&](int l, int &starts) {
        const bool st = lo <= l && l <= hi;
        const unsigned long long m = __ballot(st);
        starts = st;
        return lp.v[l] + off[wv][l] + __popcll(m & before);
    };
    int below = 0, starts_below = 0, st = 0, idx = at(nlev - 1, st);
    for (int l = nlev - 1; l >= 0; --l) {
        int st_up = 0, up = 0;
        if (l > 0) up = at(l - 1, st_up);
        if (st) {
            DevCell *o = cells + idx;
            o->level = l;
            o->ix = compact_axis(k, 0, l);
            o->iy = compact_axis(k, 1, l);
            o->iz = compact_axis(k, 2, l);
            o->first = i;
            o->parent = l > 0 ? up + st_up - 1 : -1;
            o->child0 = l < hi ? below : -1;
            o->pad2 = 0;
        }
        if (i < n && l >= lo && l <= hp) {   // the predecessor's cell of level l ends here
            cells[idx - 1].pad0 = i;
            cells[idx - 1].pad1 = below;
        }
        if (i == n - 1 && l <= hi) {
            cells[idx + st - 1].pad0 = n;
            cells[idx + st - 1].pad1 = below + starts_below;
        }
        below = idx;
        starts_below = st;
        idx = up;
        st = st_up;
    }
}

// counts and children of the cells; and the schedule's tables cleared: the
// class table, the cells' tile slots
__global__ void cells_finish_kernel(DevCell *__restrict__ cells, int nc, int32_t *__restrict__ cell_slot,
                                    uint64_t *__restrict__ table, int ntable)
{
    const int c = blockIdx.x * blockDim.x + threadIdx.x;
    for (int k = c; k < ntable; k += gridDim.x * blockDim.x) table[k] = ~0ull;
    if (c >= nc) return;
    DevCell *o = cells + c;
    o->count = o->pad0 - o->first;
    o->nchild = o->child0 < 0 ? 0 : o->pad1 - o->child0;
    o->pad0 = o->pad1 = 0;
    if (cell_slot) cell_slot[c] = -1;
}

// ---------------------------------------------------------------- traversal
struct PairAct {
    int m2l, p2p, nkids, mode;   // mode: 0 none, 1 children of A, 2 of B, 3 both
};

__device__ __forceinline__ PairAct pair_action(const DevCell &a, const DevCell &b, double th2)
{
    const int64_t ra = int64_t(1) << (kMaxLevel - a.level), rb = int64_t(1) << (kMaxLevel - b.level);
    const int64_t dx = (2 * (int64_t)b.ix + 1) * rb - (2 * (int64_t)a.ix + 1) * ra;
    const int64_t dy = (2 * (int64_t)b.iy + 1) * rb - (2 * (int64_t)a.iy + 1) * ra;
    const int64_t dz = (2 * (int64_t)b.iz + 1) * rb - (2 * (int64_t)a.iz + 1) * ra;
    const int64_t d2 = dx * dx + dy * dy + dz * dz;
    const double s = (double)(ra + rb);
    const bool leafA = a.nchild == 0, leafB = b.nchild == 0;
    PairAct r{0, 0, 0, 0};
    if (__dmul_rn(s, s) < __dmul_rn(th2, (double)d2)) {
        r.m2l = 1;
    } else if (leafA && leafB) {
        r.p2p = 1;
    } else if (leafB || (!leafA && ra > rb)) {
        r.mode = 1;
        r.nkids = a.nchild;
    } else if (leafA || rb > ra) {
        r.mode = 2;
        r.nkids = b.nchild;
    } else {
        r.mode = 3;
        r.nkids = a.nchild * b.nchild;
    }
    return r;
}

// The dual traversal from the target's side.  The pairs (A, B) with B as the
// target are those that its parent left open by splitting the target (mode 2:
// A stays, mode 3: A's children), and the children of A wherever such a pair
// splits A alone (mode 1).  One workgroup walks a target's pairs: the open
// entries of the parent eight slots each (a slot per child of A), then, where
// pairs split A alone, their children from a stack in LDS until it is empty.
// on(action, A) is called by all threads at once, with an empty action for the
// idle ones; the order of the pairs is fixed.
constexpr int kListT = 256;
constexpr int kStackCap = 4096;
constexpr uint32_t kOpenKids = 1u << 31;   // an open entry whose source was split too (mode 3)
struct ListShared {
    int stack[kStackCap];
    int sh[kListT / 64];
};

template <typename F>
__device__ void walk_pairs(const DevCell *__restrict__ cells, int B, const DevCell &b, double th2,
                           const uint32_t *__restrict__ open, int nopen, ListShared &ls, F &&on)
{
    int size = 0;   // stack entries (the same for all threads)
    auto visit = [&](int A, bool live) {
        PairAct r{0, 0, 0, 0};
        DevCell a;
        if (live) {
            a = cells[A];
            r = pair_action(a, b, th2);
        }
        on(r, A);
        const int kids = r.mode == 1 ? r.nkids : 0;
        if (__syncthreads_or(kids)) {
            int tot;
            const int o = size + block_excl_scan<kListT>(kids, ls.sh, &tot);
            for (int k = 0; k < kids; ++k) ls.stack[o + k] = a.child0 + k;
            size += tot;
            __syncthreads();
        }
    };
    const int nslots = nopen * 8;
    for (int s0 = 0; s0 < nslots; s0 += kListT) {
        const int s = s0 + threadIdx.x;
        int A = 0;
        bool live = false;
        if (s < nslots) {
            const uint32_t e = open[s >> 3];
            const int src = (int)(e & ~kOpenKids), k = s & 7;
            if (e & kOpenKids) {
                live = k < cells[src].nchild;
                A = cells[src].child0 + k;
            } else {
                live = k == 0;
                A = src;
            }
        }
        visit(A, live);
        // Take as many pairs from the top as leave room for eight children
        // each and for a descent pair by pair below that (7 entries a level);
        // with no such room one pair, whose subtree then fits the reserve.
        while (size > 0) {
            const int take = min(size, min(kListT, max(1, (kStackCap - size - 7 * (kMaxLevel + 2)) / 7)));
            const bool has = (int)threadIdx.x < take;
            const int C = has ? ls.stack[size - take + threadIdx.x] : 0;
            size -= take;
            __syncthreads();
            visit(C, has);
        }
    }
}

// lengths of the lists of every target of one level, and its open pairs in
// order, in a segment of `open_buf` that an atomic hands out (segments are
// read through open_seg, so their order does not matter).  The open pairs are
// kept in LDS on the way; a target with more than it holds walks again.  A
// segment past the buffer's end is not written: the host sees bs->down exceed
// the capacity and runs the levels again with a larger buffer.
constexpr int kOpenBuf = 2048;
__global__ __launch_bounds__(kListT) void lists_count_kernel(const DevCell *__restrict__ cells, int lb, double th2,
                                                             uint2 *__restrict__ open_seg,
                                                             uint32_t *__restrict__ open_buf, unsigned open_cap,
                                                             BuildState *bs, int32_t *__restrict__ m2l_cnt,
                                                             int32_t *__restrict__ p2p_cnt)
{
    __shared__ ListShared ls;
    __shared__ uint32_t held[kOpenBuf];
    __shared__ unsigned s_off;
    __shared__ int s_tot[2], s_write;
    const int B = lb + blockIdx.x;
    const DevCell b = cells[B];
    __shared__ uint32_t root;
    const uint32_t *open = &root;
    int nopen = 1;
    if (threadIdx.x == 0) {
        root = 0;                               // (root, root)
        s_tot[0] = s_tot[1] = 0;
    }
    if (b.parent >= 0) {
        const uint2 sg = open_seg[b.parent];
        open = open_buf + sg.x;
        nopen = (int)sg.y;
    }
    __syncthreads();
    int nm = 0, np = 0, done = 0;
    const bool leaf = b.nchild == 0;            // a leaf leaves no pair open
    walk_pairs(cells, B, b, th2, open, nopen, ls, [&](const PairAct &r, int A) {
        nm += r.m2l;
        np += r.p2p;
        if (leaf) return;
        int t;
        const int o = done + block_excl_scan<kListT>(r.mode >= 2, ls.sh, &t);
        if (r.mode >= 2 && o < kOpenBuf) held[o] = (uint32_t)A | (r.mode == 3 ? kOpenKids : 0u);
        done += t;
    });
    if (nm) atomicAdd(&s_tot[0], nm);
    if (np) atomicAdd(&s_tot[1], np);
    __syncthreads();
    if (threadIdx.x == 0) {
        m2l_cnt[B] = s_tot[0];
        p2p_cnt[B] = s_tot[1];
        unsigned o = 0;
        int c = done;
        if (done) {
            const unsigned long long at = atomicAdd(&bs->down, (unsigned long long)done);
            if (at + (unsigned long long)done > open_cap) c = 0;
            else o = (unsigned)at;
        }
        open_seg[B] = make_uint2(o, (unsigned)c);
        s_off = o;
        s_write = c;
    }
    __syncthreads();
    if (s_write == 0) return;
    uint32_t *out = open_buf + s_off;
    if (done <= kOpenBuf) {
        for (int k = threadIdx.x; k < done; k += kListT) out[k] = held[k];
        return;
    }
    done = 0;
    walk_pairs(cells, B, b, th2, open, nopen, ls, [&](const PairAct &r, int A) {
        int t;
        const int o = done + block_excl_scan<kListT>(r.mode >= 2, ls.sh, &t);
        if (r.mode >= 2) out[o] = (uint32_t)A | (r.mode == 3 ? kOpenKids : 0u);
        done += t;
    });
}

// ascending sort of v[0..n) in LDS by the workgroup: a bitonic network whose
// comparators all point upwards, so that places past n count as larger than
// everything and are left out
__device__ void block_sort(int32_t *v, int n)
{
    int np = 1;
    while (np < n) np <<= 1;
    for (int k = 2; k <= np; k <<= 1)
        for (int j = k >> 1; j > 0; j >>= 1) {
            const int x = j == k >> 1 ? k - 1 : j;
            for (int i = threadIdx.x; i < n; i += kListT) {
                const int l = i ^ x;
                if (l > i && l < n) {
                    const int32_t p = v[i], q = v[l];
                    if (p > q) {
                        v[i] = q;
                        v[l] = p;
                    }
                }
            }
            __syncthreads();
        }
}

// The lists of every cell, one workgroup each, sorted by source (already so
// where the sources are all of one level: the order of the walk), in LDS.  A
// list past its capacity is written as it comes and, where that is not sorted,
// left to sort_long_lists: its length and place go to `longs`, its number and
// its first entry among all of them come from one atomic, so that the lists lie
// in that array in the order of their entries.  With them the cell's near-field
// cost (its particles times its P2P sources' particles) and its M2L target
// key: level (5 bits) | octant (3) | lo0 hi0 lo1 hi1 lo2 hi2 (the smallest and
// largest same-level source offset per axis, 7 bits each, + 64) | 8191 - length
// (13); cells without an M2L list sort last.
constexpr uint64_t kEmptyKey = ~0ull;
constexpr int kM2LBuf = 3072, kP2PBuf = 2048;
constexpr int kLongShift = 40;
struct LongList {
    int32_t start, n;       // place in its array, length
    uint32_t first;         // its first entry among all long lists
    int32_t p2p;            // of the P2P lists, not the M2L lists
};
__global__ __launch_bounds__(kListT) void lists_emit_kernel(const DevCell *__restrict__ cells, double th2,
                                                            const uint2 *__restrict__ open_seg,
                                                            const uint32_t *__restrict__ open_buf,
                                                            const int32_t *__restrict__ m2l_ptr,
                                                            const int32_t *__restrict__ p2p_ptr, BuildState *bs,
                                                            int32_t *__restrict__ m2l_src, int32_t *__restrict__ p2p_src,
                                                            int64_t *__restrict__ cost, uint64_t *__restrict__ key,
                                                            int32_t *__restrict__ val, LongList *__restrict__ longs)
{
    __shared__ ListShared ls;
    __shared__ int32_t mbuf[kM2LBuf], pbuf[kP2PBuf];
    __shared__ uint32_t root;
    __shared__ long long s_cost;
    __shared__ int s_lo[3], s_hi[3], s_first;
    const int B = blockIdx.x;
    const DevCell b = cells[B];
    const int m0 = m2l_ptr[B], mn = m2l_ptr[B + 1] - m0, p0 = p2p_ptr[B], pn = p2p_ptr[B + 1] - p0;
    int32_t *const mv = mn <= kM2LBuf ? mbuf : m2l_src + m0, *const pv = pn <= kP2PBuf ? pbuf : p2p_src + p0;
    const uint32_t *open = &root;
    int nopen = 1;
    if (threadIdx.x == 0) {
        root = 0;
        s_cost = 0;
        s_first = INT_MAX;
    }
    if (threadIdx.x < 3) {
        s_lo[threadIdx.x] = INT_MAX;
        s_hi[threadIdx.x] = INT_MIN;
    }
    if (b.parent >= 0) {
        const uint2 sg = open_seg[b.parent];
        open = open_buf + sg.x;
        nopen = (int)sg.y;
    }
    __syncthreads();
    if (mn + pn > 0) {
        int md = 0, pd = 0;
        walk_pairs(cells, B, b, th2, open, nopen, ls, [&](const PairAct &r, int A) {
            // both positions from one scan: counts of at most 256 in two halves
            int t;
            const int o = block_excl_scan<kListT>(r.m2l | r.p2p << 16, ls.sh, &t);
            if (r.m2l) mv[md + (o & 0xffff)] = A;
            if (r.p2p) pv[pd + (o >> 16)] = A;
            md += t & 0xffff;
            pd += t >> 16;
        });
    }
    __syncthreads();
    auto finish = [&](int32_t *v, int n, int32_t *out, int start, int p2p) {
        int bad = 0;
        for (int k = threadIdx.x; k + 1 < n; k += kListT) bad |= v[k] > v[k + 1];
        if (__syncthreads_or(bad)) {
            if (v != out) {
                block_sort(v, n);
            } else if (threadIdx.x == 0) {
                const unsigned long long at = atomicAdd(&bs->longs, 1ull << kLongShift | (unsigned long long)n);
                longs[at >> kLongShift] = LongList{start, n, (uint32_t)at, p2p};
            }
        }
        if (v != out)
            for (int k = threadIdx.x; k < n; k += kListT) out[k] = v[k];
    };
    finish(mv, mn, m2l_src + m0, m0, 0);
    finish(pv, pn, p2p_src + p0, p0, 1);
    __syncthreads();
    if (pn) {
        long long c = 0;
        for (int k = threadIdx.x; k < pn; k += kListT) c += cells[pv[k]].count;
        for (int w = 32; w > 0; w >>= 1) c += __shfl_xor(c, w, 64);
        if ((threadIdx.x & 63) == 0) atomicAdd((unsigned long long *)&s_cost, (unsigned long long)c);
    }
    int lo[3] = {INT_MAX, INT_MAX, INT_MAX}, hi[3] = {INT_MIN, INT_MIN, INT_MIN};
    if (key && mn) {
        int first = INT_MAX;
        for (int k = threadIdx.x; k < mn; k += kListT) {
            first = min(first, mv[k]);
            const DevCell A = cells[mv[k]];
            if (A.level != b.level) continue;
            const int o[3] = {A.ix - b.ix, A.iy - b.iy, A.iz - b.iz};
#pragma unroll
            for (int d = 0; d < 3; ++d) {
                lo[d] = min(lo[d], o[d]);
                hi[d] = max(hi[d], o[d]);
            }
        }
#pragma unroll
        for (int d = 0; d < 3; ++d) {
            for (int w = 32; w > 0; w >>= 1) {
                lo[d] = min(lo[d], __shfl_xor(lo[d], w, 64));
                hi[d] = max(hi[d], __shfl_xor(hi[d], w, 64));
            }
            if ((threadIdx.x & 63) == 0) {
                atomicMin(&s_lo[d], lo[d]);
                atomicMax(&s_hi[d], hi[d]);
            }
        }
        for (int w = 32; w > 0; w >>= 1) first = min(first, __shfl_xor(first, w, 64));
        if ((threadIdx.x & 63) == 0) atomicMin(&s_first, first);
    }
    __syncthreads();
    if (threadIdx.x != 0) return;
    cost[B] = s_cost * (long long)b.count;
    if (!key) return;
    val[B] = B;
    if (mn == 0) {
        key[B] = kEmptyKey;
        return;
    }
#pragma unroll
    for (int d = 0; d < 3; ++d) {
        lo[d] = s_lo[d];
        hi[d] = s_hi[d];
    }
    if (lo[0] > hi[0])   // no same-level source
        for (int d = 0; d < 3; ++d) lo[d] = hi[d] = 0;
    bool ok = mn <= 8191 && b.level < 32;
    uint64_t k = ((uint64_t)b.level << 58) |
                 ((uint64_t)(((b.ix & 1) << 2) | ((b.iy & 1) << 1) | (b.iz & 1)) << 55);
    for (int d = 0; d < 3; ++d) {
        ok = ok && lo[d] >= -64 && lo[d] < 64 && hi[d] >= -64 && hi[d] < 64;
        k |= (uint64_t)((lo[d] + 64) & 127) << (48 - 14 * d);
        k |= (uint64_t)((hi[d] + 64) & 127) << (41 - 14 * d);
    }
    k |= (uint64_t)(8191 - min(mn, 8191));
    key[B] = k;
    if (!ok) atomicOr(&bs->info[1], 1ull);   // a key field overflows
    // shallowest levels (cells are level-major); read first: few cells lower them
    const unsigned long long tl = b.level, sl = cells[s_first].level;
    if (tl < __hip_atomic_load(&bs->info[4], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT)) atomicMin(&bs->info[4], tl);
    if (sl < __hip_atomic_load(&bs->info[5], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT)) atomicMin(&bs->info[5], sl);
}

// entries of long lists [l0, l0 + gridDim.x): the key is the list's first entry
// (after `base`) before the source, so one sort sorts every list in its place
__global__ void long_keys_kernel(const LongList *__restrict__ longs, int l0, uint32_t base, int bits,
                                 const int32_t *__restrict__ m2l_src, const int32_t *__restrict__ p2p_src,
                                 uint64_t *__restrict__ key, int32_t *__restrict__ val)
{
    const int l = l0 + blockIdx.x;
    const LongList L = longs[l];
    const int32_t *src = (L.p2p ? p2p_src : m2l_src) + L.start;
    const uint32_t f = L.first - base;
    for (int k = blockIdx.y * blockDim.x + threadIdx.x; k < L.n; k += gridDim.y * blockDim.x) {
        key[f + k] = (uint64_t)f << bits | (uint32_t)src[k];
        val[f + k] = l;
    }
}

__global__ void long_store_kernel(const LongList *__restrict__ longs, int n, uint32_t base, int bits,
                                  const uint64_t *__restrict__ key, const int32_t *__restrict__ val,
                                  int32_t *__restrict__ m2l_src, int32_t *__restrict__ p2p_src)
{
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= n) return;
    const LongList L = longs[val[i]];
    (L.p2p ? p2p_src : m2l_src)[L.start + (i - (int)(L.first - base))] = (int32_t)(key[i] & ((1ull << bits) - 1));
}

__global__ void last_of_scans_kernel(int32_t *mptr, int32_t *pptr, int nc, const BuildState *bs)
{
    if (threadIdx.x != 0) return;
    mptr[nc] = (int32_t)bs->nm2l;
    pptr[nc] = (int32_t)bs->np2p;
}

__global__ void zero_i32_kernel(int32_t *p, int64_t n)
{
    for (int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; i < n; i += (int64_t)gridDim.x * blockDim.x) p[i] = 0;
}

// ---------------------------------------------------------------- host side
// Scratch memory of one build.  Blocks come first from the context's
// arena by bumping a pointer (a released arena block is reused only by the
// next build on the same stream, after this one's work); what does not fit
// comes from the stream-ordered allocator, and the arena grows to this
// build's total (up to the context's cache limit) for the next build.
struct Dev {
    hipStream_t s;
    fmm_ctx *ctx;
    size_t used = 0, need = 0;
    std::vector<void *> blocks;
    hipError_t err = hipSuccess;
    template <typename T>
    T *alloc(size_t count)
    {
        void *p = nullptr;
        if (err != hipSuccess) return nullptr;
        const size_t b = (std::max<size_t>(count, 1) * sizeof(T) + 255) / 256 * 256;
        need += b;
        if (ctx->arena && used + b <= ctx->arena_cap) {
            p = ctx->arena + used;
            used += b;
            return (T *)p;
        }
        err = hipMallocAsync(&p, b, s);
        if (err != hipSuccess) return nullptr;
        blocks.push_back(p);
        return (T *)p;
    }
    void release(void *p)
    {
        auto it = std::find(blocks.begin(), blocks.end(), p);
        if (it != blocks.end()) {
            hipFreeAsync(p, s);
            blocks.erase(it);
        }
    }
    ~Dev()
    {
        for (void *p : blocks) hipFreeAsync(p, s);
        if (need > ctx->arena_cap && err == hipSuccess) {
            // twice this build's need (at least 32 MB), so that builds up to
            // twice as large grow it no further
            const size_t want = std::min(std::max(2 * need, (size_t)32 << 20), ctx_cache_limit(ctx));
            if (want > ctx->arena_cap) {
                if (ctx->arena) hipFreeAsync(ctx->arena, s);
                ctx->arena = nullptr;
                ctx->arena_cap = 0;
                void *p = nullptr;
                if (hipMallocAsync(&p, want, s) == hipSuccess) {
                    ctx->arena = (char *)p;
                    ctx->arena_cap = want;
                } else {
                    (void)hipGetLastError();
                }
            }
        }
    }
};

#define GCHK(expr)                              \
    do {                                        \
        hipError_t e_ = (expr);                 \
        if (e_ != hipSuccess) return e_;        \
    } while (0)

inline unsigned nblk(int64_t n, int t) { return (unsigned)std::max<int64_t>(1, (n + t - 1) / t); }

// exclusive scan of n int32 values into out (in place allowed); the 64-bit
// total goes to the device word *total.  No host synchronisation.
hipError_t scan_i32(Dev &dv, const int32_t *in, int32_t *out, int n, int64_t *total)
{
    if (n <= kSmallScan) {
        hipLaunchKernelGGL(scan_small_kernel, dim3(1), dim3(kSmallT), 0, dv.s, in, out, n, total);
        return hipGetLastError();
    }
    const int nb = (int)nblk(n, kScanTile);
    int32_t *sums = dv.alloc<int32_t>(nb);
    GCHK(dv.err);
    hipLaunchKernelGGL(scan_tile_kernel, dim3(nb), dim3(kScanT), 0, dv.s, in, out, n, sums);
    hipLaunchKernelGGL(scan_sums_kernel, dim3(1), dim3(kScanT), 0, dv.s, sums, nb, total);
    hipLaunchKernelGGL(scan_add_kernel, dim3(nb), dim3(kScanT), 0, dv.s, out, n, sums);
    GCHK(hipGetLastError());
    dv.release(sums);
    return hipSuccess;
}

// Read-backs of a few device words through the context's coherent host
// words: one thread copies them with system-scope stores, then stores the
// read-back's sequence number with release order, and the host polls that
// number (about 6 us from the kernel's launch to the words on the host,
// against about 14 us for a copy and a stream wait).  After kSigSpin of
// polling the host waits for the stream instead, which also reports a
// failed kernel.
constexpr int kSigWords = 64;                  // words one read-back carries; the sequence number follows
constexpr double kSigSpinUs = 1000.0;
__global__ void publish_kernel(const int64_t *__restrict__ src, int n, int64_t *host, int64_t seq)
{
    if (threadIdx.x != 0) return;
    for (int i = 0; i < n; ++i) __hip_atomic_store(&host[i], src[i], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
    __hip_atomic_store(&host[kSigWords], seq, __ATOMIC_RELEASE, __HIP_MEMORY_SCOPE_SYSTEM);
}

// the first k <= kSigWords device words (8-byte aligned), read on the host;
// this waits for the stream's work up to them
hipError_t read_words(Dev &dv, const void *dev, int k, void *host)
{
    fmm_ctx *c = dv.ctx;
    const int64_t seq = ++c->sig_seq;
    hipLaunchKernelGGL(publish_kernel, dim3(1), dim3(64), 0, dv.s, (const int64_t *)dev, k, c->sig_dev, seq);
    GCHK(hipGetLastError());
    const auto t0 = std::chrono::steady_clock::now();
    while (__atomic_load_n(&c->sig[kSigWords], __ATOMIC_ACQUIRE) != seq) {
        if (std::chrono::duration<double, std::micro>(std::chrono::steady_clock::now() - t0).count() > kSigSpinUs) {
            GCHK(hipStreamSynchronize(dv.s));
            if (__atomic_load_n(&c->sig[kSigWords], __ATOMIC_ACQUIRE) != seq) return hipErrorUnknown;
            break;
        }
    }
    memcpy(host, c->sig, sizeof(int64_t) * k);
    return hipSuccess;
}

// stable sort of (key, val) on the low `bits` bits of the key: one workgroup
// for at most kSmallSort items, else the library radix sort (8-bit digits);
// the result ends in k/v (the buffers are swapped as needed)
hipError_t radix_sort(Dev &dv, uint64_t *&k, int32_t *&v, int n, int bits)
{
    if (n <= 1) return hipSuccess;
    if (n <= kSmallSort) {
        const uint64_t mask = bits >= 64 ? ~0ull : (1ull << bits) - 1;
        hipLaunchKernelGGL(small_sort_kernel, dim3(1), dim3(kSmallSortT), 0, dv.s, k, v, n, mask);
        return hipGetLastError();
    }
    size_t tb = 0;
    GCHK(dev_sort_pairs(nullptr, tb, k, nullptr, v, nullptr, n, std::min(bits, 64), dv.s));
    uint64_t *k2 = dv.alloc<uint64_t>(n);
    int32_t *v2 = dv.alloc<int32_t>(n);
    char *tmp = dv.alloc<char>(tb);
    GCHK(dv.err);
    GCHK(dev_sort_pairs(tmp, tb, k, k2, v, v2, n, std::min(bits, 64), dv.s));
    std::swap(k, k2);
    std::swap(v, v2);
    return hipSuccess;
}

// The long lists lists_emit_kernel left unsorted (`nlong` of them, `total`
// entries), by one radix sort of all their entries, kLongBatch at most at a
// time (whole lists).  A workgroup that sorts its list in global memory keeps
// the rest waiting: dense cores with a few far particles, 30 000 points (longest
// list 18 085), lists and schedule 1.65 -> 0.53 ms; 1.2 million (109 719)
// 11.1 -> 2.4.
constexpr int64_t kLongBatch = 1 << 22;   // 150 MB of scratch
hipError_t sort_long_lists(Dev &dv, const LongList *longs, int64_t nlong, int64_t total, int nc, int32_t *m2l_src,
                           int32_t *p2p_src)
{
    hipStream_t s = dv.s;
    // list ranges and first entries of the batches
    std::vector<int64_t> l0{0, nlong}, e0{0, total};
    int64_t cap = total;
    if (total > kLongBatch) {
        std::vector<LongList> h((size_t)nlong);
        GCHK(hipMemcpyAsync(h.data(), longs, sizeof(LongList) * h.size(), hipMemcpyDeviceToHost, s));
        GCHK(hipStreamSynchronize(s));
        l0.assign(1, 0);
        e0.assign(1, 0);
        cap = 0;
        for (int64_t l = 0; l < nlong; ++l)
            if ((int64_t)h[l].first + h[l].n - e0.back() > kLongBatch && l > l0.back()) {
                l0.push_back(l);
                e0.push_back(h[l].first);
            }
        l0.push_back(nlong);
        e0.push_back(total);
        for (size_t k = 0; k + 1 < e0.size(); ++k) cap = std::max(cap, e0[k + 1] - e0[k]);
        if (cap > INT32_MAX) return hipErrorOutOfMemory;
    }
    uint64_t *key = dv.alloc<uint64_t>(cap), *key2 = dv.alloc<uint64_t>(cap);
    int32_t *val = dv.alloc<int32_t>(cap), *val2 = dv.alloc<int32_t>(cap);
    size_t tb = 0;
    auto width = [](int64_t v) { return 64 - __builtin_clzll((unsigned long long)v | 1); };
    const int bits = width(nc - 1), all = bits + width(cap);
    GCHK(dev_sort_pairs(nullptr, tb, key, key2, val, val2, (int)cap, all, s));
    char *tmp = dv.alloc<char>(tb);
    GCHK(dv.err);
    for (size_t k = 0; k + 1 < l0.size(); ++k) {
        const int n = (int)(e0[k + 1] - e0[k]);
        for (int64_t l = l0[k]; l < l0[k + 1]; l += 32768)
            hipLaunchKernelGGL(long_keys_kernel, dim3((unsigned)std::min<int64_t>(32768, l0[k + 1] - l), 16), dim3(256), 0, s,
                               longs, (int)l, (uint32_t)e0[k], bits, (const int32_t *)m2l_src, (const int32_t *)p2p_src, key,
                               val);
        GCHK(hipGetLastError());
        size_t tb2 = tb;
        GCHK(dev_sort_pairs(tmp, tb2, key, key2, val, val2, n, all, s));
        hipLaunchKernelGGL(long_store_kernel, dim3(nblk(n, 256)), dim3(256), 0, s, longs, n, (uint32_t)e0[k], bits,
                           (const uint64_t *)key2, (const int32_t *)val2, m2l_src, p2p_src);
        GCHK(hipGetLastError());
    }
    return hipSuccess;
}

// host staging of the device-to-host copies: the context's pinned buffer
// (fast, asynchronous copies), grown on demand
struct Staging {
    fmm_ctx *ctx;
    char *base = nullptr;
    hipError_t reserve(size_t bytes) { return ctx_pinned(ctx, bytes, &base); }
};

// ------------------------------------------------------------------ M2L scheduling
// The tiling of build_m2l_tiling (tree_host.cpp) on the device, with the same
// result: targets in (level, octant, same-level signature, list length
// descending, cell) order, 64 to a tile; per tile the sorted distinct pair
// geometries; class ids the ranks in the sorted union; per entry and lane
// the source (or the zero row).  Keys are packed into 64 bits in the order
// of the host comparators; a key that does not fit (or a tile with more
// distinct geometries than its hash table holds) sends the tree back to the
// host code.

constexpr int kTileHashBits = 13;
constexpr int kTileHash = 1 << kTileHashBits;   // open-addressing slots per tile (LDS)
constexpr int kTileMaxU = kTileHash / 2;        // distinct geometries a tile may have here
constexpr int64_t kClsR = 1 << 18;         // offset range of a packed pair geometry
// the table of all tiles' distinct geometries (global memory), and how many of
// them are ranked by counting; trees with more take a sort of all entries
constexpr int kClsHashBits = 16;
constexpr int kClsHash = 1 << kClsHashBits;
constexpr int kClsMax = 1 << 13;

// first probe of a key in the tile table (Fibonacci hashing)
__device__ __forceinline__ int tile_slot(uint64_t k) { return (int)((k * 0x9E3779B97F4A7C15ull) >> (64 - kTileHashBits)); }

// (dl + 32) << 57 | (d0 + R) << 38 | (d1 + R) << 19 | (d2 + R): the order
// of (dl, d0, d1, d2)
__device__ __forceinline__ bool pack_class(const DevCell &A, const DevCell &B, uint64_t &key)
{
    const int la = A.level, lb = B.level, lm = max(la, lb);
    const int64_t d0 = ((2 * (int64_t)B.ix + 1) << (lm - lb)) - ((2 * (int64_t)A.ix + 1) << (lm - la));
    const int64_t d1 = ((2 * (int64_t)B.iy + 1) << (lm - lb)) - ((2 * (int64_t)A.iy + 1) << (lm - la));
    const int64_t d2 = ((2 * (int64_t)B.iz + 1) << (lm - lb)) - ((2 * (int64_t)A.iz + 1) << (lm - la));
    const bool ok = d0 >= -kClsR && d0 < kClsR && d1 >= -kClsR && d1 < kClsR && d2 >= -kClsR && d2 < kClsR;
    key = ((uint64_t)(lb - la + 32) << 57) | ((uint64_t)(d0 + kClsR) << 38) | ((uint64_t)(d1 + kClsR) << 19) |
          (uint64_t)(d2 + kClsR);
    return ok;
}

__device__ __forceinline__ void unpack_class(uint64_t k, int &dl, int64_t &d0, int64_t &d1, int64_t &d2)
{
    const uint64_t m = (1ull << 19) - 1;
    dl = (int)(k >> 57) - 32;
    d0 = (int64_t)((k >> 38) & m) - kClsR;
    d1 = (int64_t)((k >> 19) & m) - kClsR;
    d2 = (int64_t)(k & m) - kClsR;
}

__device__ __forceinline__ void class_geom(uint64_t k, double *g)
{
    int dl;
    int64_t d0, d1, d2;
    unpack_class(k, dl, d0, d1, d2);
    const double unit = ldexp(1.0, min(0, dl));
    g[0] = (double)d0 * unit;
    g[1] = (double)d1 * unit;
    g[2] = (double)d2 * unit;
    g[3] = ldexp(1.0, dl);
}

__device__ __forceinline__ int cls_slot(uint64_t k) { return (int)((k * 0x9E3779B97F4A7C15ull) >> (64 - kClsHashBits)); }

// one workgroup per tile: the tile's distinct pair geometries in an LDS hash
// table, sorted, to a segment of `useg` that an atomic hands out (tseg: start,
// number), and added to the table of all tiles' (`table`; read before the
// compare-and-swap, since most are there already).  flags (info[1]): 2 a tile
// with too many, 4 too many in all to be ranked by counting.
constexpr int kClsT = 1024;   // threads per tile: kClsT / 64 per lane
__global__ __launch_bounds__(kClsT) void tile_classes_kernel(const DevCell *__restrict__ cells, int nc,
                                                             const uint64_t *__restrict__ tkey,
                                                             const int32_t *__restrict__ tcell,
                                                             const int32_t *__restrict__ ptr,
                                                             const int32_t *__restrict__ src, BuildState *bs,
                                                             unsigned long long *__restrict__ table,
                                                             uint64_t *__restrict__ ckey, int32_t *__restrict__ cslot,
                                                             int2 *__restrict__ tseg, int32_t *__restrict__ tcnt,
                                                             uint64_t *__restrict__ useg)
{
    __shared__ uint64_t tab[kTileHash];
    __shared__ uint64_t U[kTileMaxU];
    __shared__ int cnt, bad, fill, seg;
    const int tile = blockIdx.x;
    unsigned long long *info = bs->info;
    if (tkey[tile * kTileW] == kEmptyKey) {   // past the last target
        if (threadIdx.x == 0) tcnt[tile] = 0;
        return;
    }
    for (int h = threadIdx.x; h < kTileHash; h += blockDim.x) tab[h] = kEmptyKey;
    if (threadIdx.x == 0) {
        cnt = 0;
        bad = 0;
        fill = 0;
    }
    __syncthreads();
    // kClsT / 64 threads per lane, each taking every (kClsT / 64)-th entry of the lane's list
    const int lane = threadIdx.x & 63, part = threadIdx.x >> 6;
    const int slot = tile * kTileW + lane;
    const int B = slot < nc && tkey[slot] != kEmptyKey ? tcell[slot] : -1;
    if (part == 0 && B >= 0 && (slot + 1 == nc || tkey[slot + 1] == kEmptyKey)) info[0] = (unsigned long long)(slot + 1);
    const int e0 = B >= 0 ? ptr[B] : 0, e1 = B >= 0 ? ptr[B + 1] : 0;
    const DevCell cb = cells[B >= 0 ? B : 0];
    auto insert = [&](uint64_t k) {
        int h = tile_slot(k);
        for (int n = 0; n < kTileHash; ++n) {
            const uint64_t old = atomicCAS((unsigned long long *)&tab[h], (unsigned long long)kEmptyKey,
                                           (unsigned long long)k);
            if (old == kEmptyKey) {
                if (atomicAdd(&cnt, 1) >= kTileMaxU) bad = 1;
                return;
            }
            if (old == k) return;
            h = (h + 1) & (kTileHash - 1);
        }
        bad = 1;
    };
    // (a tile given up is left at once: in a full table every look-up walks it all)
    for (int e = e0 + part; e < e1 && !*(volatile int *)&bad; e += kClsT / 64) {
        uint64_t k;
        if (!pack_class(cells[src[e]], cb, k)) bad = 1;
        insert(k);
    }
    __syncthreads();
    if (bad) {
        if (threadIdx.x == 0) {
            atomicOr(&info[1], 2ull);
            tcnt[tile] = 0;
            tseg[tile] = make_int2(0, 0);
        }
        return;
    }
    const int nu = cnt;
    if (threadIdx.x == 0) {
        seg = atomicAdd(&bs->cursor, nu);
        tcnt[tile] = nu;
        tseg[tile] = make_int2(seg, nu);
    }
    // compact, then a bitonic sort of the next power of two
    for (int h = threadIdx.x; h < kTileHash; h += blockDim.x)
        if (tab[h] != kEmptyKey) U[atomicAdd(&fill, 1)] = tab[h];
    int np = 1;
    while (np < nu) np <<= 1;
    __syncthreads();
    for (int j = nu + threadIdx.x; j < np; j += blockDim.x) U[j] = kEmptyKey;
    __syncthreads();
    for (int k = 2; k <= np; k <<= 1)
        for (int j = k >> 1; j > 0; j >>= 1) {
            for (int i = threadIdx.x; i < np; i += blockDim.x) {
                const int l = i ^ j;
                if (l > i) {
                    const uint64_t a = U[i], b = U[l];
                    const bool up = (i & k) == 0;
                    if ((a > b) == up) {
                        U[i] = b;
                        U[l] = a;
                    }
                }
            }
            __syncthreads();
        }
    for (int j = threadIdx.x; j < nu; j += blockDim.x) {
        const uint64_t k = U[j];
        useg[seg + j] = k;
        int h = cls_slot(k);
        for (int n = 0; n < kClsHash; ++n) {
            unsigned long long old = __hip_atomic_load(&table[h], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            if (old == kEmptyKey) {
                old = atomicCAS(&table[h], (unsigned long long)kEmptyKey, (unsigned long long)k);
                if (old == kEmptyKey) {
                    const unsigned long long c = atomicAdd(&info[3], 1ull);
                    if (c < (unsigned long long)kClsMax) {
                        ckey[c] = k;
                        cslot[c] = h;
                    } else {
                        atomicOr(&info[1], 4ull);
                    }
                    break;
                }
            }
            if (old == k) break;
            if (__hip_atomic_load(&info[1], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) & 4ull) break;   // the table is not used
            h = (h + 1) & (kClsHash - 1);
        }
    }
}

// Last block: the tiles' entry offsets (scan of tcnt, its total as the last).
// The others: the rank of every distinct geometry among all, by counting the
// smaller ones (keys through LDS): class id of its table slot, and the class
// geometry.  Counting spreads over the chip and has no passes to wait for:
// 100k dipoles (418 classes) 32 -> 5 us against a sort by one workgroup.
constexpr int kRankT = 256;
constexpr int kRankKeys = kRankT / 4;        // keys per workgroup, four threads each
__global__ __launch_bounds__(kRankT) void class_rank_kernel(BuildState *bs, const int32_t *__restrict__ tcnt,
                                                            int32_t *__restrict__ uoff, int ntmax,
                                                            const uint64_t *__restrict__ ckey,
                                                            const int32_t *__restrict__ cslot,
                                                            int32_t *__restrict__ crank, double *__restrict__ geom)
{
    if (blockIdx.x == kClsMax / kRankKeys) {
        __shared__ int sh[kRankT / 64];
        const int per = (ntmax + kRankT - 1) / kRankT;
        const int b0 = min(ntmax, (int)threadIdx.x * per), b1 = min(ntmax, b0 + per);
        int s = 0, tot;
        long long s64 = 0;
        for (int b = b0; b < b1; ++b) s64 += tcnt[b];
        s = (int)s64;
        int run = block_excl_scan<kRankT>(s, sh, &tot);
        for (int b = b0; b < b1; ++b) {
            uoff[b] = run;
            run += tcnt[b];
        }
        if (s64) atomicAdd(&bs->info[2], (unsigned long long)s64);   // in 64 bits: the host checks the range
        if (threadIdx.x == 0) uoff[ntmax] = tot;
        return;
    }
    if (bs->info[1]) return;                 // another path makes the classes
    const int ncls = (int)bs->info[3];
    const int r0 = blockIdx.x * kRankKeys;
    if (r0 >= ncls) return;
    __shared__ uint64_t K[1024];
    const int q = r0 + (threadIdx.x >> 2), part = threadIdx.x & 3;
    const uint64_t k = q < ncls ? ckey[q] : 0;
    int rank = 0;
    for (int c0 = 0; c0 < ncls; c0 += 1024) {
        const int m = min(1024, ncls - c0);
        __syncthreads();
        for (int j = threadIdx.x; j < m; j += kRankT) K[j] = ckey[c0 + j];
        __syncthreads();
        for (int j = part; j < m; j += 4) rank += K[j] < k;
    }
    rank += __shfl_xor(rank, 1, 4);
    rank += __shfl_xor(rank, 2, 4);
    if (part == 0 && q < ncls) {
        crank[cslot[q]] = rank;
        class_geom(k, geom + 4 * rank);
    }
}

// one workgroup per tile: every entry's class and every (entry, lane) source
// (the zero row, cell nc, where a lane lacks the class), and the targets'
// slots.  table null: the classes come from the sort of all entries, for which
// the sorted geometries go to ukey / uidx in entry order.
__global__ __launch_bounds__(kClsT) void tile_emit_kernel(const DevCell *__restrict__ cells, int nc, int ntg,
                                                          const int32_t *__restrict__ tcell,
                                                          const int32_t *__restrict__ ptr,
                                                          const int32_t *__restrict__ src, const int2 *__restrict__ tseg,
                                                          const uint64_t *__restrict__ useg,
                                                          const int32_t *__restrict__ uoff,
                                                          const unsigned long long *__restrict__ table,
                                                          const int32_t *__restrict__ crank, int32_t *__restrict__ ucls,
                                                          int32_t *__restrict__ usrc, int32_t *__restrict__ cell_slot,
                                                          uint64_t *__restrict__ ukey, int32_t *__restrict__ uidx)
{
    __shared__ uint64_t U[kTileMaxU];
    const int tile = blockIdx.x, base = uoff[tile];
    const int2 sg = tseg[tile];
    for (int j = threadIdx.x; j < sg.y; j += kClsT) {
        const uint64_t k = useg[sg.x + j];
        U[j] = k;
        if (table) {
            int h = cls_slot(k);
            while (table[h] != k) h = (h + 1) & (kClsHash - 1);
            ucls[base + j] = crank[h];
        } else {
            ukey[base + j] = k;
            uidx[base + j] = base + j;
        }
    }
    int32_t *rows = usrc + (size_t)base * kTileW;
    for (int j = threadIdx.x; j < sg.y * kTileW; j += kClsT) rows[j] = nc;
    __syncthreads();
    const int lane = threadIdx.x & 63, part = threadIdx.x >> 6;
    const int slot = tile * kTileW + lane;
    const int B = slot < ntg ? tcell[slot] : -1;
    if (part == 0 && B >= 0) cell_slot[B] = slot;
    const int e0 = B >= 0 ? ptr[B] : 0, e1 = B >= 0 ? ptr[B + 1] : 0;
    const DevCell cb = cells[B >= 0 ? B : 0];
    for (int e = e0 + part; e < e1; e += kClsT / 64) {
        const int A = src[e];
        uint64_t k;
        pack_class(cells[A], cb, k);
        int at = 0;                          // the last j with U[j] <= k
        for (int step = sg.y > 1 ? 1 << (31 - __clz(sg.y - 1)) : 0; step > 0; step >>= 1)
            if (at + step < sg.y && U[at + step] <= k) at += step;
        rows[(size_t)at * kTileW + lane] = A;
    }
}

// after the sort of all tiles' geometries: first-of-a-kind flags
__global__ void class_flags_kernel(const uint64_t *__restrict__ k, int n, int32_t *__restrict__ f)
{
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i < n) f[i] = (i == 0 || k[i] != k[i - 1]) ? 1 : 0;
}

// class id of every tile entry (the rank of its geometry) and the class geometry
__global__ void class_ids_kernel(const uint64_t *__restrict__ k, const int32_t *__restrict__ idx,
                                 const int32_t *__restrict__ rank_excl, const int32_t *__restrict__ f, int n,
                                 int32_t *__restrict__ ucls, double *__restrict__ geom)
{
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= n) return;
    const int r = rank_excl[i] + f[i] - 1;
    ucls[idx[i]] = r;
    if (f[i]) class_geom(k[i], geom + 4 * (size_t)r);
}

// Device M2L tiling, first part: the target order, the tiles' geometries and
// their offsets, the classes.  All sizes are bounded by the cells and list
// entries, so it needs no wait; the host then reads bs->info.
struct TileState {
    int32_t *tcell = nullptr, *uoff = nullptr, *tcnt = nullptr, *crank = nullptr;
    int2 *tseg = nullptr;
    uint64_t *useg = nullptr, *ckey = nullptr;
    int32_t *cslot = nullptr;
    unsigned long long *table = nullptr;
    double *geom = nullptr;
    int ntmax = 0, ntg = 0, ntiles = 0;
    int64_t nentries = 0;
};

hipError_t launch_tiling(Dev &dv, const DevCell *cells, int nc, uint64_t *key, int32_t *val, const int32_t *ptr,
                         const int32_t *src, int64_t nsrc, BuildState *bs, TileState &ts)
{
    hipStream_t s = dv.s;
    ts.ntmax = (int)nblk(nc, kTileW);
    ts.tcnt = dv.alloc<int32_t>(ts.ntmax);
    ts.tseg = dv.alloc<int2>(ts.ntmax);
    ts.uoff = dv.alloc<int32_t>((size_t)ts.ntmax + 1);
    ts.crank = dv.alloc<int32_t>(kClsHash);
    ts.ckey = dv.alloc<uint64_t>(kClsMax);
    ts.cslot = dv.alloc<int32_t>(kClsMax);
    ts.geom = dv.alloc<double>(4 * (size_t)kClsMax);
    // a tile holds no more geometries than its lists have entries
    ts.useg = dv.alloc<uint64_t>((size_t)std::max<int64_t>(1, std::min<int64_t>(nsrc, (int64_t)ts.ntmax * kTileMaxU)));
    GCHK(dv.err);
    GCHK(radix_sort(dv, key, val, nc, 64));
    ts.tcell = val;
    hipLaunchKernelGGL(tile_classes_kernel, dim3(ts.ntmax), dim3(kClsT), 0, s, cells, nc, (const uint64_t *)key,
                       (const int32_t *)val, ptr, src, bs, ts.table, ts.ckey, ts.cslot, ts.tseg, ts.tcnt, ts.useg);
    hipLaunchKernelGGL(class_rank_kernel, dim3(kClsMax / kRankKeys + 1), dim3(kRankT), 0, s, bs,
                       (const int32_t *)ts.tcnt, ts.uoff, ts.ntmax, (const uint64_t *)ts.ckey, (const int32_t *)ts.cslot,
                       ts.crank, ts.geom);
    return hipGetLastError();
}

// Second part, with the sizes known (info): the per-entry tables the tree
// keeps.  dt.done false: back to the host code (a packed key overflows, or a
// tile has too many distinct geometries).
hipError_t finish_tiling(Dev &dv, const DevCell *cells, int nc, const int32_t *ptr, const int32_t *src,
                         BuildState *bs, unsigned long long *info, DevKeep &dt, TileState &ts)
{
    hipStream_t s = dv.s;
    if ((info[1] & 3) || info[2] * (unsigned long long)kTileW > (unsigned long long)INT32_MAX) return hipSuccess;
    ts.ntg = (int)info[0];
    ts.ntiles = (ts.ntg + kTileW - 1) / kTileW;
    ts.nentries = (int64_t)info[2];
    const int64_t ne = ts.nentries;
    GCHK(dt.keep((void **)&dt.ucls, sizeof(int32_t) * (size_t)std::max<int64_t>(1, ne)));
    GCHK(dt.keep((void **)&dt.usrc, sizeof(int32_t) * (size_t)std::max<int64_t>(1, ne * kTileW)));
    dt.done = true;
    if (ne == 0) return hipSuccess;
    const bool sorted = (info[1] & 4) != 0;   // too many classes to count ranks: a sort of all entries
    uint64_t *ukey = nullptr;
    int32_t *uidx = nullptr;
    if (sorted) {
        ukey = dv.alloc<uint64_t>(ne);
        uidx = dv.alloc<int32_t>(ne);
        GCHK(dv.err);
    }
    hipLaunchKernelGGL(tile_emit_kernel, dim3(ts.ntiles), dim3(kClsT), 0, s, cells, nc, ts.ntg,
                       (const int32_t *)ts.tcell, ptr, src, (const int2 *)ts.tseg, (const uint64_t *)ts.useg,
                       (const int32_t *)ts.uoff, sorted ? nullptr : (const unsigned long long *)ts.table,
                       (const int32_t *)ts.crank, dt.ucls, dt.usrc, dt.cell_slot, ukey, uidx);
    GCHK(hipGetLastError());
    if (sorted) {
        int32_t *flag = dv.alloc<int32_t>(ne), *rank = dv.alloc<int32_t>(ne);
        ts.geom = dv.alloc<double>(4 * (size_t)ne);
        GCHK(dv.err);
        GCHK(radix_sort(dv, ukey, uidx, (int)ne, 64));
        hipLaunchKernelGGL(class_flags_kernel, dim3(nblk(ne, 256)), dim3(256), 0, s, ukey, (int)ne, flag);
        GCHK(hipGetLastError());
        GCHK(scan_i32(dv, flag, rank, (int)ne, (int64_t *)&bs->info[3]));
        hipLaunchKernelGGL(class_ids_kernel, dim3(nblk(ne, 256)), dim3(256), 0, s, ukey, uidx, rank, flag, (int)ne,
                           dt.ucls, ts.geom);
        GCHK(hipGetLastError());
        GCHK(read_words(dv, &bs->info[3], 1, &info[3]));
    }
    return hipSuccess;
}

// the lists' offsets (ptr over nc + 1) from their lengths, totals to the state
hipError_t list_offsets(Dev &dv, const int32_t *mcnt, int32_t *mptr, const int32_t *pcnt, int32_t *pptr, int nc,
                        BuildState *bs)
{
    if (nc <= kSmallScan) {
        Scan2 a{{mcnt, pcnt}, {mptr, pptr}, {&bs->nm2l, &bs->np2p}};
        hipLaunchKernelGGL(scan_small2_kernel, dim3(2), dim3(kSmallT), 0, dv.s, a, nc);
        return hipGetLastError();
    }
    GCHK(scan_i32(dv, mcnt, mptr, nc, &bs->nm2l));
    GCHK(scan_i32(dv, pcnt, pptr, nc, &bs->np2p));
    hipLaunchKernelGGL(last_of_scans_kernel, dim3(1), dim3(64), 0, dv.s, mptr, pptr, nc, (const BuildState *)bs);
    return hipGetLastError();
}

}  // namespace

hipError_t ctx_arena_reserve(fmm_ctx *ctx, size_t bytes)
{
    bytes = std::min(bytes, ctx_cache_limit(ctx));
    if (ctx->arena_cap >= bytes) return hipSuccess;
    if (ctx->arena) (void)hipFreeAsync(ctx->arena, ctx->stream);
    ctx->arena = nullptr;
    ctx->arena_cap = 0;
    void *p = nullptr;
    const hipError_t e = hipMallocAsync(&p, bytes, ctx->stream);
    if (e != hipSuccess) {
        (void)hipGetLastError();
        return e;
    }
    ctx->arena = (char *)p;
    ctx->arena_cap = bytes;
    return hipStreamSynchronize(ctx->stream);
}

// Builds the canonical tree (and, when theta > 0, the interaction lists) of
// the n device positions on the context's stream s, and returns it in host
// form.
hipError_t gpu_build_tree(const double *pos, int64_t n, int ncrit, double theta, bool lists, hipStream_t s,
                          HostTree &t, fmm_ctx *ctx, DevKeep &dt)
{
    t = HostTree();
    t.n = n;
    Dev dv{s, ctx};
    if (!ctx->sig) {
        GCHK(hipHostMalloc((void **)&ctx->sig, sizeof(int64_t) * (kSigWords + 1),
                           hipHostMallocCoherent | hipHostMallocMapped));
        ctx->sig[kSigWords] = ctx->sig_seq;
        const hipError_t e = hipHostGetDevicePointer((void **)&ctx->sig_dev, ctx->sig, 0);
        if (e != hipSuccess) {
            (void)hipHostFree(ctx->sig);
            ctx->sig = nullptr;
            return e;
        }
    }
    // wall-clock phases for the context's profile (the device work of a
    // phase is counted where the host next waits for it)
    auto t_last = std::chrono::steady_clock::now();
    auto mark = [&](const char *nm) {
        if (!ctx->profile) return;
        const auto now = std::chrono::steady_clock::now();
        ctx->prof.push_back(ProfEntry{nm, nullptr, nullptr, std::chrono::duration<double, std::milli>(now - t_last).count()});
        t_last = now;
    };
    // root box, keys, stable sort; the sorted keys and order go to the tree
    BuildState *bs = dv.alloc<BuildState>(1);
    const int nbb = (int)std::min<int64_t>(1024, nblk(n, 256));
    double *part = dv.alloc<double>(7 * (size_t)nbb);
    uint64_t *key = nullptr;
    int32_t *idx = nullptr;
    GCHK(dt.keep((void **)&key, sizeof(uint64_t) * n));
    GCHK(dt.keep((void **)&idx, sizeof(int32_t) * n));
    dt.key = key;
    dt.perm = idx;
    const bool big = n > kSmallSort;
    uint64_t *key0 = big ? dv.alloc<uint64_t>(n) : key;
    int32_t *idx0 = big ? dv.alloc<int32_t>(n) : idx;
    GCHK(dv.err);
    hipLaunchKernelGGL(bbox_partial_kernel, dim3(nbb), dim3(256), 0, s, pos, n, part);
    hipLaunchKernelGGL(bbox_final_kernel, dim3(1), dim3(256), 0, s, part, nbb, bs);
    hipLaunchKernelGGL(keys_kernel, dim3(nblk(n, 256)), dim3(256), 0, s, pos, (int)n, (const double *)bs->box, key0, idx0);
    GCHK(hipGetLastError());
    if (big) {
        size_t tb = 0;
        GCHK(dev_sort_pairs(nullptr, tb, key0, key, idx0, idx, (int)n, 3 * kMaxLevel, s));
        char *tmp = dv.alloc<char>(tb);
        GCHK(dv.err);
        GCHK(dev_sort_pairs(tmp, tb, key0, key, idx0, idx, (int)n, 3 * kMaxLevel, s));
    } else {
        GCHK(radix_sort(dv, key, idx, (int)n, 3 * kMaxLevel));
    }
    mark("host:tree_box");

    // the cells of every level
    const int nblock = (int)nblk(n, kCellT), nw = (int)std::min<int64_t>(ncrit, n);
    uchar2 *range = dv.alloc<uchar2>(n);
    int32_t *lcnt = dv.alloc<int32_t>((size_t)kLevels * nblock);
    int8_t *wide = nullptr;
    GCHK(dv.err);
    if (nw > kWinMax) {
        int8_t *w2 = dv.alloc<int8_t>(n);
        wide = dv.alloc<int8_t>(n);
        GCHK(dv.err);
        auto step = [&](int first, int back) {
            hipLaunchKernelGGL(window_max_kernel, dim3(nblk(n, 256)), dim3(256), 0, s, (const uint64_t *)key, (int)n, nw,
                               first, back, (const int8_t *)wide, w2);
            std::swap(wide, w2);
        };
        int half = 1;
        step(1, 0);
        for (; 2 * (int64_t)half <= (int64_t)nw + 1; half *= 2) step(0, half);
        step(0, nw + 1 - half);
    }
    hipLaunchKernelGGL(cell_depth_kernel, dim3(nblock), dim3(256), 0, s, (const uint64_t *)key, (int)n, nw,
                       (const int8_t *)wide, range, lcnt);
    hipLaunchKernelGGL(level_offsets_kernel, dim3(kLevels), dim3(kSmallT), 0, s, lcnt, nblock, bs);
    GCHK(hipGetLastError());
    static_assert(sizeof(BuildState) % 8 == 0 && sizeof(BuildState) <= 8 * kSigWords,
                  "the state is read back as whole words");
    BuildState hs;
    GCHK(read_words(dv, bs, (int)(sizeof(BuildState) / 8), &hs));
    if (hs.box[6] != 0.0) return hipErrorInvalidValue;   // a position is not finite
    {
        double W = std::max(hs.box[3] - hs.box[0], std::max(hs.box[4] - hs.box[1], hs.box[5] - hs.box[2]));
        if (W == 0.0) W = 1.0;
        for (int d = 0; d < 3; ++d) t.lo[d] = hs.box[d];
        t.W = W;
        t.h = std::ldexp(W, -22);
    }
    LevelPtr lp;
    int nlev = 0;
    int64_t nc64 = 0;
    for (int l = 0; l < kLevels; ++l) {
        lp.v[l] = (int32_t)nc64;
        if (hs.totals[l] > 0) {
            nlev = l + 1;
            t.level_ptr.push_back(nc64);
            nc64 += hs.totals[l];
        }
        if (nc64 > INT32_MAX) return hipErrorOutOfMemory;
    }
    lp.v[kLevels] = (int32_t)nc64;
    t.level_ptr.push_back(nc64);
    const int nc = (int)nc64;
    DevCell *cells = nullptr;
    GCHK(dt.keep((void **)&cells, sizeof(DevCell) * nc));
    dt.cells = cells;
    const bool tiling = lists && dt.tiling;
    TileState ts;
    if (tiling) {
        GCHK(dt.keep((void **)&dt.cell_slot, sizeof(int32_t) * (size_t)nc));
        ts.table = dv.alloc<unsigned long long>(kClsHash);
        GCHK(dv.err);
    }
    hipLaunchKernelGGL(cells_emit_kernel, dim3(nblock), dim3(kCellT), 0, s, (const uint64_t *)key, (int)n,
                       (const uchar2 *)range, (const int32_t *)lcnt, lp, nlev, cells);
    hipLaunchKernelGGL(cells_finish_kernel, dim3(std::max(nblk(nc, 256), 64u)), dim3(256), 0, s, cells, nc, dt.cell_slot,
                       (uint64_t *)ts.table, tiling ? kClsHash : 0);
    GCHK(hipGetLastError());
    mark("host:tree_sort_levels");

    // host staging: the cells now, the lists' offsets and costs and the
    // schedule's host parts later
    auto al = [](size_t b) { return (b + 255) / 256 * 256; };
    const int ntmax = (int)nblk(nc, kTileW);
    const size_t o_cells = 0, o_pp = o_cells + al(sizeof(DevCell) * nc), o_pk = o_pp + al(sizeof(int32_t) * (nc + 1)),
                 o_tc = o_pk + al(sizeof(int64_t) * nc), o_tu = o_tc + al(sizeof(int32_t) * nc),
                 o_end = o_tu + al(sizeof(int32_t) * (ntmax + 1));
    Staging st{ctx};
    GCHK(st.reserve(o_end));
    GCHK(hipMemcpyAsync(st.base + o_cells, cells, sizeof(DevCell) * nc, hipMemcpyDeviceToHost, s));
    auto host_cells = [&]() {
        const DevCell *hc = (const DevCell *)(st.base + o_cells);
        t.level.resize(nc);
        t.ix.resize(3 * (size_t)nc);
        t.first.resize(nc);
        t.count.resize(nc);
        t.parent.resize(nc);
        t.child0.resize(nc);
        t.nchild.resize(nc);
        for (int c = 0; c < nc; ++c) {
            const DevCell &d = hc[c];
            t.level[c] = d.level;
            t.ix[3 * c] = d.ix;
            t.ix[3 * c + 1] = d.iy;
            t.ix[3 * c + 2] = d.iz;
            t.first[c] = d.first;
            t.count[c] = d.count;
            t.parent[c] = d.parent;
            t.child0[c] = d.child0;
            t.nchild[c] = d.nchild;
        }
    };
    if (!lists) {
        GCHK(hipStreamSynchronize(s));
        mark("host:tree_copy");
        host_cells();
        mark("host:tree_copyback");
        return hipSuccess;
    }

    // the lists
    const double th2 = theta * theta;
    int32_t *mcnt = dv.alloc<int32_t>(nc), *pcnt = dv.alloc<int32_t>(nc);
    uint2 *open_seg = dv.alloc<uint2>(nc);
    int32_t *mptr = nullptr, *pptr = dv.alloc<int32_t>((size_t)nc + 1);
    GCHK(dv.err);
    if (tiling) {
        GCHK(dt.keep((void **)&dt.m2l_ptr, sizeof(int32_t) * ((size_t)nc + 1)));
        mptr = dt.m2l_ptr;
    } else {
        mptr = dv.alloc<int32_t>((size_t)nc + 1);
        GCHK(dv.err);
    }
    // Open pairs a cell leaves to its children: those too near to be accepted,
    // 4/3 pi theta^-3 of its size (33 at theta 0.5), over the cells that split
    // (an eighth of a uniform tree's, more of a clustered one's); a margin
    // over both (never more than every pair of cells, and at first no more than a
    // sixteenth of what the context may keep, 256 MB of the default budget),
    // and again with what was asked for where it does not do.
    const double rth = 0.5 / theta;
    unsigned cap = (unsigned)std::min(20.0 * rth * rth * rth * nc + 65536.0,
                                      std::min((double)nc * nc + 1.0, (double)(ctx_cache_limit(ctx) / 16 / sizeof(uint32_t))));
    cap = std::max(cap, 1u);
    uint32_t *open_buf = dv.alloc<uint32_t>(cap);
    GCHK(dv.err);
    for (;;) {
        for (int l = 0; l < nlev; ++l)
            hipLaunchKernelGGL(lists_count_kernel, dim3((unsigned)hs.totals[l]), dim3(kListT), 0, s,
                               (const DevCell *)cells, lp.v[l], th2, open_seg, open_buf, cap, bs, mcnt, pcnt);
        GCHK(hipGetLastError());
        GCHK(list_offsets(dv, mcnt, mptr, pcnt, pptr, nc, bs));
        GCHK(read_words(dv, bs, (int)(sizeof(BuildState) / 8), &hs));
        if (hs.down <= cap) break;
        if (cap == 4000000000u) return hipErrorOutOfMemory;
        cap = (unsigned)std::min(2.0 * (double)hs.down, 4.0e9);
        dv.release(open_buf);
        open_buf = dv.alloc<uint32_t>(cap);
        GCHK(dv.err);
        hipLaunchKernelGGL(zero_i32_kernel, dim3(1), dim3(64), 0, s, (int32_t *)&bs->down, (int64_t)2);
    }
    const int64_t n_m2l = hs.nm2l, n_p2p = hs.np2p;
    if (n_m2l > INT32_MAX || n_p2p > INT32_MAX) return hipErrorOutOfMemory;
    mark("host:tree_traverse");
    int32_t *msrc = nullptr, *psrc = nullptr;
    GCHK(dt.keep((void **)&psrc, sizeof(int32_t) * (size_t)std::max<int64_t>(1, n_p2p)));
    dt.p2p_src = psrc;
    if (tiling) {
        GCHK(dt.keep((void **)&dt.m2l_src, sizeof(int32_t) * (size_t)std::max<int64_t>(1, n_m2l)));
        msrc = dt.m2l_src;
    } else {
        msrc = dv.alloc<int32_t>(n_m2l);
    }
    int64_t *cost = dv.alloc<int64_t>(nc);
    LongList *longs = dv.alloc<LongList>((size_t)(n_m2l / kM2LBuf + n_p2p / kP2PBuf));
    uint64_t *tkey = tiling ? dv.alloc<uint64_t>(nc) : nullptr;
    int32_t *tval = tiling ? dv.alloc<int32_t>(nc) : nullptr;
    GCHK(dv.err);
    hipLaunchKernelGGL(lists_emit_kernel, dim3((unsigned)nc), dim3(kListT), 0, s, (const DevCell *)cells, th2,
                       (const uint2 *)open_seg, (const uint32_t *)open_buf, (const int32_t *)mptr, (const int32_t *)pptr,
                       bs, msrc, psrc, cost, tkey, tval, longs);
    GCHK(hipGetLastError());
    GCHK(hipMemcpyAsync(st.base + o_pp, pptr, sizeof(int32_t) * (nc + 1), hipMemcpyDeviceToHost, s));
    GCHK(hipMemcpyAsync(st.base + o_pk, cost, sizeof(int64_t) * nc, hipMemcpyDeviceToHost, s));
    mark("host:tree_lists");
    if (tiling) {
        GCHK(launch_tiling(dv, cells, nc, tkey, tval, mptr, msrc, n_m2l, bs, ts));
        GCHK(hipMemcpyAsync(st.base + o_tc, ts.tcell, sizeof(int32_t) * nc, hipMemcpyDeviceToHost, s));
        GCHK(hipMemcpyAsync(st.base + o_tu, ts.uoff, sizeof(int32_t) * (ts.ntmax + 1), hipMemcpyDeviceToHost, s));
    }
    // the cells arrived with the list lengths: the host takes them over while
    // the device works
    host_cells();
    GCHK(read_words(dv, bs, (int)(sizeof(BuildState) / 8), &hs));
    // (the schedule does not depend on the order within a list)
    if (hs.longs)
        GCHK(sort_long_lists(dv, longs, (int64_t)(hs.longs >> kLongShift),
                             (int64_t)(hs.longs & ((1ull << kLongShift) - 1)), nc, msrc, psrc));
    dt.done = false;
    if (tiling) GCHK(finish_tiling(dv, cells, nc, mptr, msrc, bs, hs.info, dt, ts));
    mark("host:tree_tiling");
    const int32_t *pp = (const int32_t *)(st.base + o_pp);
    t.p2p_ptr.assign(pp, pp + nc + 1);
    const int64_t *pk = (const int64_t *)(st.base + o_pk);
    t.p2p_cost.assign(pk, pk + nc);
    if (tiling && dt.done) {
        M2LTiling &tl = *dt.tl;
        tl = M2LTiling();
        tl.on_device = true;
        tl.ntiles = ts.ntiles;
        tl.nentries = ts.nentries;
        tl.nclasses = ts.nentries ? (int)hs.info[3] : 0;
        dt.tgt_top = ts.ntg ? (int)hs.info[4] : -1;
        dt.src_top = ts.ntg ? (int)hs.info[5] : -1;
        tl.pairs = n_m2l;
        tl.tile_cell.assign((size_t)ts.ntiles * kTileW, -1);
        const int32_t *tc = (const int32_t *)(st.base + o_tc), *tu = (const int32_t *)(st.base + o_tu);
        std::copy(tc, tc + ts.ntg, tl.tile_cell.begin());
        tl.tile_uoff.assign(tu, tu + ts.ntiles + 1);
        GCHK(dt.keep((void **)&dt.cls_geom, sizeof(double) * 4 * (size_t)std::max(1, tl.nclasses)));
        if (tl.nclasses)
            GCHK(hipMemcpyAsync(dt.cls_geom, ts.geom, sizeof(double) * 4 * tl.nclasses, hipMemcpyDeviceToDevice, s));
    } else {
        // the host makes the schedule, from its own copy of the M2L lists: what
        // the tree holds for the device's goes back
        // (the staging buffer is free again: what came through it is taken over)
        const size_t o_src = al(sizeof(int32_t) * ((size_t)nc + 1));
        GCHK(st.reserve(o_src + sizeof(int32_t) * (size_t)n_m2l));
        GCHK(hipMemcpyAsync(st.base, mptr, sizeof(int32_t) * ((size_t)nc + 1), hipMemcpyDeviceToHost, s));
        if (n_m2l)
            GCHK(hipMemcpyAsync(st.base + o_src, msrc, sizeof(int32_t) * (size_t)n_m2l, hipMemcpyDeviceToHost, s));
        GCHK(hipStreamSynchronize(s));
        mark("host:tree_copy");
        const int32_t *hp = (const int32_t *)st.base, *hsrc = (const int32_t *)(st.base + o_src);
        t.m2l_ptr.assign(hp, hp + nc + 1);
        t.m2l_src.resize(n_m2l);
        for (int64_t k = 0; k < n_m2l; ++k) t.m2l_src[k] = hsrc[k];
        for (int32_t **p : {&dt.m2l_ptr, &dt.m2l_src, &dt.cell_slot}) {
            if (*p) dt.drop(*p);
            *p = nullptr;
        }
    }
    mark("host:tree_copyback");
    return hipSuccess;
}
