// Barnes-Hut evaluation of potential and field (the kernel is in
// bh_kernel.h; its instantiations, with and without the field gradient, per
// source order, are generated translation units, gen_bh.py).
#include "bh_kernel.h"

static bh_fn bh_select(bool grad, int s, int p, bool f32, bool h)
{
    switch (s) {
    case 0: return grad ? bh_select_g_s0(p, f32, h) : bh_select_f_s0(p, f32, h);
    case 1: return grad ? bh_select_g_s1(p, f32, h) : bh_select_f_s1(p, f32, h);
    case 2: return grad ? bh_select_g_s2(p, f32, h) : bh_select_f_s2(p, f32, h);
    case 3: return grad ? bh_select_g_s3(p, f32, h) : bh_select_f_s3(p, f32, h);
    default: return nullptr;
    }
}

namespace {

// counters are cleared by a kernel, not a memset, so that the launch
// sequence can be captured into a graph
__global__ void zero_u64_kernel(unsigned long long *p, int n)
{
    if ((int)threadIdx.x < n) p[threadIdx.x] = 0;
}

// the sums of the wavefronts that share a group, in their order, to the
// caller's order; no = 4 (phi, E) or 10 (and the gradient) a particle
__global__ void bh_reduce_kernel(int n, int split, int no, int outputs, const double *__restrict__ part,
                                 const int32_t *__restrict__ perm, double *__restrict__ phi,
                                 double *__restrict__ field, double *__restrict__ grad)
{
    const int id = blockIdx.x * blockDim.x + threadIdx.x;
    if (id >= n * no) return;
    const int i = id / no, c = id % no;
    double v = 0.0;
    for (int k = 0; k < split; ++k) v += part[(size_t)k * n * no + id];
    const size_t o = (size_t)perm[i];
    if (c == 0) {
        if (outputs & FMM_POT) phi[o] = v;
    } else if (c < 4) {
        if (outputs & FMM_FIELD) field[3 * o + c - 1] = v;
    } else if (outputs & FMM_GRAD) {
        grad[6 * o + c - 4] = v;
    }
}

}  // namespace

// Wavefronts a group of 64 particles: as many, up to eight, as keep them within
// one a SIMD (what fits of the kernels of the highest orders): they all run
// side by side then and the launch takes as long as the longest.
// Passes of 2001 Plummer dipoles, p 6: 569 -> 370 us; 5001 octupoles, FP64:
// 707 -> 157; 30 011 charges, p 10 (two a group): 1067 -> 627.  With up to 3072
// wavefronts the orders that fit one a SIMD queue for it and lose (30 011
// dipoles, p 8, FP64: 1732 -> 2343 us; 1642 with this limit).
static int bh_split(int64_t n, int ncu)
{
    const int64_t groups = (n + 63) / 64;
    int k = 1;
    while (k < 8 && 2 * k * groups <= 4 * ncu) k *= 2;
    return k;
}
// doubles of the sums of n particles, and the most any n takes: 64 particles a
// wavefront, phi, E and the gradient
size_t bh_part_doubles(int64_t n, int ncu)
{
    const int k = bh_split(n, ncu);
    return k > 1 ? (size_t)k * n * 10 : 0;
}
size_t bh_part_max(int ncu) { return (size_t)4 * ncu * 64 * 10; }

hipError_t launch_bh(fmm_tree *t, int outputs, double *phi, double *field, double *grad, hipStream_t s)
{
    const bool f32 = t->prec == FMM_PREC_MIXED, h = t->basis == FMM_M2L_HARMONIC;
    bh_fn k = bh_select((outputs & FMM_GRAD) != 0, t->order, t->p, f32, h);
    if (!k) return hipErrorInvalidValue;
    BHArgs a;
    a.cells = t->d_cells;
    a.xs = t->d_x;
    a.m64 = t->d_mom;
    a.m32 = t->d_mom32;
    a.M = h ? (const void *)t->d_Mh : (f32 ? (const void *)t->d_M32 : (const void *)t->d_M64);
    a.perm = t->d_perm;
    a.phi = phi;
    a.field = field;
    a.n = (int)t->ht.n;
    a.nmp = h ? (hterms(t->p) - hterms(t->order - 1) + 3) / 4 * 4 : (nterms(t->p) - nterms(t->order - 1) + 3) / 4 * 4;
    a.outputs = outputs;
    a.theta2 = t->theta * t->theta;
    for (int d = 0; d < 3; ++d) a.g.lo[d] = t->ht.lo[d];
    a.g.h = t->ht.h;
    a.counts = t->d_bhcount;
    a.mask = t->smask;
    a.w = mask_width(t->smask);
    a.grad = grad;
    a.part = t->d_bhpart ? t->d_bhpart : t->ctx->bh_part;
    a.split = a.part ? bh_split(t->ht.n, t->ctx->ncu) : 1;
    hipLaunchKernelGGL(zero_u64_kernel, dim3(1), dim3(64), 0, s, t->d_bhcount, 2);
    hipLaunchKernelGGL(k, dim3((unsigned)((t->ht.n + 63) / 64) * a.split), dim3(64), 0, s, a);
    if (a.split > 1) {
        const int no = (outputs & FMM_GRAD) ? 10 : 4;
        hipLaunchKernelGGL(bh_reduce_kernel, dim3((unsigned)((t->ht.n * no + 255) / 256)), dim3(256), 0, s, (int)t->ht.n,
                           a.split, no, outputs, (const double *)a.part, t->d_perm, phi, field, grad);
    }
    return hipGetLastError();
}
