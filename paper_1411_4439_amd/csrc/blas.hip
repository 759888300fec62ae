// CG vector kernels for gfx950: the masked p-update,
// precision conversions for the reliable updates, and FP64 reductions.
#include "hisq_device.h"

namespace hisq {

// ---------------------------------------------------------------------------
// p = r + beta_k p for every active rhs k.  A stream of three field passes with
// no reduction (|p|^2 is summed by D_oe, which reads p anyway): the field is
// walked as a flat array of 16-byte chunks with a stride that is a multiple of
// the rhs period, so every thread always touches the same rhs while each load
// instruction covers a contiguous stretch of memory.  The first chunks are
// requested before the scalars of the iteration are worked out.
template <typename T, int NRHS>
__device__ __forceinline__ void pupdate_flat(const PupdateArgs<T>& a, const CgState* src, CgState* dst,
                                             int fresh, int nblk, int bid)
{
    using C = cplx<T>;
    constexpr int NV = 16 / sizeof(C);  // complex numbers per chunk
    constexpr int U = 2;                // chunks in flight
    const int nchunks = (int)((long)a.lat.Vh * 3 * NRHS / NV);
    const int tid = bid * (int)blockDim.x + (int)threadIdx.x;
    const int stride = nblk * (int)blockDim.x;  // times NV a multiple of NRHS
    C rv[U][NV], pv[U][NV];
    auto fetch = [&](int j) {
#pragma unroll
        for (int u = 0; u < U; ++u)
            if (j + u * stride < nchunks) {
                load_rhs<NV>(a.r + (size_t)(j + u * stride) * NV, rv[u]);
                load_rhs<NV>(a.p + (size_t)(j + u * stride) * NV, pv[u]);
            }
    };
    fetch(tid);
    bool on;
    double b;
    cg_scalars<NRHS>(src, dst, a.rr, fresh, bid == 0 && threadIdx.x < 64, on, b);
    if (!__any(on)) return;  // every rhs converged: nothing to do
    bool act[NV], any_act = false;
    T beta[NV];
#pragma unroll
    for (int v = 0; v < NV; ++v) {
        const int k = (int)((long)tid * NV + v) % NRHS;
        act[v] = __shfl((int)on, k, 64) != 0;
        beta[v] = __shfl((T)b, k, 64);
        any_act = any_act || act[v];
    }
    if (!any_act) return;
    for (int j = tid; j < nchunks; j += U * stride) {
        if (j != tid) fetch(j);
#pragma unroll
        for (int u = 0; u < U; ++u)
            if (j + u * stride < nchunks) {
#pragma unroll
                for (int v = 0; v < NV; ++v)
                    // beta = 0 starts (or restarts) the recursion: p = r exactly,
                    // even if p held non-finite values
                    pv[u][v] = beta[v] == T(0) ? rv[u][v]
                                               : C{rv[u][v].x + beta[v] * pv[u][v].x,
                                                   rv[u][v].y + beta[v] * pv[u][v].y};
                // converged rhs are not written
                store_rhs_on<NV>(a.p + (size_t)(j + u * stride) * NV, pv[u], act);
            }
    }
}

template <typename T, int NRHS>
__global__ __launch_bounds__(kMaxBlock) void k_pupdate(const PupdateArgs<T> a)
{
    pupdate_flat<T, NRHS>(a, a.src, a.dst, a.fresh, gridDim.x, blockIdx.x);
}

// One launch over the problems of a batch: each has its own range of work-groups.
template <typename T>
__global__ __launch_bounds__(kMaxBlock) void k_pupdate_batched(const BatchTable<T>* __restrict__ tab, int phase)
{
    int q = 0;
    for (int j = 1; j < tab->nprob; ++j)
        if ((int)blockIdx.x >= tab->p[j].pup_start) q = j;
    const BatchProb<T>& bp = tab->p[q];
    const int bid = (int)blockIdx.x - bp.pup_start;
    const int nb = bp.pup_blocks;
    if (bid >= nb) return;
    const CgState* src = bp.state[state_of_phase(phase, 0)];
    CgState* dst = bp.state[state_of_phase(phase, 1)];
    const int fresh = phase == 0;
    // a problem that has ended within the poll block reads no field (its first
    // work-group still passes the scalars on)
    bool any = bid == 0;
    for (int k = 0; k < bp.n; ++k) any = any || src->active[k] != 0;
    if (!any) return;
    switch (bp.n) {
    case 1: pupdate_flat<T, 1>(bp.k1, src, dst, fresh, nb, bid); break;
    case 2: pupdate_flat<T, 2>(bp.k1, src, dst, fresh, nb, bid); break;
    case 3: pupdate_flat<T, 3>(bp.k1, src, dst, fresh, nb, bid); break;
    case 4: pupdate_flat<T, 4>(bp.k1, src, dst, fresh, nb, bid); break;
    case 5: pupdate_flat<T, 5>(bp.k1, src, dst, fresh, nb, bid); break;
    case 6: pupdate_flat<T, 6>(bp.k1, src, dst, fresh, nb, bid); break;
    case 7: pupdate_flat<T, 7>(bp.k1, src, dst, fresh, nb, bid); break;
    case 8: pupdate_flat<T, 8>(bp.k1, src, dst, fresh, nb, bid); break;
    default: break;
    }
}

constexpr int kPupBlock = 256, kPupMaxBlocks = 2048;

// Enough work-groups for one pass, at most 8 per CU, a multiple of the rhs period.
int pupdate_blocks(int nrhs, int Vh, size_t elem)
{
    const long nchunks = (long)Vh * 3 * nrhs * 2 * (long)elem / 16;
    long blocks = (nchunks + kPupBlock - 1) / kPupBlock;
    if (blocks > kPupMaxBlocks) blocks = kPupMaxBlocks;
    return (int)((blocks + nrhs - 1) / nrhs * nrhs);
}

template <typename T>
static hipError_t launch_pupdate(int nrhs, const PupdateArgs<T>& a, hipStream_t s)
{
    const dim3 grid(pupdate_blocks(nrhs, a.lat.Vh, sizeof(T))), block(kPupBlock);
    switch (nrhs) {
    case 1: hipLaunchKernelGGL((k_pupdate<T, 1>), grid, block, 0, s, a); break;
    case 2: hipLaunchKernelGGL((k_pupdate<T, 2>), grid, block, 0, s, a); break;
    case 3: hipLaunchKernelGGL((k_pupdate<T, 3>), grid, block, 0, s, a); break;
    case 4: hipLaunchKernelGGL((k_pupdate<T, 4>), grid, block, 0, s, a); break;
    case 5: hipLaunchKernelGGL((k_pupdate<T, 5>), grid, block, 0, s, a); break;
    case 6: hipLaunchKernelGGL((k_pupdate<T, 6>), grid, block, 0, s, a); break;
    case 7: hipLaunchKernelGGL((k_pupdate<T, 7>), grid, block, 0, s, a); break;
    case 8: hipLaunchKernelGGL((k_pupdate<T, 8>), grid, block, 0, s, a); break;
    default: return hipErrorInvalidValue;
    }
    return hipGetLastError();
}

hipError_t launch_pupdate_f64(int nrhs, const PupdateArgs<double>& a, hipStream_t s)
{
    return launch_pupdate<double>(nrhs, a, s);
}

hipError_t launch_pupdate_f32(int nrhs, const PupdateArgs<float>& a, hipStream_t s)
{
    return launch_pupdate<float>(nrhs, a, s);
}

hipError_t launch_pupdate_batched_f64(const BatchTable<double>* tab, int total_blocks, int phase,
                                      hipStream_t s)
{
    hipLaunchKernelGGL(k_pupdate_batched<double>, dim3(total_blocks), dim3(kPupBlock), 0, s, tab, phase);
    return hipGetLastError();
}

hipError_t launch_pupdate_batched_f32(const BatchTable<float>* tab, int total_blocks, int phase,
                                      hipStream_t s)
{
    hipLaunchKernelGGL(k_pupdate_batched<float>, dim3(total_blocks), dim3(kPupBlock), 0, s, tab, phase);
    return hipGetLastError();
}

// ---------------------------------------------------------------------------
// Elementwise kernels over complex arrays [Vh][3][n] (rhs index = element mod n).

static inline int blocks_for(size_t n, int bs)
{
    size_t b = (n + bs - 1) / bs;
    return (int)(b > 65535u * 16u ? 65535u * 16u : b);
}

__global__ void k_zero(uint32_t* p, size_t words)
{
    for (size_t e = blockIdx.x * (size_t)blockDim.x + threadIdx.x; e < words;
         e += (size_t)gridDim.x * blockDim.x)
        p[e] = 0u;
}

hipError_t launch_zero(void* p, size_t bytes, hipStream_t s)
{
    if (bytes == 0) return hipSuccess;
    const size_t words = bytes / 4;  // every workspace region is 256-byte aligned
    hipLaunchKernelGGL(k_zero, dim3(blocks_for(words, 256)), dim3(256), 0, s, (uint32_t*)p, words);
    return hipGetLastError();
}

__global__ void k_state_reset(CgState* st, int nrhs, int active)
{
    if (threadIdx.x == 0) {
        *st = CgState{};
        for (int k = 0; k < nrhs; ++k) {
            st->sel[k] = 1;
            st->active[k] = active;
        }
        st->frozen = active;  // armed for timing: the kernels run, the state stays put
    }
}

hipError_t launch_state_reset(CgState* st, int nrhs, int active, hipStream_t s)
{
    hipLaunchKernelGGL(k_state_reset, dim3(1), dim3(64), 0, s, st, nrhs, active);
    return hipGetLastError();
}

// One wave per problem: the end of a poll block.
template <int NP>
__device__ __forceinline__ void fold_one(const FoldArgs::One& f)
{
    bool act;
    double beta;
    cg_scalars<NP>(f.src, f.dst, f.rr, 0, true, act, beta);
}

__global__ void k_fold(FoldArgs a)
{
    const FoldArgs::One& f = a.p[blockIdx.x];
    switch (sum_stride(f.nrhs)) {
    case 1: fold_one<1>(f); break;
    case 2: fold_one<2>(f); break;
    case 4: fold_one<4>(f); break;
    default: fold_one<8>(f); break;
    }
}

hipError_t launch_fold(const FoldArgs& a, int nprob, hipStream_t s)
{
    hipLaunchKernelGGL(k_fold, dim3(nprob), dim3(64), 0, s, a);
    return hipGetLastError();
}

template <int NP>
__global__ void k_sum_final(SumIn in, int nrhs, double scale, double* out)
{
    const double t = sum_rows<NP>(in);
    if ((int)threadIdx.x < nrhs) out[threadIdx.x] = scale * t;
}

hipError_t launch_sum_final(SumIn in, int nrhs, double scale, double* out, hipStream_t s)
{
    switch (sum_stride(nrhs)) {
    case 1: hipLaunchKernelGGL(k_sum_final<1>, dim3(1), dim3(64), 0, s, in, nrhs, scale, out); break;
    case 2: hipLaunchKernelGGL(k_sum_final<2>, dim3(1), dim3(64), 0, s, in, nrhs, scale, out); break;
    case 4: hipLaunchKernelGGL(k_sum_final<4>, dim3(1), dim3(64), 0, s, in, nrhs, scale, out); break;
    default: hipLaunchKernelGGL(k_sum_final<8>, dim3(1), dim3(64), 0, s, in, nrhs, scale, out); break;
    }
    return hipGetLastError();
}

__global__ void k_to_f32_sel(const d2* __restrict__ src, f2* __restrict__ dst, size_t ncplx,
                             int nrhs, const CgState* st)
{
    for (size_t e = blockIdx.x * (size_t)blockDim.x + threadIdx.x; e < ncplx;
         e += (size_t)gridDim.x * blockDim.x) {
        if (st->sel[e % nrhs]) {
            const d2 v = src[e];
            dst[e] = f2{(float)v.x, (float)v.y};
        }
    }
}

hipError_t launch_to_f32_sel(const d2* src, f2* dst, size_t ncplx, int nrhs, const CgState* st,
                             hipStream_t s)
{
    hipLaunchKernelGGL(k_to_f32_sel, dim3(blocks_for(ncplx, 256)), dim3(256), 0, s, src, dst, ncplx,
                       nrhs, st);
    return hipGetLastError();
}

// x_hi += x_lo; x_lo = 0 for the selected rhs (solution accumulation of a
// reliable update).
__global__ void k_accum_sel(d2* __restrict__ xh, f2* __restrict__ xl, size_t ncplx, int nrhs,
                            const CgState* st)
{
    for (size_t e = blockIdx.x * (size_t)blockDim.x + threadIdx.x; e < ncplx;
         e += (size_t)gridDim.x * blockDim.x) {
        if (st->sel[e % nrhs]) {
            const f2 l = xl[e];
            d2 h = xh[e];
            h.x += (double)l.x;
            h.y += (double)l.y;
            xh[e] = h;
            xl[e] = f2{0.0f, 0.0f};
        }
    }
}

hipError_t launch_accum_sel(d2* xh, f2* xl, size_t ncplx, int nrhs, const CgState* st,
                            hipStream_t s)
{
    hipLaunchKernelGGL(k_accum_sel, dim3(blocks_for(ncplx, 256)), dim3(256), 0, s, xh, xl, ncplx,
                       nrhs, st);
    return hipGetLastError();
}

__global__ void k_copy_f64(const d2* __restrict__ src, d2* __restrict__ dst, size_t ncplx)
{
    for (size_t e = blockIdx.x * (size_t)blockDim.x + threadIdx.x; e < ncplx;
         e += (size_t)gridDim.x * blockDim.x)
        dst[e] = src[e];
}

hipError_t launch_copy_f64(const d2* src, d2* dst, size_t ncplx, hipStream_t s)
{
    hipLaunchKernelGGL(k_copy_f64, dim3(blocks_for(ncplx, 256)), dim3(256), 0, s, src, dst, ncplx);
    return hipGetLastError();
}

__global__ void k_zero_sel(d2* __restrict__ v, size_t ncplx, int nrhs, const CgState* st)
{
    for (size_t e = blockIdx.x * (size_t)blockDim.x + threadIdx.x; e < ncplx;
         e += (size_t)gridDim.x * blockDim.x)
        if (st->sel[e % nrhs]) v[e] = d2{0.0, 0.0};
}

hipError_t launch_zero_sel(d2* v, size_t ncplx, int nrhs, const CgState* st, hipStream_t s)
{
    hipLaunchKernelGGL(k_zero_sel, dim3(blocks_for(ncplx, 256)), dim3(256), 0, s, v, ncplx, nrhs, st);
    return hipGetLastError();
}

// ---------------------------------------------------------------------------
// Layout conversions between the canonical site-major field [Vh][3][n] and the
// solver's colour-major field [3][Vh][n] (FP64).
__global__ void k_to_colour_major(const d2* __restrict__ src, d2* __restrict__ dst, int Vh, int nrhs)
{
    const size_t total = (size_t)Vh * 3 * nrhs;
    for (size_t e = blockIdx.x * (size_t)blockDim.x + threadIdx.x; e < total;
         e += (size_t)gridDim.x * blockDim.x) {
        const size_t k = e % nrhs, rest = e / nrhs;  // dst index = (c * Vh + i) * n + k
        const size_t i = rest % Vh, c = rest / Vh;
        dst[e] = src[(i * 3 + c) * nrhs + k];
    }
}

__global__ void k_to_site_major(const d2* __restrict__ src, d2* __restrict__ dst, int Vh, int nrhs)
{
    const size_t total = (size_t)Vh * 3 * nrhs;
    for (size_t e = blockIdx.x * (size_t)blockDim.x + threadIdx.x; e < total;
         e += (size_t)gridDim.x * blockDim.x) {
        const size_t k = e % nrhs, rest = e / nrhs;  // dst index = (i * 3 + c) * n + k
        const size_t c = rest % 3, i = rest / 3;
        dst[e] = src[(c * Vh + i) * nrhs + k];
    }
}

hipError_t launch_layout(const d2* src, d2* dst, int Vh, int nrhs, bool to_colour_major, hipStream_t s)
{
    const size_t total = (size_t)Vh * 3 * nrhs;
    if (to_colour_major)
        hipLaunchKernelGGL(k_to_colour_major, dim3(blocks_for(total, 256)), dim3(256), 0, s, src, dst, Vh, nrhs);
    else
        hipLaunchKernelGGL(k_to_site_major, dim3(blocks_for(total, 256)), dim3(256), 0, s, src, dst, Vh, nrhs);
    return hipGetLastError();
}

// ---------------------------------------------------------------------------
// Per-rhs |v_k|^2 of an FP64 colour-major half field, one thread per site.
template <int NRHS>
__global__ __launch_bounds__(kMaxBlock) void k_norm2(const d2* __restrict__ v, int Vh, SumOut o)
{
    double part[1][NRHS];
#pragma unroll
    for (int k = 0; k < NRHS; ++k) part[0][k] = 0.0;
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i < Vh) {
#pragma unroll
        for (int c = 0; c < 3; ++c)
#pragma unroll
            for (int k = 0; k < NRHS; ++k) {
                const d2 e = v[((size_t)c * Vh + i) * NRHS + k];
                part[0][k] += e.x * e.x + e.y * e.y;
            }
    }
    if (sum_post<NRHS, NRHS, 1>(part, o, gridDim.x, blockIdx.x))
        sum_finish<NRHS, 1>(o, gridDim.x, blockIdx.x);
}

hipError_t launch_norm2_f64(const d2* v, int Vh, int nrhs, double* out, SumOut o, hipStream_t s)
{
    const int bs = 256, grid = (Vh + bs - 1) / bs;
    o.group = sum_group(grid, nrhs);
    switch (nrhs) {
#define HISQ_NORM_CASE(N)                                                                   \
    case N:                                                                                 \
        hipLaunchKernelGGL(k_norm2<N>, dim3(grid), dim3(bs), 0, s, v, Vh, o);             \
        break;
        HISQ_NORM_CASE(1)
        HISQ_NORM_CASE(2)
        HISQ_NORM_CASE(3)
        HISQ_NORM_CASE(4)
        HISQ_NORM_CASE(5)
        HISQ_NORM_CASE(6)
        HISQ_NORM_CASE(7)
        HISQ_NORM_CASE(8)
#undef HISQ_NORM_CASE
    default: return hipErrorInvalidValue;
    }
    const hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    return launch_sum_final(SumIn{o.rows, sum_row_count(grid, nrhs)}, nrhs, 1.0, out, s);
}

// out = scale * sum over sites, colours and rhs of Re(conj(y) x).
__global__ __launch_bounds__(kMaxBlock) void k_redot(const d2* __restrict__ y,
                                                     const d2* __restrict__ x, int Vh, int nrhs,
                                                     SumOut o)
{
    double part[1][1] = {{0.0}};
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i < Vh) {
        for (int e = 0; e < 3 * nrhs; ++e) {
            const d2 a = y[(size_t)i * 3 * nrhs + e];
            const d2 b = x[(size_t)i * 3 * nrhs + e];
            part[0][0] += a.x * b.x + a.y * b.y;
        }
    }
    if (sum_post<1, 1, 1>(part, o, gridDim.x, blockIdx.x)) sum_finish<1, 1>(o, gridDim.x, blockIdx.x);
}

hipError_t launch_redot(const d2* y, const d2* x, int Vh, int nrhs, double scale, double* out,
                        SumOut o, hipStream_t s)
{
    const int bs = 256, grid = (Vh + bs - 1) / bs;
    o.group = sum_group(grid, 1);
    hipLaunchKernelGGL(k_redot, dim3(grid), dim3(bs), 0, s, y, x, Vh, nrhs, o);
    const hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    return launch_sum_final(SumIn{o.rows, sum_row_count(grid, 1)}, 1, scale, out, s);
}

// ---------------------------------------------------------------------------
// out = alpha a + beta b over n complex numbers (real scalars).
__global__ void k_axpby(const d2* __restrict__ a, const d2* __restrict__ b, d2* __restrict__ out,
                        size_t n, double alpha, double beta)
{
    for (size_t e = blockIdx.x * (size_t)blockDim.x + threadIdx.x; e < n;
         e += (size_t)gridDim.x * blockDim.x) {
        const d2 x = a[e], y = b[e];
        out[e] = d2{alpha * x.x + beta * y.x, alpha * x.y + beta * y.y};
    }
}

hipError_t launch_axpby(const d2* a, const d2* b, d2* out, size_t n, double alpha, double beta,
                        hipStream_t s)
{
    hipLaunchKernelGGL(k_axpby, dim3(blocks_for(n, 256)), dim3(256), 0, s, a, b, out, n, alpha, beta);
    return hipGetLastError();
}

// Per-rhs complex dot products sum_i conj(a_i) b_i over an even and an odd half
// field (site-major, n rhs), in a fixed order: stage 1 writes one partial per
// work-group and rhs (re, im), stage 2 sums the partials in work-group order.
template <int NRHS>
__global__ __launch_bounds__(256) void k_cdot_partial(const d2* __restrict__ ae, const d2* __restrict__ be,
                                                      const d2* __restrict__ ao, const d2* __restrict__ bo,
                                                      int Vh, double* __restrict__ part)
{
    __shared__ double sh[4][2 * NRHS];
    double re[NRHS], im[NRHS];
#pragma unroll
    for (int k = 0; k < NRHS; ++k) re[k] = im[k] = 0.0;
    const int j = blockIdx.x * blockDim.x + threadIdx.x;
    if (j < 2 * Vh) {
        const bool even = j < Vh;
        const size_t i = even ? j : j - Vh;
        const d2* a = even ? ae : ao;
        const d2* b = even ? be : bo;
#pragma unroll
        for (int c = 0; c < 3; ++c)
#pragma unroll
            for (int k = 0; k < NRHS; ++k) {
                const d2 x = a[(i * 3 + c) * NRHS + k], y = b[(i * 3 + c) * NRHS + k];
                re[k] += x.x * y.x + x.y * y.y;
                im[k] += x.x * y.y - x.y * y.x;
            }
    }
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
#pragma unroll
    for (int k = 0; k < NRHS; ++k) {
        re[k] = wave_sum(re[k]);
        im[k] = wave_sum(im[k]);
    }
    if (lane == 0) {
#pragma unroll
        for (int k = 0; k < NRHS; ++k) {
            sh[wave][2 * k] = re[k];
            sh[wave][2 * k + 1] = im[k];
        }
    }
    __syncthreads();
    if (threadIdx.x < 2 * NRHS) {
        double t = 0.0;
        for (int w = 0; w < (int)(blockDim.x >> 6); ++w) t += sh[w][threadIdx.x];
        part[(size_t)blockIdx.x * 2 * NRHS + threadIdx.x] = t;
    }
}

__global__ void k_cdot_final(const double* __restrict__ part, int nblk, int m2, double* __restrict__ out)
{
    const int k = threadIdx.x;
    if (k >= m2) return;
    double t = 0.0;
    for (int b = 0; b < nblk; ++b) t += part[(size_t)b * m2 + k];
    out[k] = t;
}

size_t cdot_scratch_doubles(int Vh, int nrhs) { return (size_t)((2 * Vh + 255) / 256) * 2 * nrhs; }

hipError_t launch_cdot(const d2* ae, const d2* be, const d2* ao, const d2* bo, int Vh, int nrhs,
                       double* scratch, double* out, hipStream_t s)
{
    const int nblk = (2 * Vh + 255) / 256;
    switch (nrhs) {
#define HISQ_CDOT_CASE(N)                                                                      \
    case N:                                                                                    \
        hipLaunchKernelGGL(k_cdot_partial<N>, dim3(nblk), dim3(256), 0, s, ae, be, ao, bo, Vh, \
                           scratch);                                                           \
        break;
        HISQ_CDOT_CASE(1)
        HISQ_CDOT_CASE(2)
        HISQ_CDOT_CASE(3)
        HISQ_CDOT_CASE(4)
        HISQ_CDOT_CASE(5)
        HISQ_CDOT_CASE(6)
        HISQ_CDOT_CASE(7)
        HISQ_CDOT_CASE(8)
#undef HISQ_CDOT_CASE
    default: return hipErrorInvalidValue;
    }
    hipLaunchKernelGGL(k_cdot_final, dim3(1), dim3(64), 0, s, scratch, nblk, 2 * nrhs, out);
    return hipGetLastError();
}

}  // namespace hisq
