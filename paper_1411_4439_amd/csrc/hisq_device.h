// Device helpers shared by the HIP kernels: tile scheduling and the per-rhs
// FP64 reductions of the CG dot products.
#pragma once

#include "hisq_internal.h"

namespace hisq {

// Work-group -> tile map (a bijection on [0, nb); correctness never depends on
// it, only cache locality does).  Work-groups are dealt to the 8 XCDs of the
// chip round-robin (work-group b starts on XCD b mod 8).
//   order 0: tile = b.
//   order 1: the tiles are split into 8 contiguous ranges and XCD j walks range
//            j in order, so each XCD's L2 sees a contiguous slab of the lattice.
//   order 2: as 1, but the walk visits all Lt time slices of one position of the
//            slice before moving on (t fastest).  An input site is read by the
//            outputs at t+-1 and t+-3; in canonical order those run a whole time
//            slice apart and the site is fetched again for each, in this order
//            they run back to back and hit L2.  Needs nb = Lt * (tiles per slice).
__device__ inline int tile_of_block(int b, int nb, int order, const Lat& lat, int tile_sites)
{
    if (order == 0 || nb < 8) return b;
    const int j = b & 7, m = b >> 3;
    if (order == 3) {
        // XCD j owns the z-chunk [j*zc, (j+1)*zc) of every time slice and walks
        // it with the (y, x) plane position outermost, then t, then z, so the
        // +-1 and +-3 neighbours in every direction but the chunk's z faces
        // are read while they are still in that XCD's L2.
        const int zc = lat.L[2] >> 3, C = lat.L[0] * lat.L[1] / 2 / tile_sites;
        const int zl = m % zc, t = (m / zc) % lat.L[3], c = m / (zc * lat.L[3]);
        return ((t * lat.L[2] + j * zc + zl) * C) + c;
    }
    const int q = nb >> 3, rem = nb & 7;
    const int c = j * q + (j < rem ? j : rem) + m;  // XCD-contiguous position
    if (order == 1) return c;
    const int per_slice = nb / lat.L[3];
    return (c % lat.L[3]) * per_slice + c / lat.L[3];
}

// Lanes of a wave -> (site, rhs group, direction).  A site takes G = NRHS / NR
// rhs groups of SPL lanes each, adjacent; where that does not divide 64 the last
// lanes of every wave idle.
// (One rhs per lane for 3, 5 and 7 rhs: 7 x 8400 sites are 934 waves instead of
// the 132 that whole bundles per lane give; the 20 x 14 x 10 x 6 mixed solve takes
// 10.6 ms instead of 14.5.)
template <int NRHS, int NR, int SPL>
struct LaneMap {
    static constexpr int G = NRHS / NR;
    static constexpr int LPS = G * SPL;     // lanes per site
    static constexpr int SPW = 64 / LPS;    // sites per wave
    static constexpr bool kFull = 64 % LPS == 0;
    __device__ static __forceinline__ int lane() { return threadIdx.x & 63; }
    __device__ static __forceinline__ int group() { return lane() % LPS / SPL; }
    __device__ static __forceinline__ int dir() { return lane() % SPL; }
    __device__ static __forceinline__ bool live() { return kFull || lane() < SPW * LPS; }
    __device__ static __forceinline__ int sites(int threads) { return threads / 64 * SPW; }
    __device__ static __forceinline__ int site(int tile)
    {
        return tile * sites(blockDim.x) + (int)(threadIdx.x >> 6) * SPW + lane() / LPS;
    }
};

__device__ inline double shfl_xor_d(double v, int m) { return __shfl_xor(v, m, 64); }

// Coherent accesses for the cross-work-group reduction.  Plain stores stay in
// the L2 of the XCD that wrote them; agent-scope atomic accesses are performed
// at the device-coherent level, so a work-group on another XCD sees them.
// (No release fence is used: on this chip an agent-scope release writes back
// the whole L2, far too costly once per work-group.)
__device__ __forceinline__ void store_coherent(double* p, double v)
{
    __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ void store_coherent(uint32_t* p, uint32_t v)
{
    __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ double load_coherent(const double* p)
{
    return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ uint32_t add_coherent(uint32_t* p, uint32_t v)
{
    return __hip_atomic_fetch_add(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
// Wait until this wave's outstanding memory operations have completed, i.e.
// its coherent stores have been performed, before it signals a counter.
__device__ __forceinline__ void wait_memory() { asm volatile("s_waitcnt vmcnt(0)" ::: "memory"); }
// The reading side: once a work-group has seen from the counter that it
// arrived last, an agent-scope acquire keeps its loads of the partials after
// that observation (the compiler may not hoist them, and the vector L1 is
// invalidated, so no line cached before the counter update is reused).
__device__ __forceinline__ void acquire_agent() { __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "agent"); }

// Sum over all 64 lanes by an xor butterfly: every lane ends with the same,
// bitwise identical total (each step adds the same two values).
__device__ __forceinline__ double wave_sum(double v)
{
#pragma unroll
    for (int off = 32; off >= 1; off >>= 1) v += shfl_xor_d(v, off);
    return v;
}

// Per-rhs FP64 sums over the whole grid, in a fixed order (bitwise
// reproducible, no floating-point atomics).  Each thread contributes part[k]
// to rhs g*NR + k, where g = lane mod G is its rhs group.
//   stage 1 (sum_post): wave butterflies + LDS -> one partial per work-group
//            and rhs.  Where the grid has no more work-groups than rows, the
//            partial is the row and the kernel is done: no counter, no wait.
//   stage 2 (sum_post, sum_finish): else the last work-group of each group of
//            `group` (atomic counter) sums the group's partials into its row.
//   stage 3 (sum_rows): the kernel that needs the sum adds the rows: the p-update
//            in every wave, D_eo in the first wave of each work-group.  The end of
//            the producing kernel orders the rows before it.
// A third stage inside the producer (the last group sums the group sums) cost
// each reducing kernel 2-3 us of counter and load round trips at its end, and
// counters in one cache line another 10 ns per work-group: together 5 us of a
// 16^3 x 4 to 32^3 x 8 kernel that streams for 5-25 us.
//
// Ordering within a group.  A writer stores its partials with agent-scope
// atomic stores, waits (s_waitcnt vmcnt(0)) until the memory system has
// acknowledged them -- an agent-scope atomic store is acknowledged once it is
// visible at the device-coherent level, bypassing the XCD's non-coherent L2 --
// and only then issues its counter increment.  The last arriving work-group
// observes the final count through the returned value of its own
// read-modify-write, then executes an agent-scope acquire before it loads the
// partials with agent-scope atomic loads.  So every partial was performed at
// the coherent level before the increment that counted it, and every load of
// the reader follows its observation of that count.  The writer side uses no
// release fence: on this chip an agent-scope release writes back the XCD's
// whole L2, which one work-group per launch can afford but every work-group
// cannot; the completion wait orders exactly the stores the reader needs.
//
// sum_post returns true in wave 0 of the work-group that arrived last in its
// group, which must then call sum_finish.  A kernel may issue stores that the
// reduction does not read (its output fields) between the two calls, so that
// the completion wait before the counter update covers only the partials.
// M sums at once: part[m][k].
template <int NRHS, int NR, int M, int SPL = 1>
__device__ bool sum_post(double (&part)[M][NR], const SumOut& o, int nblk, int bid)
{
    using Map = LaneMap<NRHS, NR, SPL>;
    constexpr int NP = sum_stride(NRHS);
    __shared__ double sred[kMaxBlockLds / 64][M * kMaxRhs];
    const int lane = threadIdx.x & 63;
    const int wave = threadIdx.x >> 6;
    const int nwaves = blockDim.x >> 6;
#pragma unroll
    for (int m = 0; m < M; ++m)
#pragma unroll
        for (int k = 0; k < NR; ++k) {
            // over the directions, then over the sites of the wave
#pragma unroll
            for (int off = SPL / 2; off >= 1; off >>= 1) part[m][k] += shfl_xor_d(part[m][k], off);
            if constexpr (Map::kFull) {
#pragma unroll
                for (int off = 32; off >= Map::LPS; off >>= 1) part[m][k] += shfl_xor_d(part[m][k], off);
            } else {
                // a tree over SPW sites, any number: the total ends in site 0
#pragma unroll
                for (int rows = Map::SPW; rows > 1; rows = (rows + 1) / 2) {
                    const int off = (rows + 1) / 2;
                    const double o2 = __shfl(part[m][k], (lane + off * Map::LPS) & 63, 64);
                    if (lane / Map::LPS + off < rows) part[m][k] += o2;
                }
            }
        }
    if (lane < Map::LPS && lane % SPL == 0) {
        const int g = lane / SPL;
#pragma unroll
        for (int m = 0; m < M; ++m)
#pragma unroll
            for (int k = 0; k < NR; ++k) sred[wave][m * NP + g * NR + k] = part[m][k];
    }
    __syncthreads();
    if (wave != 0) return false;
    double s = 0;
    const int k = lane % NP, m = lane / NP;
    if (k < NRHS && m < M)
        for (int w = 0; w < nwaves; ++w) s += sred[w][lane];
    if (o.group == 1) {
        if (m < M) o.rows[m * kSumDoubles + (size_t)bid * NP + k] = s;
        return false;
    }
    if (m < M) store_coherent(&o.part[(size_t)bid * (M * NP) + lane], s);
    wait_memory();
    const int grp = bid / o.group;
    const int gn = min(o.group, nblk - grp * o.group);
    uint32_t prev = 0;
    if (lane == 0) prev = add_coherent(&o.cnt[counter_index(grp)], 1u);
    prev = __shfl(prev, 0, 64);
    return prev == (uint32_t)(gn - 1);
}

// Stage 2, in wave 0 of a work-group for which sum_post returned true.
template <int NRHS, int M>
__device__ void sum_finish(const SumOut& o, int nblk, int bid)
{
    constexpr int NV = M * sum_stride(NRHS);
    constexpr int RL = 64 / NV;  // rows per pass: lane = (row, sum, rhs)
    const int lane = threadIdx.x & 63;
    const int grp = bid / o.group;
    const int g0 = grp * o.group;
    const int gn = min(o.group, nblk - g0);
    acquire_agent();
    double v = 0;
    for (int r0 = lane / NV; r0 < gn; r0 += 8 * RL) {
        double x[8];
#pragma unroll
        for (int j = 0; j < 8; ++j) {  // all loads in flight
            const int r = r0 + j * RL;
            x[j] = r < gn ? load_coherent(&o.part[(size_t)(g0 + r) * NV + lane % NV]) : 0.0;
        }
#pragma unroll
        for (int j = 0; j < 8; ++j) v += x[j];
    }
#pragma unroll
    for (int off = 32; off >= NV; off >>= 1) v += shfl_xor_d(v, off);
    constexpr int NP = sum_stride(NRHS);
    if (lane < NV) o.rows[lane / NP * kSumDoubles + (size_t)grp * NP + lane % NP] = v;
    if (lane == 0) store_coherent(&o.cnt[counter_index(grp)], 0u);
}

// Stage 3, in any wave with all lanes active: the total of rhs (lane mod
// sum_stride(NRHS)), the same bits in every wave.
template <int NRHS>
__device__ __forceinline__ double sum_rows(const SumIn& in)
{
    constexpr int NP = sum_stride(NRHS);
    constexpr int RL = 64 / NP;
    const int lane = threadIdx.x & 63;
    double x[8];
#pragma unroll
    for (int j = 0; j < 8; ++j) {
        const int r = lane / NP + j * RL;
        x[j] = r < in.n ? in.rows[(size_t)r * NP + lane % NP] : 0.0;
    }
    double v = 0;
#pragma unroll
    for (int j = 0; j < 8; ++j) v += x[j];
#pragma unroll
    for (int off = 32; off >= NP; off >>= 1) v += shfl_xor_d(v, off);
    return v;
}

__device__ inline bool finite_d(double v) { return v - v == 0.0; }

// The scalars of rhs k = lane mod sum_stride(NRHS) at the start of an iteration:
// those of src, advanced by the |r|^2 that the previous iteration left (unless
// fresh: a poll block starts from what the host decided).  The wave that is the
// launch's writer stores them to dst.  Every lane must be active.
template <int NRHS>
__device__ __forceinline__ void cg_scalars(const CgState* src, CgState* dst, const SumIn& rows, int fresh,
                                           bool writer, bool& act, double& beta)
{
    constexpr int NP = sum_stride(NRHS);
    const int lane = threadIdx.x & 63, k = lane % NP;
    act = src->active[k] != 0;
    beta = src->beta[k];
    double rr = src->rr[k], rrmax = src->rrmax[k];
    int iters = src->iters[k], status = src->status[k];
    const double thresh = src->thresh[k];
    if (!fresh) {
        const double tot = sum_rows<NRHS>(rows);
        if (act) {
            if (src->brk[k]) {  // <p, A p> failed: x and r were not updated
                status = HISQ_BREAKDOWN;
                act = false;
            } else {
                iters += 1;
                if (!finite_d(tot)) {
                    status = HISQ_BREAKDOWN;
                    act = false;
                } else {
                    beta = tot / rr;
                    rr = tot;
                    if (tot > rrmax) rrmax = tot;
                    if (tot <= thresh || iters >= src->maxiter) act = false;
                }
            }
        }
    }
    if (writer && lane < NP) {
        dst->rr[k] = rr;
        dst->beta[k] = beta;
        dst->thresh[k] = thresh;
        dst->rrmax[k] = rrmax;
        dst->active[k] = act;
        dst->status[k] = status;
        dst->iters[k] = iters;
        dst->brk[k] = 0;
        if (lane == 0) {
            dst->maxiter = src->maxiter;
            dst->frozen = 0;
        }
    }
}

// Spinor field layouts, element (site i, colour c, rhs k) of an n-rhs field:
//   site-major   [Vh][3][n]  (CM = false, the canonical layout at the boundary)
//   colour-major [3][Vh][n]  (CM = true, the solver's internal layout)
// Both keep the rhs of a site innermost.  In colour-major order the lanes of a
// wave, which own consecutive sites, read one contiguous stretch per colour;
// in site-major order they stride by 3n complex numbers, and every load
// instruction touches about three times as many cache lines.
template <int NRHS, bool CM>
struct Layout {
    __device__ static __forceinline__ int site(int i) { return CM ? i * NRHS : i * 3 * NRHS; }
    __device__ static __forceinline__ int colour(int c, int Vh) { return CM ? c * Vh * NRHS : c * NRHS; }
};

// Loads and stores of NR consecutive complex numbers (rhs of one colour).
// NT: streamed data, read or written once per launch; the non-temporal hint
// keeps it from evicting the gathered neighbour field from L2.
template <bool NT, typename V>
__device__ __forceinline__ V ld(const V* p)
{
    if constexpr (NT) return __builtin_nontemporal_load(p);
    else return *p;
}

template <bool NT, typename V>
__device__ __forceinline__ void st(V* p, V v)
{
    if constexpr (NT) __builtin_nontemporal_store(v, p);
    else *p = v;
}

template <int NR, bool NT = false>
__device__ __forceinline__ void load_rhs(const f2* __restrict__ p, f2 (&v)[NR])
{
    if constexpr (NR % 2 == 0) {
        const f4* q = reinterpret_cast<const f4*>(p);
#pragma unroll
        for (int k = 0; k < NR / 2; ++k) {
            f4 w = ld<NT>(q + k);
            v[2 * k] = f2{w.x, w.y};
            v[2 * k + 1] = f2{w.z, w.w};
        }
    } else {
#pragma unroll
        for (int k = 0; k < NR; ++k) v[k] = ld<NT>(p + k);
    }
}

template <int NR, bool NT = false>
__device__ __forceinline__ void load_rhs(const d2* __restrict__ p, d2 (&v)[NR])
{
#pragma unroll
    for (int k = 0; k < NR; ++k) v[k] = ld<NT>(p + k);
}

template <int NR, bool NT = false>
__device__ __forceinline__ void store_rhs(f2* __restrict__ p, const f2 (&v)[NR])
{
    if constexpr (NR % 2 == 0) {
        f4* q = reinterpret_cast<f4*>(p);
#pragma unroll
        for (int k = 0; k < NR / 2; ++k)
            st<NT>(q + k, f4{v[2 * k].x, v[2 * k].y, v[2 * k + 1].x, v[2 * k + 1].y});
    } else {
#pragma unroll
        for (int k = 0; k < NR; ++k) st<NT>(p + k, v[k]);
    }
}

template <int NR, bool NT = false>
__device__ __forceinline__ void store_rhs(d2* __restrict__ p, const d2 (&v)[NR])
{
#pragma unroll
    for (int k = 0; k < NR; ++k) st<NT>(p + k, v[k]);
}

// Masked stores for the CG updates: rhs k is written only if on[k] (converged
// rhs keep their values untouched in memory); a 16-byte FP32 pair with one rhs
// on stores that rhs alone.
template <int NR>
__device__ __forceinline__ void store_rhs_on(f2* __restrict__ p, const f2 (&v)[NR], const bool (&on)[NR])
{
    if constexpr (NR % 2 == 0) {
        f4* q = reinterpret_cast<f4*>(p);
#pragma unroll
        for (int k = 0; k < NR / 2; ++k) {
            if (on[2 * k] && on[2 * k + 1])
                q[k] = f4{v[2 * k].x, v[2 * k].y, v[2 * k + 1].x, v[2 * k + 1].y};
            else if (on[2 * k])
                p[2 * k] = v[2 * k];
            else if (on[2 * k + 1])
                p[2 * k + 1] = v[2 * k + 1];
        }
    } else {
#pragma unroll
        for (int k = 0; k < NR; ++k)
            if (on[k]) p[k] = v[k];
    }
}

template <int NR>
__device__ __forceinline__ void store_rhs_on(d2* __restrict__ p, const d2 (&v)[NR], const bool (&on)[NR])
{
#pragma unroll
    for (int k = 0; k < NR; ++k)
        if (on[k]) p[k] = v[k];
}

}  // namespace hisq
