// Internal declarations shared by the HIP kernels and the host driver of libhisq.
//
// Data layout in HBM (all sizes in complex elements of the storage precision):
//
//  * Spinor fields: [Vh][3][n], rhs innermost, one parity.  A thread that owns
//    `NR` rhs of a site reads NR contiguous complex numbers per colour.
//
//  * Packed links: a 256-byte header, then one block per OUTPUT parity P.  The
//    block of parity P holds, for every site z of parity P (index i = s/2), the
//    sixteen matrices that the Dslash of Sec. 1 eq. (3) applies at z:
//        slot  0..3   U_{z,mu}                    (forward one-hop)
//        slot  4..7  -U^dag_{z-mu,mu}              (backward one-hop)
//        slot  8..11  N_{z,mu}                    (forward three-hop, Naik)
//        slot 12..15 -N^dag_{z-3mu,mu}             (backward three-hop)
//    so that w_z = sum_slot W_slot v_{neighbour(slot)}, and every half-Dslash
//    streams exactly one block (each link once, as eq. (3) needs), perfectly
//    coalesced: slot-major, then matrix element, then site ([slot][elem][Vh]).
//    Each link is therefore stored twice (once per parity block) -- memory is
//    traded for contiguous reads, the byte count per half-Dslash is unchanged.
//    Naik slots in r14 storage keep 7 complex: rows 0 and 1 and c, with
//    row2 = c * conj(row0 x row1)  (14 reals, Table 1 "r14").
#pragma once

#include <hip/hip_runtime.h>

#include <cstddef>
#include <cstdint>

#include "hisq.h"

namespace hisq {

typedef float f2 __attribute__((ext_vector_type(2)));
typedef float f4 __attribute__((ext_vector_type(4)));
typedef double d2 __attribute__((ext_vector_type(2)));

template <typename T>
struct CplxOf;
template <>
struct CplxOf<float> {
    using type = f2;
};
template <>
struct CplxOf<double> {
    using type = d2;
};
template <typename T>
using cplx = typename CplxOf<T>::type;

constexpr int kMaxRhs = HISQ_MAX_RHS;
constexpr size_t kLinkHeaderBytes = 256;
constexpr uint32_t kLinkMagic = 0x51534948u;  // "HISQ"
constexpr int kMaxBlock = 256;
// LDS-staged Dslash: up to 512 threads per work-group, up to 64 KB of staged
// neighbour rows.
constexpr int kMaxBlockLds = 512;
constexpr int kMaxStageBytes = 64 * 1024;
// r14 / r13: bound on the relative error of the FP64 fit row2 = c conj(row0 x row1)
// (before rounding to FP32); exact fits of s*U(3) links stay near 1e-15
constexpr float kNaikTolerance = 1e-10f;
constexpr float kR9Tolerance = 4e-6f;    // r9: bounded by the FP32 rounding of H
constexpr float kR9ScaleSpread = 1e-6f;  // r9: relative spread of the Naik scales

struct LinkHeader {
    uint32_t magic;
    int32_t L[4];
    int32_t prec;
    int32_t naik;
    uint32_t naik_err_bits;  // r14 / r13 / r9: max relative round-trip error, float bits (atomicMax)
    uint32_t scale_min_bits;  // r9: smallest and largest Naik scale |det N|^(1/3), float bits
    uint32_t scale_max_bits;
    float naik_scale;         // r9: the scale the kernels apply (set after packing)
};

// Lattice description as the kernels see it.
struct Lat {
    int32_t L[4];
    int32_t Lh0;  // L0 / 2
    int32_t Vh;   // sites per parity
    int32_t sy, sz, st;  // index strides of x1, x2, x3 within a parity
};

inline Lat make_lat(const hisq_geom& g)
{
    Lat l;
    for (int mu = 0; mu < 4; ++mu) l.L[mu] = g.L[mu];
    l.Lh0 = g.L[0] / 2;
    l.sy = l.Lh0;
    l.sz = l.Lh0 * g.L[1];
    l.st = l.sz * g.L[2];
    l.Vh = l.st * g.L[3];
    return l;
}

// Packed link block of one output parity: 16 slots (U fwd, -U^dag bwd, N fwd,
// -N^dag bwd per direction), each one matrix per site.  Sizes in reals (float or
// double).  U slots hold 18 reals; a Naik slot holds 18 (FULL), 14 (R14: rows 0
// and 1 and one complex c with row2 = c conj(row0 x row1)) or 13 (R13: rows 0
// and 1 and the phase phi of c = exp(i phi) / |row0|) or 9 (R9: Hermitian H,
// N = s exp(iH) with s in the header).  R14, R13 and R9 are FP32.
__host__ __device__ constexpr int naik_reals(int nk)
{
    return nk == HISQ_NAIK_R14 ? 14 : nk == HISQ_NAIK_R13 ? 13 : nk == HISQ_NAIK_R9 ? 9 : 18;
}

__host__ __device__ constexpr int slot_reals(int slot, int nk) { return slot < 8 ? 18 : naik_reals(nk); }

__host__ __device__ constexpr int slot_real_start(int slot, int nk)
{
    return slot < 8 ? 18 * slot : 144 + naik_reals(nk) * (slot - 8);
}

__host__ __device__ inline size_t link_block_reals(int Vh, int nk)
{
    return size_t(144 + 8 * naik_reals(nk)) * size_t(Vh);
}

// Per-rhs sums over a grid.  The kernel that produces a sum leaves at most
// kSumDoubles / np rows of partial sums (np: the bundle size rounded up to a
// power of two, the row's stride), and the kernel that needs the sum adds the rows
// itself, in every work-group: 8 loads per lane, no wait for a last work-group.
// A grid of more work-groups than rows first sums groups of `sum_group`
// consecutive work-groups into one row each.
constexpr int kSumDoubles = 512;
// Group counters are dealt over 64 cache lines of 128 bytes: atomics on one
// line are served one after another (about 10 ns each), on different lines in
// parallel.
constexpr int kCounterLines = 64, kCounterStride = 32;
__host__ __device__ constexpr int counter_index(int grp)
{
    return grp % kCounterLines * kCounterStride + grp / kCounterLines;
}
__host__ __device__ constexpr int sum_stride(int n) { return n <= 1 ? 1 : n <= 2 ? 2 : n <= 4 ? 4 : 8; }
inline int sum_group(int nblk, int n)
{
    const int most = kSumDoubles / sum_stride(n);
    return (nblk + most - 1) / most;
}
inline int sum_row_count(int nblk, int n)
{
    const int g = sum_group(nblk, n);
    return (nblk + g - 1) / g;
}

// Where a reducing kernel leaves its sums (one, or two at a time).
struct SumOut {
    double* rows;   // [sum_row_count][sum_stride] of each sum, kSumDoubles apart, read by the consumer
    double* part;   // per-work-group partials (groups of more than one), [work-group][sum][sum_stride]
    uint32_t* cnt;  // group counters (zero between launches)
    int group;      // work-groups per row
};

// A finished sum as its consumer sees it.
struct SumIn {
    const double* rows;
    int n;
};

// Per-problem CG scalars, in device memory (FP64).  The host reads and writes
// one copy; inside a poll block the scalars pass through two further copies:
// the p-update that starts an iteration reads the previous copy and the |r|^2
// rows, and writes the next one, which the iteration's Dslash kernels read (so
// no work-group reads a scalar that another one is writing).
struct CgState {
    double rr[kMaxRhs];      // current (iterated) |r|^2
    double beta[kMaxRhs];
    double thresh[kMaxRhs];  // device-side masking threshold on rr
    double rr_true[kMaxRhs]; // |b - A x|^2 of the last true-residual pass
    double aux[kMaxRhs];     // |b|^2
    double rrmax[kMaxRhs];   // largest iterated |r|^2 since the last true-residual pass
    int32_t active[kMaxRhs];
    int32_t status[kMaxRhs];
    int32_t iters[kMaxRhs];
    int32_t sel[kMaxRhs];    // rhs selected for the next true-residual pass
    int32_t brk[kMaxRhs];    // <p, A p> of this iteration was not positive and finite
    int32_t maxiter;
    int32_t frozen;          // 1 while the autotuner times kernels: alpha = 0, nothing is recorded
    int32_t pad[6];
};

enum Epi {
    EPI_PLAIN = 0,  // out = D in
    EPI_NORM = 1,   // t = D_oe p; |p|^2 and |t|^2
    EPI_CG = 2,     // alpha from |p|^2, |t|^2; u = D_eo t; q = 4m^2 p - u; x += alpha p; r -= alpha q; |r|^2
    EPI_RESID = 3   // (FP64) r = b - (4m^2 x - D_eo t) for selected rhs; |r|^2
};

// Arguments of one Dslash launch (one problem).
template <typename T>
struct DslashArgs {
    Lat lat;
    int parity;  // output parity
    const cplx<T>* links;  // link block of the output parity
    const cplx<T>* in;
    cplx<T>* out;
    // CG epilogue
    const cplx<T>* p;
    cplx<T>* x;
    cplx<T>* r;
    // residual epilogue (FP64 b, x)
    const d2* b;
    const d2* xh;
    double mass4;  // 4 m^2
    CgState* state;
    SumOut sum;    // where |p|^2 and |t|^2, or |r|^2, go
    SumIn pp, tt;  // EPI_CG: |p|^2 and |t|^2 of this iteration
    int ntiles;
    int remap;
    int rows;  // LDS-staged x-rows per tile (0: unstaged)
    const float* naik_scale;  // r9 links: the scale in their header
};

template <typename T>
struct PupdateArgs {
    Lat lat;
    const cplx<T>* r;
    cplx<T>* p;
    const CgState* src;  // scalars of the previous iteration, or the host's copy
    CgState* dst;        // scalars of this iteration
    SumIn rr;            // |r|^2 of the previous iteration (not with fresh)
    int fresh;           // 1: beta and the masks stand in src as they are
};

// One problem of a batched launch: the arguments of its three CG phases and
// its range of work-groups in the flattened (problem, tile) grid.
// k1.src / k1.dst / k2.state / k3.state are set from `state` by the launch's
// phase (state_of_phase).
template <typename T>
struct BatchProb {
    PupdateArgs<T> k1;
    DslashArgs<T> k2;
    DslashArgs<T> k3;
    CgState* state[3];  // the host's copy, then the two of the poll block
    int n;
    int nr;
    int block_start;  // of the Dslash launches
    int nblocks;
    int pup_start;  // of the p-update launch
    int pup_blocks;
};

template <typename T>
struct BatchTable {
    BatchProb<T> p[HISQ_MAX_PROBLEMS];
    int nprob;
    int total_blocks;
};

// Launch shape: rhs per thread, work-group size (one tile of bs threads per
// work-group), XCD-contiguous tile order.
struct Tile {
    int nr;
    int bs;
    int remap;
    int rows = 0;  // > 0: LDS-staged Dslash, the work-group covers `rows` x-rows
    int split = 0;  // 1: four lanes per site and rhs, one per direction (nr = 1)
};

// Sites per work-group and work-groups of a Dslash launch of n rhs: a wave holds
// as many whole sites as its 64 lanes allow.
inline int tile_sites(const Lat& lat, int n, const Tile& t)
{
    return t.rows > 0 ? t.rows * lat.Lh0 : t.bs / 64 * (64 / (n / t.nr * (t.split ? 4 : 1)));
}
inline int tile_blocks(const Lat& lat, int n, const Tile& t)
{
    const int ts = tile_sites(lat, n, t);
    return (lat.Vh + ts - 1) / ts;
}

// Iteration j of a poll block runs in phase 0 (j = 0), 1 (j odd) or 2 (j even):
// it reads the copy state_of_phase(phase, 0) and writes state_of_phase(phase, 1).
__host__ __device__ constexpr int state_of_phase(int phase, int dst)
{
    return dst ? (phase == 1 ? 2 : 1) : phase;
}
inline int phase_of(int j) { return j == 0 ? 0 : (j & 1) ? 1 : 2; }

// Reduction scratch for a grid of up to `blocks` work-groups: the rows of the
// three sums of an iteration (|p|^2, |t|^2, |r|^2), then the partials.
enum SumSlot { SUM_PP = 0, SUM_TT = 1, SUM_RR = 2, SUM_SLOTS = 3 };
// Every reducing work-group covers at least kLeastSites sites (whole waves, at most
// kMaxRhs lanes per site; split_tile sees to it for four times that) and leaves at
// most two sums.
constexpr int kLeastSites = 8;
static_assert(64 / kMaxRhs >= kLeastSites, "sites of a one-wave work-group");
inline size_t red_doubles(int Vh, int n)
{
    return (size_t)SUM_SLOTS * kSumDoubles + ((size_t)Vh / kLeastSites + 1) * 2 * sum_stride(n);
}
constexpr size_t kRedCounters = (size_t)kCounterLines * kCounterStride;
static_assert(kSumDoubles <= kCounterLines * kCounterStride, "a counter for every group");

// Launchers, defined in the per-precision kernel objects.  cm selects the
// colour-major field layout [3][Vh][n] (the solver's); the plain Dslash also
// exists for the site-major canonical layout [Vh][3][n].
hipError_t launch_dslash_f64(int epi, int nrhs, const Tile& t, const DslashArgs<double>& a,
                             hipStream_t s, bool cm);
// nk: Naik storage of the FP32 links (HISQ_NAIK_FULL, _R14, _R13)
hipError_t launch_dslash_f32(int epi, int nk, int nrhs, const Tile& t, const DslashArgs<float>& a,
                             hipStream_t s, bool cm);
hipError_t launch_dslash_batched_f64(int epi, const BatchTable<double>* tab, int total_blocks,
                                     int bs, int phase, hipStream_t s);
hipError_t launch_dslash_batched_f32(int epi, int nk, const BatchTable<float>* tab,
                                     int total_blocks, int bs, int phase, hipStream_t s);
hipError_t launch_pupdate_batched_f64(const BatchTable<double>* tab, int total_blocks, int phase,
                                      hipStream_t s);
hipError_t launch_pupdate_batched_f32(const BatchTable<float>* tab, int total_blocks, int phase,
                                      hipStream_t s);
// End of a poll block: folds the last iteration (src, |r|^2 rows) into the
// host's copy dst, for each of nprob problems.
struct FoldArgs {
    struct One {
        const CgState* src;
        CgState* dst;
        SumIn rr;
        int nrhs;
    } p[HISQ_MAX_PROBLEMS];
};
hipError_t launch_fold(const FoldArgs& a, int nprob, hipStream_t s);
// rhs-per-thread tiles the batched kernels are built for
inline bool batched_nr_ok(int n, int nr) { return nr == n || (n % 2 == 0 && nr == n / 2); }
// work-groups of a p-update; elem: bytes of a real
int pupdate_blocks(int nrhs, int Vh, size_t elem);
hipError_t launch_pupdate_f64(int nrhs, const PupdateArgs<double>& a, hipStream_t s);
hipError_t launch_pupdate_f32(int nrhs, const PupdateArgs<float>& a, hipStream_t s);

// Elementwise and reduction helpers (blas.hip).
hipError_t launch_zero(void* p, size_t bytes, hipStream_t s);
hipError_t launch_state_reset(CgState* st, int nrhs, int active, hipStream_t s);
// out[k] = scale * (sum of rows, rhs k)
hipError_t launch_sum_final(SumIn in, int nrhs, double scale, double* out, hipStream_t s);
// per-rhs |v|^2 of a colour-major FP64 field; o: the reduction scratch (group is set here)
hipError_t launch_norm2_f64(const d2* v, int Vh, int nrhs, double* out, SumOut o, hipStream_t s);
hipError_t launch_to_f32_sel(const d2* src, f2* dst, size_t ncplx, int nrhs, const CgState* st,
                             hipStream_t s);
hipError_t launch_accum_sel(d2* xh, f2* xl, size_t ncplx, int nrhs, const CgState* st,
                            hipStream_t s);
hipError_t launch_copy_f64(const d2* src, d2* dst, size_t ncplx, hipStream_t s);
hipError_t launch_layout(const d2* src, d2* dst, int Vh, int nrhs, bool to_colour_major, hipStream_t s);
hipError_t launch_axpby(const d2* a, const d2* b, d2* out, size_t n, double alpha, double beta,
                        hipStream_t s);
size_t cdot_scratch_doubles(int Vh, int nrhs);
// out[2k], out[2k+1] = re, im of sum conj(a) b over both half fields, rhs k
hipError_t launch_cdot(const d2* ae, const d2* be, const d2* ao, const d2* bo, int Vh, int nrhs,
                       double* scratch, double* out, hipStream_t s);
// d^n D / d mu^n at mu = 0 (n >= 1), FP64 links of the output parity, site-major
hipError_t launch_dslash_dmu(const Lat& lat, int parity, int nrhs, int nder, const d2* lk,
                             const d2* in, d2* out, hipStream_t s);
hipError_t launch_zero_sel(d2* v, size_t ncplx, int nrhs, const CgState* st, hipStream_t s);
hipError_t launch_redot(const d2* y, const d2* x, int Vh, int nrhs, double scale, double* out,
                        SumOut o, hipStream_t s);

// The solve of hisq_cg_solve over a workspace region (api.cpp); host_buf, if
// not NULL, holds HISQ_MAX_PROBLEMS host copies of the CG state in place of
// the calling thread's pinned buffer.
int cg_solve_on(const hisq_geom* g, double mass, int nrhs, const hisq_params* p,
                const void* links64, const void* links32, const double* b_e, double* x_e,
                void* ws, size_t ws_bytes, hisq_info* info, void* stream, CgState* host_buf);
// The size that the limit of hisq_cg_solve_noalloc is counted in: the solve's
// fields with 8 doubles of reduction scratch per 8 sites, whatever scratch the
// kernels use (0 on invalid input).
size_t no_alloc_bytes(const hisq_geom* g, int nrhs, int mode);
// Sets the message of hisq_last_error() for this thread; returns code.
int report_error(int code, const char* fmt, ...);

// Link packing (pack.hip) and the link force (force.hip).
hipError_t launch_pack(const Lat& lat, const d2* U, const d2* N, int prec, int naik,
                       void* packed, hipStream_t s);
// link force from colour-major FP64 fields x, y (even) and D_oe x, D_oe y (odd)
hipError_t launch_force(const Lat& lat, int nrhs, const d2* xc, const d2* yc, const d2* txc,
                        const d2* syc, d2* GU, d2* GN, hipStream_t s);

}  // namespace hisq
