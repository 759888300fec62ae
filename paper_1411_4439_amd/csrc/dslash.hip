// HISQ half-Dslash kernels for gfx950 (Sec. 1, eqs. (3) and (4)).
//
// One thread computes NR rhs of one output site; the G = n/NR threads of a
// site are adjacent lanes, so their spinor loads are contiguous and their link
// loads hit the same cache line.  Per output site the thread streams the 16
// matrices of its parity block once (non-temporal loads: links have no reuse
// within a half-Dslash) and gathers the 16 neighbour colour vectors of its rhs
// tile; the neighbour vectors are re-read by up to 16 sites and are served from
// L2 / Infinity Cache.  All accumulation is in the storage precision; the CG
// dot products are accumulated in FP64.
//
// This file is compiled once per (precision, Naik storage, epilogue):
//   HISQ_KPREC 0 = FP64, 1 = FP32, 2 = FP32 with r14 Naik links,
//              3 = FP32 with r13 Naik links, 4 = FP32 with r9 Naik links
//   HISQ_KEPI  one of EPI_PLAIN, EPI_NORM, EPI_CG, EPI_RESID
#include <type_traits>

#include "naik.h"
#include "stencil.h"

#ifndef HISQ_KPREC
#error "HISQ_KPREC must be defined"
#endif
#ifndef HISQ_KEPI
#error "HISQ_KEPI must be defined"
#endif

namespace hisq {

#if HISQ_KPREC == 0
using KT = double;
constexpr int kNK = HISQ_NAIK_FULL;
#elif HISQ_KPREC == 1
using KT = float;
constexpr int kNK = HISQ_NAIK_FULL;
#elif HISQ_KPREC == 2
using KT = float;
constexpr int kNK = HISQ_NAIK_R14;
#elif HISQ_KPREC == 3
using KT = float;
constexpr int kNK = HISQ_NAIK_R13;
#else
using KT = float;
constexpr int kNK = HISQ_NAIK_R9;
#endif

template <typename T, int NRHS, int NR, bool CM>
__device__ __forceinline__ void load_vec(const cplx<T>* __restrict__ in, int Vh, int nbr, int g,
                                         cplx<T> (&v)[3][NR])
{
    using Lay = Layout<NRHS, CM>;
    const cplx<T>* vp = in + Lay::site(nbr) + g * NR;
#pragma unroll
    for (int b = 0; b < 3; ++b) load_rhs<NR>(vp + Lay::colour(b, Vh), v[b]);
}

// Naik storage r13: c = exp(i phi) / |row0|, phi loaded into m[6].x (for
// N = s V, V in U(3): |row0| = s and c = det V / s)
template <typename T>
__device__ __forceinline__ cplx<T> r13_coefficient(const cplx<T> (&m)[9])
{
    static_assert(sizeof(T) == 4, "r13 is an FP32 storage");
    const float n2 = m[0].x * m[0].x + m[0].y * m[0].y + m[1].x * m[1].x + m[1].y * m[1].y +
                     m[2].x * m[2].x + m[2].y * m[2].y;
    float cs, sn;
    unit_phase(m[6].x, &cs, &sn);
    const float inv = __builtin_amdgcn_rsqf(n2);
    return cplx<T>{cs * inv, sn * inv};
}

// Naik storage r9: m[0..3] and m[4].x hold the 9 reals of H; the matrix is
// ns exp(iH), ns the field's Naik scale.
template <typename T>
__device__ __forceinline__ void r9_matrix(cplx<T> (&m)[9], T ns)
{
    static_assert(sizeof(T) == 4, "r9 is an FP32 storage");
    const T h[9] = {m[0].x, m[0].y, m[1].x, m[1].y, m[2].x, m[2].y, m[3].x, m[3].y, m[4].x};
    T re[9], im[9];
    expi_hermitian<T>(h, ns, re, im);
#pragma unroll
    for (int e = 0; e < 9; ++e) m[e] = cplx<T>{re[e], im[e]};
}

template <typename T, int NR, int NK, int S>
__device__ __forceinline__ void apply_slot(cplx<T> (&m)[9], const cplx<T> (&v)[3][NR],
                                           cplx<T> (&acc)[3][NR], T ns)
{
    if constexpr (NK == HISQ_NAIK_R9 && S >= 8) {
        r9_matrix<T>(m, ns);
    } else if constexpr (NK != HISQ_NAIK_FULL && S >= 8) {
        // row 2 = c * conj(row0 x row1); r14 loaded c into m[6], r13 its phase
        cplx<T> cc = m[6];
        if constexpr (NK == HISQ_NAIK_R13) cc = r13_coefficient<T>(m);
        m[6] = cmul(cc, cconj(cmul(m[1], m[5]) - cmul(m[2], m[4])));
        m[7] = cmul(cc, cconj(cmul(m[2], m[3]) - cmul(m[0], m[5])));
        m[8] = cmul(cc, cconj(cmul(m[0], m[4]) - cmul(m[1], m[3])));
    }
#pragma unroll
    for (int b = 0; b < 3; ++b)
#pragma unroll
        for (int a = 0; a < 3; ++a)
#pragma unroll
            for (int k = 0; k < NR; ++k) cfma(acc[a][k], m[3 * a + b], v[b][k]);
}

// lanes that share one site's link loads: the site's lanes, quads when there are
// 8, none when their number is not a power of two (they do not fill quads)
template <int NRHS, int NR>
constexpr int link_group()
{
    constexpr int G = NRHS / NR;
    return G == 1 || G == 2 || G == 4 ? G : G == 8 ? 4 : 1;
}

// Pipeline step k -> slot: even steps take the z and t slots, odd steps the x
// and y slots, hops +1, -1, +3, -3 within each direction.  The LDS-staged
// kernel reads the x and y neighbours from LDS and overlaps them with the
// global z and t reads; the unstaged kernel sums the slots in the same order,
// so the two give bitwise identical results.
__host__ __device__ constexpr int slot_at(int k)
{
    return ((k & 1) ? ((k >> 3) & 1) : 2 + ((k >> 3) & 1)) + 4 * ((k >> 1) & 3);
}

template <typename T>
__device__ __forceinline__ double norm2c(cplx<T> v)
{
    return (double)v.x * (double)v.x + (double)v.y * (double)v.y;
}

template <typename T, int NR>
__device__ __forceinline__ void own_norm(const cplx<T> (&v)[3][NR], double (&own)[NR])
{
#pragma unroll
    for (int k = 0; k < NR; ++k)
        own[k] = norm2c<T>(v[0][k]) + norm2c<T>(v[1][k]) + norm2c<T>(v[2][k]);
}

// acc[c][k] = (D in)_{i}, colour c, rhs g*NR + k, output parity P.
// Slot s = 4*hop + mu applies matrix s of the parity block to the neighbour
// reached by hop (+1, -1, +3, -3) in direction mu.  The 16 slots run as a
// software pipeline: while one slot is multiplied, the neighbour vectors of
// the next slot and its matrix are in flight (links stream from HBM and see
// the longest latency; neighbour vectors mostly hit L2).  The scheduling
// barriers keep the compiler from hoisting further loads, which would
// otherwise exhaust the register file.
//
// With PN, own[k] = |in_i|^2, the field at the site's own index: the half-site
// of the other parity one step away in x, a line that the +1 or -1 x-slot has
// brought already.  It is read as a 17th slot without a link, into the buffer
// that the last slot leaves free; summing it from the x-slot itself (which of
// the two it is depends on x) broke the pipeline and spilled.
template <typename T, int NRHS, int NR, int NK, bool CM, bool PN>
__device__ __forceinline__ void dslash_site(const Lat& lat, int P, int i, int g,
                                            const cplx<T>* __restrict__ lk,
                                            const cplx<T>* __restrict__ in,
                                            cplx<T> (&acc)[3][NR], T ns, double (&own)[NR])
{
    using C = cplx<T>;
    const int Vh = lat.Vh;
    const SiteCoord sc = site_coord(lat, P, i);
#pragma unroll
    for (int c = 0; c < 3; ++c)
#pragma unroll
        for (int k = 0; k < NR; ++k) acc[c][k] = C{0, 0};

    // link lookahead: two slots in FP32; one in FP64, whose 36-register
    // matrices would otherwise cost a wave of occupancy
#ifndef HISQ_FP32_LINK_LOOKAHEAD
#define HISQ_FP32_LINK_LOOKAHEAD 1
#endif
    constexpr int LD = sizeof(T) == 4 ? HISQ_FP32_LINK_LOOKAHEAD : 1;
    constexpr int G = link_group<NRHS, NR>();
    const int gl = g % G;
    LinkRaw<T, G> lr[LD + 1];
    C v[2][3][NR];
    load_link_part<T, NK, slot_at(0), G>(lk, Vh, i, gl, lr[0]);
    if constexpr (LD == 2) load_link_part<T, NK, slot_at(1), G>(lk, Vh, i, gl, lr[1]);
    load_vec<T, NRHS, NR, CM>(in, Vh, neighbour<slot_at(0)>(lat, sc), g, v[0]);
    static_for<0, 16>([&](auto K) {
        constexpr int k = decltype(K)::value;
        if constexpr (k + LD < 16)
            load_link_part<T, NK, slot_at(k + LD), G>(lk, Vh, i, gl, lr[(k + LD) % (LD + 1)]);
        if constexpr (k + 1 < 16)
            load_vec<T, NRHS, NR, CM>(in, Vh, neighbour<slot_at(k + 1)>(lat, sc), g, v[(k + 1) & 1]);
        else if constexpr (PN)
            load_vec<T, NRHS, NR, CM>(in, Vh, i, g, v[(k + 1) & 1]);
        __builtin_amdgcn_sched_barrier(0);
        C m[9];
        share_link<T, NK, slot_at(k), G>(lr[k % (LD + 1)], m);
        apply_slot<T, NR, NK, slot_at(k)>(m, v[k & 1], acc, ns);
        __builtin_amdgcn_sched_barrier(0);
    });
    if constexpr (PN) own_norm<T, NR>(v[0], own);
}

// ---------------------------------------------------------------------------
// Split form, for launches too small to fill the chip: four adjacent lanes share
// a site and its rhs tile, lane mu takes the four hops of direction mu, issues
// all their loads at once and the quad adds the four partial results with DPP
// permutes.  A wave then waits for one memory round trip instead of 16 in a
// row, and there are four times as many waves; but every rhs loads its site's links
// for itself.  Both sides, and where the line lies, stand with the launch rule
// (kSplitLanes in api.cpp).
template <typename T, int NK, int HH>
__device__ __forceinline__ void load_link_dir(const cplx<T>* __restrict__ lk, int Vh, int i, int mu,
                                              cplx<T> (&m)[9])
{
    // as load_link, for slot 4 * HH + mu
    constexpr int nr = slot_reals(4 * HH, NK);
    const T* base = reinterpret_cast<const T*>(lk) +
                    (size_t)(slot_real_start(4 * HH, NK) + mu * nr) * Vh;
    if constexpr (sizeof(T) == 4) {
        constexpr int nw = nr / 4, rem = nr % 4;
        const f4* wp = reinterpret_cast<const f4*>(base) + i;
#pragma unroll
        for (int w = 0; w < nw; ++w) {
            const f4 q = __builtin_nontemporal_load(wp + (size_t)w * Vh);
            m[2 * w] = cplx<T>{q.x, q.y};
            m[2 * w + 1] = cplx<T>{q.z, q.w};
        }
        const T* tail = base + (size_t)4 * nw * Vh;
        if constexpr (rem == 2)
            m[2 * nw] = __builtin_nontemporal_load(reinterpret_cast<const cplx<T>*>(tail) + i);
        else if constexpr (rem == 1)
            m[2 * nw] = cplx<T>{__builtin_nontemporal_load(tail + i), T(0)};
    } else {
        const cplx<T>* lp = reinterpret_cast<const cplx<T>*>(base) + i;
#pragma unroll
        for (int e = 0; e < 9; ++e) m[e] = __builtin_nontemporal_load(lp + (size_t)e * Vh);
    }
}

template <typename T, int NRHS, int NR, int NK>
__device__ __forceinline__ void dslash_site_split(const Lat& lat, int P, int i, int g, int mu,
                                                  const cplx<T>* __restrict__ lk,
                                                  const cplx<T>* __restrict__ in,
                                                  cplx<T> (&acc)[3][NR], T ns)
{
    using C = cplx<T>;
    const SiteCoord sc = site_coord(lat, P, i);
    // scalar registers first: a select between members of the argument struct
    // becomes an indexed load from a copy of it in scratch memory
    auto scalar = [](int v) { return __builtin_amdgcn_readfirstlane(v); };
    const int l0 = scalar(lat.L[0]), l1 = scalar(lat.L[1]), l2 = scalar(lat.L[2]), l3 = scalar(lat.L[3]);
    const int s1 = scalar(lat.sy), s2 = scalar(lat.sz), s3 = scalar(lat.st);
    const int c = mu == 0 ? sc.x : mu == 1 ? sc.c[1] : mu == 2 ? sc.c[2] : sc.c[3];
    const int ext = mu == 0 ? l0 : mu == 1 ? l1 : mu == 2 ? l2 : l3;
    const int stride = mu == 1 ? s1 : mu == 2 ? s2 : s3;
    C m[4][9], v[4][3][NR];
    static_for<0, 4>([&](auto H) {
        constexpr int hh = decltype(H)::value;
        constexpr int h = hh == 0 ? 1 : hh == 1 ? -1 : hh == 2 ? 3 : -3;
        const int d = wrap_delta(c, h, ext);
        const int nbr = mu == 0 ? sc.row + ((c + d) >> 1) : i + d * stride;
        load_vec<T, NRHS, NR, true>(in, lat.Vh, nbr, g, v[hh]);
        load_link_dir<T, NK, hh>(lk, lat.Vh, i, mu, m[hh]);
    });
#pragma unroll
    for (int a = 0; a < 3; ++a)
#pragma unroll
        for (int k = 0; k < NR; ++k) acc[a][k] = C{0, 0};
    static_for<0, 4>([&](auto H) {
        constexpr int hh = decltype(H)::value;
        apply_slot<T, NR, NK, 4 * hh>(m[hh], v[hh], acc, ns);
    });
#pragma unroll
    for (int a = 0; a < 3; ++a)
#pragma unroll
        for (int k = 0; k < NR; ++k) {
            acc[a][k].x = quad_sum(acc[a][k].x);
            acc[a][k].y = quad_sum(acc[a][k].y);
        }
}

// ---------------------------------------------------------------------------
// LDS-staged form.  A work-group covers R whole x-rows
// of one (z, t) plane.  The input rows y0-3 .. y0+R+2 of that plane (periodic
// in y) are copied to LDS once, laid out [3][R+6][L0/2][n] (colour-major fields)
// or [R+6][L0/2][3][n] (site-major ones, plain Dslash only); the x and y
// neighbours (8 of the 16 slots) are then read from LDS and only the z and t
// neighbours and the links come from global memory.

template <typename T, int NRHS, bool CM>
__device__ __forceinline__ void stage_rows(const cplx<T>* __restrict__ in, cplx<T>* lds,
                                           const Lat& lat, int row0, int R)
{
    const int Ly = lat.L[1];
    const int plane = row0 / Ly, y0 = row0 - plane * Ly;
    const unsigned rows = (unsigned)R + 6;
    // half-site of staged row j (y0 - 3 + j, periodic; Ly >= 4 > 3)
    auto row_site = [&](unsigned j) -> size_t {
        int yy = y0 - 3 + (int)j;
        yy += yy < 0 ? Ly : 0;
        yy -= yy >= Ly ? Ly : 0;
        return (size_t)(plane * Ly + yy) * lat.Lh0;
    };
    // Each thread copies its units in batches of kStageBatch: all the batch's
    // reads are issued before the first LDS write, so a thread waits for one
    // memory round trip per batch instead of one per unit.
    constexpr unsigned kStageBatch = 16;
    const unsigned nt = blockDim.x;
    // unit u -> (colour c, staged row j, offset): u / chunk through a float
    // reciprocal with a one-step correction (u < 2^16 here, so the estimate
    // is off by at most one), c by comparisons (c < 3)
    auto split = [rows](unsigned u, unsigned chunk, float inv, unsigned& c, unsigned& j,
                        unsigned& off) {
        unsigned cj = (unsigned)((float)u * inv);
        int r = (int)u - (int)(cj * chunk);
        if (r < 0) {
            --cj;
            r += (int)chunk;
        } else if (r >= (int)chunk) {
            ++cj;
            r -= (int)chunk;
        }
        off = (unsigned)r;
        c = (cj >= rows ? 1u : 0u) + (cj >= 2 * rows ? 1u : 0u);
        j = cj - c * rows;
    };
    if constexpr (!CM) {
        // a row is one contiguous stretch of all three colours, in LDS as in memory
        constexpr unsigned elt = sizeof(cplx<T>);
        if (elt == 16 || (lat.Lh0 * 3 * NRHS) % 2 == 0) {
            const unsigned chunk = (unsigned)(lat.Lh0 * 3 * NRHS) * elt / 16;
            const unsigned total = rows * chunk;
            const float inv = 1.0f / (float)chunk;
            const f4* src = reinterpret_cast<const f4*>(in);
            f4* dst = reinterpret_cast<f4*>(lds);
            for (unsigned u0 = threadIdx.x; u0 < total; u0 += kStageBatch * nt) {
                f4 buf[kStageBatch];
#pragma unroll
                for (unsigned q = 0; q < kStageBatch; ++q) {
                    const unsigned u = u0 + q * nt;
                    if (u < total) {
                        unsigned c, j, off;
                        split(u, chunk, inv, c, j, off);
                        j += c * rows;
                        buf[q] = src[row_site(j) * (3 * NRHS) * elt / 16 + off];
                    }
                }
#pragma unroll
                for (unsigned q = 0; q < kStageBatch; ++q)
                    if (u0 + q * nt < total) dst[u0 + q * nt] = buf[q];
            }
        } else {
            const unsigned chunk = (unsigned)(lat.Lh0 * 3 * NRHS);
            for (unsigned u = threadIdx.x; u < rows * chunk; u += nt) {
                const unsigned j = u / chunk;
                lds[u] = in[row_site(j) * (3 * NRHS) + (u - j * chunk)];
            }
        }
        return;
    }
    if constexpr (sizeof(T) == 4) {
        if ((lat.Lh0 * NRHS) % 2 == 0) {
            // 16-byte units of two complex numbers
            const unsigned chunk = (unsigned)(lat.Lh0 * NRHS / 2);
            const unsigned total = 3u * rows * chunk;
            const float inv = 1.0f / (float)chunk;
            const f4* src = reinterpret_cast<const f4*>(in);
            f4* dst = reinterpret_cast<f4*>(lds);
            for (unsigned u0 = threadIdx.x; u0 < total; u0 += kStageBatch * nt) {
                f4 buf[kStageBatch];
#pragma unroll
                for (unsigned q = 0; q < kStageBatch; ++q) {
                    const unsigned u = u0 + q * nt;
                    if (u < total) {
                        unsigned c, j, off;
                        split(u, chunk, inv, c, j, off);
                        buf[q] = src[((size_t)c * lat.Vh + row_site(j)) * NRHS / 2 + off];
                    }
                }
#pragma unroll
                for (unsigned q = 0; q < kStageBatch; ++q)
                    if (u0 + q * nt < total) dst[u0 + q * nt] = buf[q];
            }
            return;
        }
    }
    const unsigned chunk = (unsigned)(lat.Lh0 * NRHS);
    const unsigned total = 3u * rows * chunk;
    const float inv = 1.0f / (float)chunk;
    for (unsigned u0 = threadIdx.x; u0 < total; u0 += kStageBatch * nt) {
        cplx<T> buf[kStageBatch];
#pragma unroll
        for (unsigned q = 0; q < kStageBatch; ++q) {
            const unsigned u = u0 + q * nt;
            if (u < total) {
                unsigned c, j, off;
                split(u, chunk, inv, c, j, off);
                buf[q] = in[((size_t)c * lat.Vh + row_site(j)) * NRHS + off];
            }
        }
#pragma unroll
        for (unsigned q = 0; q < kStageBatch; ++q)
            if (u0 + q * nt < total) lds[u0 + q * nt] = buf[q];
    }
}

template <typename T, int NRHS, int NR, bool CM>
__device__ __forceinline__ void load_vec_lds(const cplx<T>* lds, int cstride, int site, int g,
                                             cplx<T> (&v)[3][NR])
{
    const cplx<T>* vp = lds + site * (CM ? NRHS : 3 * NRHS) + g * NR;
#pragma unroll
    for (int b = 0; b < 3; ++b) load_rhs<NR>(vp + b * cstride, v[b]);
}

// Staged row-local index of the x / y neighbour of slot S (mu = 0 or 1) of the
// output site in row r of the tile, half-x xh, full x coordinate x.
template <int S>
__device__ __forceinline__ int lds_neighbour(const Lat& lat, int r, int xh, int x)
{
    constexpr int mu = S & 3;
    constexpr int hh = S >> 2;
    constexpr int h = hh == 0 ? 1 : hh == 1 ? -1 : hh == 2 ? 3 : -3;
    static_assert(mu < 2, "only x and y neighbours are staged");
    if constexpr (mu == 0) {
        const int xp = x + wrap_delta(x, h, lat.L[0]);
        return (r + 3) * lat.Lh0 + (xp >> 1);
    } else {
        return (r + 3 + h) * lat.Lh0 + xh;
    }
}

// As dslash_site, for the site in row r of an LDS-staged tile.  Issue order
// follows use order, because a wait for one global read is a wait for every
// read issued before it: an even (global) step issues the next link, computes,
// then issues the link after that and the global neighbour of four steps ahead
// (two global slots of lookahead), and the LDS neighbour of the next step.
// The global reads that open the pipeline (slot 0's link, the first two
// global neighbours): issued before the work-group's staging barrier, so
// that their latency overlaps the staging reads instead of following them.
template <typename T, int NRHS, int NR, int NK>
struct LdsHead {
    LinkRaw<T, link_group<NRHS, NR>()> m;
    cplx<T> v0[3][NR], v1[3][NR];
};

template <typename T, int NRHS, int NR, int NK, bool CM>
__device__ __forceinline__ void lds_head(const Lat& lat, int P, int i, int g,
                                         const cplx<T>* __restrict__ lk,
                                         const cplx<T>* __restrict__ in, LdsHead<T, NRHS, NR, NK>& h)
{
    const SiteCoord sc = site_coord(lat, P, i);
    constexpr int G = link_group<NRHS, NR>();
    load_link_part<T, NK, slot_at(0), G>(lk, lat.Vh, i, g % G, h.m);
    load_vec<T, NRHS, NR, CM>(in, lat.Vh, neighbour<slot_at(0)>(lat, sc), g, h.v0);
    load_vec<T, NRHS, NR, CM>(in, lat.Vh, neighbour<slot_at(2)>(lat, sc), g, h.v1);
}

template <typename T, int NRHS, int NR, int NK, bool CM, bool PN>
__device__ __forceinline__ void dslash_site_lds(const Lat& lat, int P, int i, int g, int r,
                                                const cplx<T>* __restrict__ lk,
                                                const cplx<T>* __restrict__ in,
                                                const cplx<T>* lds, int rows,
                                                const LdsHead<T, NRHS, NR, NK>& h,
                                                cplx<T> (&acc)[3][NR], T ns, double (&own)[NR])
{
    using C = cplx<T>;
    const int Vh = lat.Vh;
    const SiteCoord sc = site_coord(lat, P, i);
    const int xh = i - sc.row;
    const int cstride = CM ? rows * lat.Lh0 * NRHS : NRHS;
#pragma unroll
    for (int c = 0; c < 3; ++c)
#pragma unroll
        for (int k = 0; k < NR; ++k) acc[c][k] = C{0, 0};
    constexpr int G = link_group<NRHS, NR>();
    const int gl = g % G;
    LinkRaw<T, G> m[2];
    C vg[2][3][NR];
    C vl[3][NR];
    m[0] = h.m;
#pragma unroll
    for (int b = 0; b < 3; ++b)
#pragma unroll
        for (int k = 0; k < NR; ++k) {
            vg[0][b][k] = h.v0[b][k];
            vg[1][b][k] = h.v1[b][k];
        }
    static_for<0, 16>([&](auto K) {
        constexpr int k = decltype(K)::value;
        if constexpr (k % 2 == 0) {
            load_link_part<T, NK, slot_at(k + 1), G>(lk, Vh, i, gl, m[(k + 1) & 1]);
            __builtin_amdgcn_sched_barrier(0);
            C mk[9];
            share_link<T, NK, slot_at(k), G>(m[k & 1], mk);
            apply_slot<T, NR, NK, slot_at(k)>(mk, vg[(k >> 1) & 1], acc, ns);
            __builtin_amdgcn_sched_barrier(0);
            if constexpr (k + 2 < 16) load_link_part<T, NK, slot_at(k + 2), G>(lk, Vh, i, gl, m[k & 1]);
            if constexpr (k + 4 < 16)
                load_vec<T, NRHS, NR, CM>(in, Vh, neighbour<slot_at(k + 4)>(lat, sc), g,
                                          vg[(k >> 1) & 1]);
            load_vec_lds<T, NRHS, NR, CM>(lds, cstride,
                                          lds_neighbour<slot_at(k + 1)>(lat, r, xh, sc.x), g, vl);
        } else {
            C mk[9];
            share_link<T, NK, slot_at(k), G>(m[k & 1], mk);
            apply_slot<T, NR, NK, slot_at(k)>(mk, vl, acc, ns);
        }
        __builtin_amdgcn_sched_barrier(0);
    });
    if constexpr (PN) {
        load_vec_lds<T, NRHS, NR, CM>(lds, cstride, (r + 3) * lat.Lh0 + xh, g, vl);
        own_norm<T, NR>(vl, own);
    }
}

// An empty asm that reads every accumulator: keeps the compiler from sinking
// the site's arithmetic into a later conditional block (past the loads of all
// 16 slots, which would keep every loaded operand live at once).
template <typename C, int NR>
__device__ __forceinline__ void pin_acc(C (&acc)[3][NR])
{
#pragma unroll
    for (int c = 0; c < 3; ++c)
#pragma unroll
        for (int k = 0; k < NR; ++k) asm volatile("" ::"v"(acc[c][k].x), "v"(acc[c][k].y));
}

// One tile (one work-group's worth of sites) of a half-Dslash with epilogue
// EPI; `tile` is the tile index, the problem's grid has nblk work-groups and
// this one is number bid (for the reductions).
template <typename T, int NRHS, int NR, int NK, int EPI, bool CM, bool ST = false, int SPL = 1>
__device__ __forceinline__ void dslash_tile(const DslashArgs<T>& a, CgState* state, int tile,
                                            int nblk, int bid, cplx<T>* lds = nullptr)
{
    using C = cplx<T>;
    using Map = LaneMap<NRHS, NR, SPL>;
    constexpr int G = Map::G;
    if constexpr (EPI == EPI_NORM || EPI == EPI_CG) {
        // every rhs of the bundle converged: the iteration is a no-op
        bool any_prob = false;
#pragma unroll
        for (int k = 0; k < NRHS; ++k) any_prob = any_prob || (state->active[k] != 0);
        if (!any_prob) return;
    }
    // a staged tile's lanes run on from site to site, across waves; where they
    // do not fill the last wave (plain Dslash only), its last lanes idle
    const int g = ST ? (int)threadIdx.x % G : Map::group();
    const int mu = Map::dir();  // split form: this lane's direction, then its colour
    constexpr int M = EPI == EPI_NORM ? 2 : 1;  // |p|^2 and |t|^2, or one sum
    double part[M][NR];
#pragma unroll
    for (int m = 0; m < M; ++m)
#pragma unroll
        for (int k = 0; k < NR; ++k) part[m][k] = 0.0;

    bool act[NR];
    T alpha[NR];
    bool any_act = false;
#pragma unroll
    for (int k = 0; k < NR; ++k) {
        act[k] = false;
        alpha[k] = T(0);
        if constexpr (EPI == EPI_RESID) act[k] = state->sel[g * NR + k] != 0;
        any_act = any_act || act[k];
    }
    // alpha = rr / <p, A p>, with <p, A p> = 4m^2 |p|^2 + |D_oe p|^2
    // (D_eo^dag = -D_oe); a rhs whose <p, A p> is not positive and finite is
    // masked here and reported.  The first wave works it out, before its sites,
    // and leaves it in LDS (in every wave it was 15% more load instructions:
    // 331 us instead of 324 at 48^3 x 12, 8 rhs, 256 threads).
    __shared__ T cg_alpha[EPI == EPI_CG ? kMaxRhs : 1];
    __shared__ int cg_live[EPI == EPI_CG ? kMaxRhs : 1];
    if constexpr (EPI == EPI_CG) {
        if (threadIdx.x < 64) {
            constexpr int NP = sum_stride(NRHS);
            const int kl = (int)threadIdx.x % NP;
            const double den = a.mass4 * sum_rows<NRHS>(a.pp) + sum_rows<NRHS>(a.tt);
            const bool on = kl < NRHS && state->active[kl] != 0;
            const bool good = den > 0.0 && finite_d(den);
            const bool frozen = state->frozen != 0;
            if (threadIdx.x < NRHS) {
                cg_alpha[kl] = on && good && !frozen ? (T)(state->rr[kl] / den) : T(0);
                cg_live[kl] = on && (good || frozen);
                if (bid == 0 && on && !good && !frozen) state->brk[kl] = 1;
            }
        }
    }
    const T m4 = (T)a.mass4;
    T ns = T(1);  // r9: the Naik scale of the links
    if constexpr (NK == HISQ_NAIK_R9) ns = (T)*a.naik_scale;

    const int stage_sites = ST ? a.rows * a.lat.Lh0 : 0;
    const int i = ST ? tile * stage_sites + (int)threadIdx.x / G : Map::site(tile);
    const bool live = ST ? (int)threadIdx.x < stage_sites * G : Map::live();
    LdsHead<T, NRHS, NR, NK> head;
    if constexpr (ST) {
        // the tile is `rows` whole x-rows: stage them and their +-3 row halo
        if (live) lds_head<T, NRHS, NR, NK, CM>(a.lat, a.parity, i, g, a.links, a.in, head);
        stage_rows<T, NRHS, CM>(a.in, lds, a.lat, tile * a.rows, a.rows);
        __syncthreads();
    }
    // The epilogue computes everything before its stores, posts the
    // work-group's reduction partials, and only then stores the outputs: the
    // completion wait that orders the partials before the counter update does
    // not wait for the output stores.
    bool on_site = live && i < a.lat.Vh;
    using Lay = Layout<NRHS, CM>;
    const int base = Lay::site(on_site ? i : 0) + g * NR;
    constexpr int NC = SPL == 1 ? 3 : 1;  // colours this lane stores
    C acc[3][NR];
    C xo[NC][NR], ro[NC][NR];  // EPI_CG: updated x and r
    d2 rr[NC][NR];             // EPI_RESID: the FP64 residual
    auto colour = [&](int c) { return base + Lay::colour(SPL == 1 ? c : mu, a.lat.Vh); };
    if (on_site) {
        if constexpr (SPL > 1) {
            static_assert(CM && !ST, "split form: colour-major fields, not staged");
            C pv[NR];
            if constexpr (EPI == EPI_NORM) load_rhs<NR>(a.in + base + Lay::colour(mu < 3 ? mu : 0, a.lat.Vh), pv);
            dslash_site_split<T, NRHS, NR, NK>(a.lat, a.parity, i, g, mu, a.links, a.in, acc, ns);
            if constexpr (EPI == EPI_NORM) {
#pragma unroll
                for (int k = 0; k < NR; ++k) part[0][k] = mu < 3 ? norm2c<T>(pv[k]) : 0.0;
            }
#pragma unroll
            for (int k = 0; k < NR; ++k) acc[0][k] = mu == 0 ? acc[0][k] : mu == 1 ? acc[1][k] : acc[2][k];
        } else if constexpr (ST)
            dslash_site_lds<T, NRHS, NR, NK, CM, EPI == EPI_NORM>(
                a.lat, a.parity, i, g, ((int)threadIdx.x / G) / a.lat.Lh0, a.links, a.in, lds,
                a.rows + 6, head, acc, ns, part[0]);
        else
            dslash_site<T, NRHS, NR, NK, CM, EPI == EPI_NORM>(a.lat, a.parity, i, g, a.links, a.in,
                                                              acc, ns, part[0]);
        pin_acc(acc);
    }
    // split form: lanes 0..2 of a quad each store one colour
    if constexpr (SPL > 1) on_site = on_site && mu < 3;
    if constexpr (EPI == EPI_CG) {
        __syncthreads();
#pragma unroll
        for (int k = 0; k < NR; ++k) {
            alpha[k] = cg_alpha[g * NR + k];
            act[k] = cg_live[g * NR + k] != 0;
            any_act = any_act || act[k];
        }
    }
    if (on_site) {
        if constexpr (EPI == EPI_NORM) {
#pragma unroll
            for (int c = 0; c < NC; ++c)
#pragma unroll
                for (int k = 0; k < NR; ++k) part[M - 1][k] += norm2c<T>(acc[c][k]);
        } else if constexpr (EPI == EPI_CG) {
            if (any_act) {
            // converged (masked) rhs are not written (and not read where the
            // whole tile of the thread is masked); their partial sums stay
            // zero and are ignored
#pragma unroll
            for (int c = 0; c < NC; ++c) {
                C pv[NR];
                load_rhs<NR, true>(a.p + colour(c), pv);
                load_rhs<NR, true>(a.x + colour(c), xo[c]);
                load_rhs<NR, true>(a.r + colour(c), ro[c]);
#pragma unroll
                for (int k = 0; k < NR; ++k) {
                    const C q = C{m4 * pv[k].x - acc[c][k].x, m4 * pv[k].y - acc[c][k].y};
                    xo[c][k] = C{xo[c][k].x + alpha[k] * pv[k].x, xo[c][k].y + alpha[k] * pv[k].y};
                    ro[c][k] = C{ro[c][k].x - alpha[k] * q.x, ro[c][k].y - alpha[k] * q.y};
                    if (act[k]) part[0][k] += norm2c<T>(ro[c][k]);
                }
            }
            }
        } else if constexpr (EPI == EPI_RESID) {
            if (any_act) {
#pragma unroll
            for (int c = 0; c < NC; ++c) {
                d2 bv[NR], xv[NR];
                load_rhs<NR>(a.b + colour(c), bv);
                load_rhs<NR>(a.xh + colour(c), xv);
#pragma unroll
                for (int k = 0; k < NR; ++k) {
                    rr[c][k] = d2{bv[k].x - (m4 * xv[k].x - acc[c][k].x),
                                  bv[k].y - (m4 * xv[k].y - acc[c][k].y)};
                    part[0][k] += norm2c<double>(rr[c][k]);
                }
            }
            }
        }
    }

    bool last = false;
    if constexpr (EPI != EPI_PLAIN) last = sum_post<NRHS, NR, M, SPL>(part, a.sum, nblk, bid);

    if (on_site) {
        if constexpr (EPI == EPI_PLAIN || EPI == EPI_NORM) {
#pragma unroll
            for (int c = 0; c < NC; ++c) store_rhs<NR>(a.out + colour(c), acc[c]);
        } else if constexpr (EPI == EPI_CG) {
            if (any_act) {
                // plain stores: L2 merges the partial lines of consecutive
                // store instructions before they reach HBM
#pragma unroll
                for (int c = 0; c < NC; ++c) {
                    store_rhs_on<NR>(a.x + colour(c), xo[c], act);
                    store_rhs_on<NR>(a.r + colour(c), ro[c], act);
                }
            }
        } else if constexpr (EPI == EPI_RESID) {
            if (any_act) {
#pragma unroll
                for (int c = 0; c < NC; ++c)
                    store_rhs_on<NR>(a.out + colour(c), rr[c], act);
            }
        }
    }

    if constexpr (EPI != EPI_PLAIN) {
        if (last) sum_finish<NRHS, M>(a.sum, nblk, bid);
    }
}

#ifdef HISQ_WAVES_PER_EU
#define HISQ_KATTR __attribute__((amdgpu_waves_per_eu(HISQ_WAVES_PER_EU)))
#else
#define HISQ_KATTR
#endif

template <typename T, int NRHS, int NR, int NK, int EPI>
__global__ __launch_bounds__(kMaxBlock) void k_dslash_split(const DslashArgs<T> a)
{
    dslash_tile<T, NRHS, NR, NK, EPI, true, false, 4>(a, a.state, blockIdx.x, gridDim.x, blockIdx.x);
}

template <typename T, int NRHS, int NR, int NK, int EPI, bool CM>
__global__ __launch_bounds__(kMaxBlock) HISQ_KATTR void k_dslash(const DslashArgs<T> a)
{
    const int tile_sites = LaneMap<NRHS, NR, 1>::sites(blockDim.x);
    dslash_tile<T, NRHS, NR, NK, EPI, CM>(
        a, a.state, tile_of_block(blockIdx.x, gridDim.x, a.remap, a.lat, tile_sites), gridDim.x, blockIdx.x);
}

template <typename T, int NRHS, int NR, int NK, int EPI, bool CM>
__global__ __launch_bounds__(kMaxBlockLds) void k_dslash_lds(const DslashArgs<T> a)
{
    extern __shared__ __align__(16) unsigned char hisq_stage[];
    const int sites = a.rows * a.lat.Lh0;
    dslash_tile<T, NRHS, NR, NK, EPI, CM, true>(
        a, a.state, tile_of_block(blockIdx.x, gridDim.x, a.remap, a.lat, sites), gridDim.x, blockIdx.x,
        reinterpret_cast<cplx<T>*>(hisq_stage));
}

// Batched form: one launch covers the tiles of every problem of a BatchTable;
// each work-group finds its problem (uniform scalar search over <= 16 entries)
// and runs the body specialised for that problem's bundle size and tile.
template <typename T, int NK, int EPI>
__global__ __launch_bounds__(kMaxBlock) void k_dslash_batched(const BatchTable<T>* __restrict__ tab, int phase)
{
    int q = 0;
    for (int j = 1; j < tab->nprob; ++j)
        if ((int)blockIdx.x >= tab->p[j].block_start) q = j;
    const BatchProb<T>& bp = tab->p[q];
    const int bid = (int)blockIdx.x - bp.block_start;
    if (bid >= bp.nblocks) return;
    const DslashArgs<T>& a = EPI == EPI_NORM ? bp.k2 : bp.k3;
    const int nb = bp.nblocks;
    CgState* st = bp.state[state_of_phase(phase, 1)];
    // the problem's tile order, on its own block range (the blocks with equal
    // bid mod 8 still share one XCD)
    const int tile = tile_of_block(bid, nb, a.remap, a.lat, (int)blockDim.x / (bp.n / bp.nr));
    switch (bp.n * 16 + bp.nr) {
    case 1 * 16 + 1: dslash_tile<T, 1, 1, NK, EPI, true>(a, st, tile, nb, bid); break;
    case 2 * 16 + 2: dslash_tile<T, 2, 2, NK, EPI, true>(a, st, tile, nb, bid); break;
    case 2 * 16 + 1: dslash_tile<T, 2, 1, NK, EPI, true>(a, st, tile, nb, bid); break;
    case 3 * 16 + 3: dslash_tile<T, 3, 3, NK, EPI, true>(a, st, tile, nb, bid); break;
    case 4 * 16 + 4: dslash_tile<T, 4, 4, NK, EPI, true>(a, st, tile, nb, bid); break;
    case 4 * 16 + 2: dslash_tile<T, 4, 2, NK, EPI, true>(a, st, tile, nb, bid); break;
    case 5 * 16 + 5: dslash_tile<T, 5, 5, NK, EPI, true>(a, st, tile, nb, bid); break;
    case 6 * 16 + 6: dslash_tile<T, 6, 6, NK, EPI, true>(a, st, tile, nb, bid); break;
    case 6 * 16 + 3: dslash_tile<T, 6, 3, NK, EPI, true>(a, st, tile, nb, bid); break;
    case 7 * 16 + 7: dslash_tile<T, 7, 7, NK, EPI, true>(a, st, tile, nb, bid); break;
    case 8 * 16 + 8: dslash_tile<T, 8, 8, NK, EPI, true>(a, st, tile, nb, bid); break;
    case 8 * 16 + 4: dslash_tile<T, 8, 4, NK, EPI, true>(a, st, tile, nb, bid); break;
    default: break;
    }
}

template <typename T, int NK, int EPI, int NRHS, int NR>
static hipError_t go(const Tile& t, DslashArgs<T> a, hipStream_t s, bool cm)
{
    a.ntiles = tile_blocks(a.lat, NRHS, t);
    a.remap = t.remap;
    a.rows = t.rows;
    // each kernel is built for a maximum work-group size; the grid
    // reductions need whole waves
    if (t.bs < 64 || t.bs % 64 != 0 || t.bs > (t.rows > 0 ? kMaxBlockLds : kMaxBlock))
        return hipErrorInvalidValue;
    if (t.split) {
        // one rhs per lane, the kernels of a solve
        if constexpr (NR == 1 && (EPI == EPI_NORM || EPI == EPI_CG || sizeof(T) == 8)) {
            if (!cm || t.rows > 0) return hipErrorInvalidValue;
            hipLaunchKernelGGL((k_dslash_split<T, NRHS, NR, NK, EPI>), dim3(a.ntiles), dim3(t.bs), 0, s, a);
            return hipGetLastError();
        } else {
            return hipErrorInvalidValue;
        }
    }
    if (t.rows > 0) {
        // LDS-staged: the host has checked that a tile is t.rows whole x-rows of
        // one plane and that the rows fit in LDS.  The reducing kernels need the
        // tile to fill its waves, and a site's lanes to divide one.
        const size_t lds = (size_t)3 * (t.rows + 6) * a.lat.Lh0 * NRHS * sizeof(cplx<T>);
        const int used = t.rows * a.lat.Lh0 * (NRHS / NR);
        if (used > t.bs || t.bs - used >= 64) return hipErrorInvalidValue;
        if constexpr (EPI == EPI_PLAIN) {
            if (cm)
                hipLaunchKernelGGL((k_dslash_lds<T, NRHS, NR, NK, EPI, true>), dim3(a.ntiles), dim3(t.bs), lds, s, a);
            else
                hipLaunchKernelGGL((k_dslash_lds<T, NRHS, NR, NK, EPI, false>), dim3(a.ntiles), dim3(t.bs), lds, s, a);
            return hipGetLastError();
        } else if constexpr (64 % (NRHS / NR) == 0) {
            if (!cm || used != t.bs) return hipErrorInvalidValue;
            hipLaunchKernelGGL((k_dslash_lds<T, NRHS, NR, NK, EPI, true>), dim3(a.ntiles), dim3(t.bs), lds, s, a);
            return hipGetLastError();
        } else {
            return hipErrorInvalidValue;
        }
    }
    // the solver's kernels exist in colour-major form only; the plain Dslash in both
    if (cm)
        hipLaunchKernelGGL((k_dslash<T, NRHS, NR, NK, EPI, true>), dim3(a.ntiles), dim3(t.bs), 0, s, a);
    else if constexpr (EPI == EPI_PLAIN)
        hipLaunchKernelGGL((k_dslash<T, NRHS, NR, NK, EPI, false>), dim3(a.ntiles), dim3(t.bs), 0, s, a);
    else
        return hipErrorInvalidValue;
    return hipGetLastError();
}

template <typename T, int NK, int EPI, int NRHS>
static hipError_t pick_nr(const Tile& t, const DslashArgs<T>& a, hipStream_t s, bool cm)
{
    // every divisor of the bundle
    if (t.nr == NRHS) return go<T, NK, EPI, NRHS, NRHS>(t, a, s, cm);
    if constexpr (NRHS % 2 == 0 && NRHS > 2)
        if (t.nr == NRHS / 2) return go<T, NK, EPI, NRHS, NRHS / 2>(t, a, s, cm);
    if constexpr (NRHS % 3 == 0 && NRHS > 3)
        if (t.nr == NRHS / 3) return go<T, NK, EPI, NRHS, NRHS / 3>(t, a, s, cm);
    if constexpr (NRHS == 8)
        if (t.nr == 2) return go<T, NK, EPI, NRHS, 2>(t, a, s, cm);
    if constexpr (NRHS > 1)
        if (t.nr == 1) return go<T, NK, EPI, NRHS, 1>(t, a, s, cm);
    return hipErrorInvalidValue;
}

#define HISQ_CAT2(a, b) a##b
#define HISQ_CAT(a, b) HISQ_CAT2(a, b)
#define HISQ_LAUNCH_NAME HISQ_CAT(HISQ_CAT(HISQ_CAT(launch_dslash_p, HISQ_KPREC), _e), HISQ_KEPI)

hipError_t HISQ_LAUNCH_NAME(int nrhs, const Tile& t, const DslashArgs<KT>& a, hipStream_t s, bool cm)
{
    constexpr int EPI = HISQ_KEPI;
    if constexpr (EPI == EPI_RESID && HISQ_KPREC != 0) {
        return hipErrorInvalidValue;
    } else {
        switch (nrhs) {
        case 1: return pick_nr<KT, kNK, EPI, 1>(t, a, s, cm);
        case 2: return pick_nr<KT, kNK, EPI, 2>(t, a, s, cm);
        case 3: return pick_nr<KT, kNK, EPI, 3>(t, a, s, cm);
        case 4: return pick_nr<KT, kNK, EPI, 4>(t, a, s, cm);
        case 5: return pick_nr<KT, kNK, EPI, 5>(t, a, s, cm);
        case 6: return pick_nr<KT, kNK, EPI, 6>(t, a, s, cm);
        case 7: return pick_nr<KT, kNK, EPI, 7>(t, a, s, cm);
        case 8: return pick_nr<KT, kNK, EPI, 8>(t, a, s, cm);
        default: return hipErrorInvalidValue;
        }
    }
}

#if HISQ_KEPI == 1 || HISQ_KEPI == 2
#define HISQ_BNAME HISQ_CAT(HISQ_CAT(HISQ_CAT(launch_dslash_batched_p, HISQ_KPREC), _e), HISQ_KEPI)
hipError_t HISQ_BNAME(const BatchTable<KT>* tab, int total_blocks, int bs, int phase, hipStream_t s)
{
    // built for at most kMaxBlock threads, whole waves (the grid reductions)
    if (bs < 64 || bs > kMaxBlock || bs % 64 != 0) return hipErrorInvalidValue;
    hipLaunchKernelGGL((k_dslash_batched<KT, kNK, HISQ_KEPI>), dim3(total_blocks), dim3(bs), 0, s,
                       tab, phase);
    return hipGetLastError();
}
#endif

}  // namespace hisq
