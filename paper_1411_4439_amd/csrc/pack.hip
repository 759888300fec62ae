// Link packing: canonical [4][V][3][3] complex128 U, N -> the per-parity slot
// blocks the Dslash kernels stream (layout described in hisq_internal.h).
//
// For output site z the 16 slots are U_{z,mu}, -U^dag_{z-mu,mu}, N_{z,mu} and
// -N^dag_{z-3mu,mu} (the four terms of Sec. 1 eq. (3), sign folded in).  In r14
// storage a Naik slot keeps rows 0 and 1 and c = <w, row2> / |w|^2 with
// w = conj(row0 x row1), so that row2 = c w exactly when the matrix is a
// positive multiple of a U(3) matrix; the worst relative round-trip error is
// kept in the buffer header (atomicMax on the float's bits, valid for
// non-negative floats).  In r9 storage a Naik slot keeps H = -i log(M / s),
// s = |det M|^(1/3); the header tracks the smallest and largest s, and the
// round trip is checked through the FP32 decoder on the FP32-rounded H.
#include "hisq_device.h"
#include "naik.h"

namespace hisq {

__device__ __forceinline__ d2 cmul_d(d2 a, d2 b)
{
    return d2{a.x * b.x - a.y * b.y, a.x * b.y + a.y * b.x};
}

__device__ __forceinline__ int site_of(const Lat& lat, const int x[4])
{
    return x[0] + lat.L[0] * (x[1] + lat.L[1] * (x[2] + lat.L[2] * x[3]));
}

// The reals that slot S (U: S < 8, Naik: S >= 8) stores for matrix m; for
// compressed Naik storage also the relative error of the round trip, and for r9
// the matrix's scale.
template <int NK, bool NAIK>
__device__ __forceinline__ void encode(const d2 (&m)[9], double (&re)[18], float& err_out, float& scale)
{
    if constexpr (NAIK && NK == HISQ_NAIK_R9) {
        // s = |det M|^(1/3), W = M / s, H = -i log W
        Cx<double> Wm[9];
        for (int e = 0; e < 9; ++e) Wm[e] = Cx<double>{m[e].x, m[e].y};
        const Cx<double> a1 = cx_mul(Wm[4], Wm[8]), a2 = cx_mul(Wm[5], Wm[7]);
        const Cx<double> b1 = cx_mul(Wm[3], Wm[8]), b2 = cx_mul(Wm[5], Wm[6]);
        const Cx<double> g1 = cx_mul(Wm[3], Wm[7]), g2 = cx_mul(Wm[4], Wm[6]);
        const Cx<double> t0 = cx_mul(Wm[0], Cx<double>{a1.re - a2.re, a1.im - a2.im});
        const Cx<double> t1 = cx_mul(Wm[1], Cx<double>{b1.re - b2.re, b1.im - b2.im});
        const Cx<double> t2 = cx_mul(Wm[2], Cx<double>{g1.re - g2.re, g1.im - g2.im});
        const double dre = t0.re - t1.re + t2.re, dim = t0.im - t1.im + t2.im;
        const double sc = cbrt(sqrt(dre * dre + dim * dim));
        double hreal[9];
        double fro = 0, err = 0;
        for (int e = 0; e < 9; ++e) fro += m[e].x * m[e].x + m[e].y * m[e].y;
        if (sc > 0) {
            for (int e = 0; e < 9; ++e) Wm[e] = Cx<double>{m[e].x / sc, m[e].y / sc};
            log_unitary(Wm, hreal);
            float hf[9], ore[9], oim[9];
            for (int e = 0; e < 9; ++e) hf[e] = (float)hreal[e];
            expi_hermitian<float>(hf, (float)sc, ore, oim);
            for (int e = 0; e < 9; ++e) {
                const double dx = ore[e] - m[e].x, dy = oim[e] - m[e].y;
                err += dx * dx + dy * dy;
            }
        } else {
            for (int e = 0; e < 9; ++e) hreal[e] = 0;
            err = fro;
        }
        const double rel = fro > 0 ? sqrt(err / fro) : 0.0;
        err_out = (rel == rel) ? (float)rel : 3.0e38f;
        scale = (float)sc;
        for (int e = 0; e < 9; ++e) re[e] = hreal[e];
    } else if constexpr (NAIK && NK != HISQ_NAIK_FULL) {
        // w = conj(row0 x row1); c = <w, row2> / |w|^2
        d2 w[3];
        w[0] = cmul_d(m[1], m[5]) - cmul_d(m[2], m[4]);
        w[1] = cmul_d(m[2], m[3]) - cmul_d(m[0], m[5]);
        w[2] = cmul_d(m[0], m[4]) - cmul_d(m[1], m[3]);
        for (int j = 0; j < 3; ++j) w[j].y = -w[j].y;
        d2 num = d2{0, 0};
        double den = 0, fro = 0, err = 0;
        for (int j = 0; j < 3; ++j) {
            num += cmul_d(d2{w[j].x, -w[j].y}, m[6 + j]);
            den += w[j].x * w[j].x + w[j].y * w[j].y;
        }
        d2 cc = den > 0 ? d2{num.x / den, num.y / den} : d2{0, 0};
        double phi = 0;
        if constexpr (NK == HISQ_NAIK_R13) {
            // r13 keeps only the phase; the modulus is 1 / |row0|
            phi = atan2(cc.y, cc.x);
            const double r0 = sqrt(m[0].x * m[0].x + m[0].y * m[0].y + m[1].x * m[1].x +
                                   m[1].y * m[1].y + m[2].x * m[2].x + m[2].y * m[2].y);
            cc = r0 > 0 ? d2{cos(phi) / r0, sin(phi) / r0} : d2{0, 0};
        }
        for (int e = 0; e < 9; ++e) fro += m[e].x * m[e].x + m[e].y * m[e].y;
        for (int j = 0; j < 3; ++j) {
            const d2 d = m[6 + j] - cmul_d(cc, w[j]);
            err += d.x * d.x + d.y * d.y;
        }
        const double rel = fro > 0 ? sqrt(err / fro) : 0.0;
        err_out = (rel == rel) ? (float)rel : 3.0e38f;
        for (int e = 0; e < 6; ++e) {
            re[2 * e] = m[e].x;
            re[2 * e + 1] = m[e].y;
        }
        re[12] = NK == HISQ_NAIK_R14 ? cc.x : phi;
        re[13] = cc.y;
    } else {
        for (int e = 0; e < 9; ++e) {
            re[2 * e] = m[e].x;
            re[2 * e + 1] = m[e].y;
        }
    }
}

// Site i's NR reals of one slot, 16 bytes per store.  FP32: reals group into 16-byte
// words, [r / 4][Vh][4], so that one load brings two complex numbers; the NR % 4
// remaining reals follow as a plane [Vh][NR % 4].  FP64: [element][Vh] complex.  Slot
// starts stay 16-byte aligned because Vh is a multiple of 8.
template <typename T, int NR>
__device__ __forceinline__ void store_slot(T* slot, int Vh, int i, const double (&re)[18])
{
    if constexpr (sizeof(T) == 4) {
        constexpr int nw = NR / 4, rem = NR % 4;
        f4* wp = reinterpret_cast<f4*>(slot) + i;
#pragma unroll
        for (int w = 0; w < nw; ++w)
            wp[(size_t)w * Vh] = f4{(float)re[4 * w], (float)re[4 * w + 1], (float)re[4 * w + 2], (float)re[4 * w + 3]};
        T* tail = slot + (size_t)4 * nw * Vh;
        if constexpr (rem == 2)
            reinterpret_cast<f2*>(tail)[i] = f2{(float)re[4 * nw], (float)re[4 * nw + 1]};
        else if constexpr (rem == 1)
            tail[i] = (float)re[4 * nw];
    } else {
        d2* lp = reinterpret_cast<d2*>(slot) + i;
#pragma unroll
        for (int e = 0; e < 9; ++e) lp[(size_t)e * Vh] = d2{re[2 * e], re[2 * e + 1]};
    }
}

// Largest (smallest) of non-negative floats over the wave, by their bits, into a
// header word.  As integers, not as floats: fmaxf and fminf drop a NaN, the bits of
// one exceed every finite float's, so that a NaN scale (a NaN link) reaches the
// header and the host refuses the field.  Waves whose value is no larger than what
// they find there issue no atomic: atomics on one address are served one after another.
__device__ __forceinline__ void header_max(uint32_t* word, uint32_t bits)
{
#pragma unroll
    for (int off = 32; off >= 1; off >>= 1) bits = max(bits, (uint32_t)__shfl_xor((int)bits, off, 64));
    if ((threadIdx.x & 63) == 0 && bits > __hip_atomic_load(word, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT))
        atomicMax(word, bits);
}
__device__ __forceinline__ void header_min(uint32_t* word, uint32_t bits)
{
#pragma unroll
    for (int off = 32; off >= 1; off >>= 1) bits = min(bits, (uint32_t)__shfl_xor((int)bits, off, 64));
    if ((threadIdx.x & 63) == 0 && bits < __hip_atomic_load(word, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT))
        atomicMin(word, bits);
}

// One thread per link: it reads the link once and writes both of its uses, the
// forward slot at its root z and the backward slot, -W^dag, at z + h mu (the
// other parity's block).  The links of kPackSites consecutive sites of one
// direction are one contiguous stretch, which the work-group copies to LDS with
// 16-byte loads; consecutive sites alternate between the parity blocks, so the
// 16-byte stores of a wave are two contiguous runs of 512 bytes.  What bounds
// it: the bytes, V (1152 read + 2304 written in FP64, 1024 in r14): 32^3 x 8 takes
// 159 us in FP64 (5.7 TB/s) and 115-126 us in r14.  One thread per output site,
// reading every link twice at a 144-byte stride and storing single reals, took
// 259 and 205 us.
constexpr int kPackSites = 256;

template <typename T, int NK, bool NAIK>
__device__ __forceinline__ void pack_link(const Lat& lat, const d2 (&m)[9], int mu, const int (&c)[4],
                                          T* __restrict__ out, bool on, uint32_t& worst, uint32_t& smin, uint32_t& smax)
{
    constexpr int NR = NAIK ? naik_reals(NK) : 18;
    constexpr int h = NAIK ? 3 : 1;
    const int Vh = lat.Vh;
    const int P = (c[0] + c[1] + c[2] + c[3]) & 1;
    int y[4] = {c[0], c[1], c[2], c[3]};
#pragma unroll
    for (int nu = 0; nu < 4; ++nu)
        if (nu == mu) y[nu] = (c[nu] + h) % lat.L[nu];
    worst = 0u;
    smin = 0x7f800000u;  // +inf
    smax = 0u;
    if (!on) return;
#pragma unroll
    for (int back = 0; back < 2; ++back) {
        d2 w[9];
#pragma unroll
        for (int a = 0; a < 3; ++a)
#pragma unroll
            for (int b = 0; b < 3; ++b)
                w[3 * a + b] = back ? d2{-m[3 * b + a].x, m[3 * b + a].y} : m[3 * a + b];
        double re[18];
        float err = 0.0f, sc = 0.0f;
        encode<NK, NAIK>(w, re, err, sc);
        T* blk = out + (size_t)(back ? 1 - P : P) * link_block_reals(Vh, NK);
        const int slot = (NAIK ? 8 : 0) + 4 * back + mu;
        store_slot<T, NR>(blk + (size_t)slot_real_start(slot, NK) * Vh, Vh,
                          site_of(lat, back ? y : c) >> 1, re);
        worst = max(worst, __float_as_uint(err));
        smin = min(smin, __float_as_uint(sc));
        smax = max(smax, __float_as_uint(sc));
    }
}

template <typename T, int NK>
__global__ __launch_bounds__(kPackSites) void k_pack(Lat lat, const d2* __restrict__ U, const d2* __restrict__ N,
                                                     T* __restrict__ out, LinkHeader* hdr)
{
    __shared__ d2 sm[kPackSites * 9];
    const int V = 2 * lat.Vh;
    const int mu = blockIdx.y & 3;
    const bool naik = blockIdx.y >= 4;
    const int s0 = blockIdx.x * kPackSites;
    const int ns = min(kPackSites, V - s0);
    const d2* src = (naik ? N : U) + ((size_t)mu * V + s0) * 9;
    for (int q = threadIdx.x; q < ns * 9; q += kPackSites) sm[q] = __builtin_nontemporal_load(src + q);
    __syncthreads();
    const bool on = (int)threadIdx.x < ns;
    const int s = s0 + (on ? (int)threadIdx.x : 0);
    int c[4], r = s;
#pragma unroll
    for (int nu = 0; nu < 3; ++nu) {
        c[nu] = r % lat.L[nu];
        r /= lat.L[nu];
    }
    c[3] = r;
    d2 m[9];
#pragma unroll
    for (int e = 0; e < 9; ++e) m[e] = sm[(s - s0) * 9 + e];
    uint32_t worst, smin, smax;
    if (!naik) {
        pack_link<T, NK, false>(lat, m, mu, c, out, on, worst, smin, smax);
    } else {
        pack_link<T, NK, true>(lat, m, mu, c, out, on, worst, smin, smax);
        if constexpr (NK != HISQ_NAIK_FULL) header_max(&hdr->naik_err_bits, worst);
        if constexpr (NK == HISQ_NAIK_R9) {
            header_min(&hdr->scale_min_bits, smin);
            header_max(&hdr->scale_max_bits, smax);
        }
    }
}

__global__ void k_pack_header(LinkHeader h, LinkHeader* dst) { *dst = h; }

hipError_t launch_pack(const Lat& lat, const d2* U, const d2* N, int prec, int naik, void* packed,
                       hipStream_t s)
{
    LinkHeader h{};
    h.magic = kLinkMagic;
    for (int mu = 0; mu < 4; ++mu) h.L[mu] = lat.L[mu];
    h.prec = prec;
    h.naik = naik;
    h.naik_err_bits = 0u;
    h.scale_min_bits = 0x7f800000u;  // +inf
    h.scale_max_bits = 0u;
    h.naik_scale = 1.0f;
    LinkHeader* hdr = reinterpret_cast<LinkHeader*>(packed);
    hipLaunchKernelGGL(k_pack_header, dim3(1), dim3(1), 0, s, h, hdr);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    char* body = reinterpret_cast<char*>(packed) + kLinkHeaderBytes;
    const int V = 2 * lat.Vh;
    const dim3 grid((V + kPackSites - 1) / kPackSites, 8), block(kPackSites);
    if (prec == HISQ_PREC_F64)
        hipLaunchKernelGGL((k_pack<double, HISQ_NAIK_FULL>), grid, block, 0, s, lat, U, N,
                           reinterpret_cast<double*>(body), hdr);
    else if (naik == HISQ_NAIK_R14)
        hipLaunchKernelGGL((k_pack<float, HISQ_NAIK_R14>), grid, block, 0, s, lat, U, N,
                           reinterpret_cast<float*>(body), hdr);
    else if (naik == HISQ_NAIK_R13)
        hipLaunchKernelGGL((k_pack<float, HISQ_NAIK_R13>), grid, block, 0, s, lat, U, N,
                           reinterpret_cast<float*>(body), hdr);
    else if (naik == HISQ_NAIK_R9)
        hipLaunchKernelGGL((k_pack<float, HISQ_NAIK_R9>), grid, block, 0, s, lat, U, N,
                           reinterpret_cast<float*>(body), hdr);
    else
        hipLaunchKernelGGL((k_pack<float, HISQ_NAIK_FULL>), grid, block, 0, s, lat, U, N,
                           reinterpret_cast<float*>(body), hdr);
    return hipGetLastError();
}

}  // namespace hisq
