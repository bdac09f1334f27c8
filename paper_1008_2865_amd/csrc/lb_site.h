// What every kernel that updates a site shares: the storage policies, the
// pull, the psi stencil, and the force and collision of one site.  Internal
// to the HIP sources.
#pragma once

#include "lb_internal.h"

#include <hip/hip_runtime.h>

namespace lbk {
namespace {

constexpr int kXcds = 8;  // gfx950: 8 XCDs, workgroups dispatched round-robin

// ---------------------------------------------------------------------------
// Storage policies: how a stored population becomes a value of the
// arithmetic type C and back.
// ---------------------------------------------------------------------------
struct PF64 {
    using S = double;
    using C = double;
    static constexpr bool kDev = false;
    __device__ static C ld(const S* p, C) { return *p; }
    __device__ static void st(S* p, C v, C) { *p = v; }
};
struct PF32 {
    using S = float;
    using C = float;
    static constexpr bool kDev = false;
    __device__ static C ld(const S* p, C) { return *p; }
    __device__ static void st(S* p, C v, C) { *p = v; }
};
// Half-precision deviation from the rest-state equilibrium w_i rho', rho'
// within 2^-20 of rho_ref (the offsets of dev_axis_offset).  Decoding is one
// rounding of off + h and encoding one rounding of v - off followed by the
// conversion (the step's collision forms the deviation itself, at tau = 1
// as one fma), in every kernel and at every call site, with contraction
// off, so that the same stored value decodes to the same float everywhere.
struct PF16 {
    using S = _Float16;
    using C = float;
    static constexpr bool kDev = true;
    __device__ static C ld(const S* p, C off)
    {
#pragma clang fp contract(off)
        return off + (C)(*p);
    }
    __device__ static void st(S* p, C v, C off)
    {
#pragma clang fp contract(off)
        C d = v - off;
        asm("" : "+v"(d));  // round d, then convert (never one fused rounding)
        *p = (S)d;
    }
};

// Counter-based hash of (site, step): 32 well-mixed bits (the murmur3
// finaliser applied to a combination of the coordinates).
__device__ __forceinline__ uint32_t site_hash(uint32_t x, uint32_t y, uint32_t t)
{
    uint32_t h = x * 0x9E3779B1u ^ (y + 0x7F4A7C15u) * 0x85EBCA77u ^ (t + 0x165667B1u) * 0xC2B2AE3Du;
    h ^= h >> 16;
    h *= 0x85EBCA6Bu;
    h ^= h >> 13;
    h *= 0xC2B2AE35u;
    h ^= h >> 16;
    return h;
}

template <typename C>
struct CoefT {
    C K1, K2, K4, K5, K8, KE0, tau, omega, sqrt_rho0, inv_rho0, rho_ref;
    C K4x2, K8x2;   // 2 K4 and 2 K8 (the |c_x| = 2 link pairs)
    uint32_t step;  // time step of the launch (seeds the stochastic rounding)
};

template <typename C>
__host__ __device__ CoefT<C> convert(const Coef& c)
{
    return CoefT<C>{(C)c.K1, (C)c.K2, (C)c.K4, (C)c.K5, (C)c.K8, (C)c.KE0,
                    (C)c.tau, (C)c.omega, (C)c.sqrt_rho0, (C)c.inv_rho0,
                    (C)c.rho_ref, (C)(2.0 * c.K4), (C)(2.0 * c.K8), c.step};
}

// Single-precision arithmetic uses the hardware exponential and reciprocal
// (about 1 ulp each; the single-precision path is held to the error the
// rounding of single precision itself produces, far above that).  Double
// precision uses the correctly rounded library functions.
__device__ __forceinline__ double exp_c(double v) { return exp(v); }
__device__ __forceinline__ float exp_c(float v) { return __expf(v); }
__device__ __forceinline__ double rcp_c(double v) { return 1.0 / v; }
__device__ __forceinline__ double fma_c(double a, double b, double c) { return __builtin_fma(a, b, c); }
__device__ __forceinline__ float fma_c(float a, float b, float c) { return __builtin_fmaf(a, b, c); }
__device__ __forceinline__ float rcp_c(float v) { return __builtin_amdgcn_rcpf(v); }

template <typename C>
__device__ __forceinline__ C psi_of(C rho, const CoefT<C>& k)
{
    return k.sqrt_rho0 * ((C)1 - exp_c(-rho * k.inv_rho0));
}

// Periodic wrap for v in [-n, 2n).
__device__ __forceinline__ int wrapi(int v, int n)
{
    v = v < 0 ? v + n : v;
    return v >= n ? v - n : v;
}

// Logical tile of hardware workgroup b: workgroups are dispatched to the
// XCDs round-robin, so give each XCD a contiguous run of logical tiles; the
// vertical neighbours of a tile, whose halo rows it re-reads, then share
// its L2.
__device__ __forceinline__ int xcd_remap(int b, int nb)
{
    const int per = nb / kXcds, rem = nb % kXcds;
    const int xcd = b % kXcds, idx = b / kXcds;
    return xcd < rem ? xcd * (per + 1) + idx
                     : rem * (per + 1) + (xcd - rem) * per + idx;
}

// Deviation offsets w_i rho' of the half storage (zero otherwise), and
// the decoding of a stored value.
template <class P>
struct Offs {
    using S = typename P::S;
    using C = typename P::C;
    C o0, o1, o2;  // rest, axis, diagonal
    C osum;        // o0 + 4 o1 + 4 o2, the offsets of all nine populations
    _Float16 one;  // 1, opaque to the compiler (see ld)
    __device__ Offs(C rho_ref)
    {
#pragma clang fp contract(off)
        // Offsets and their sum exact in single precision (dev_axis_offset).
        if constexpr (P::kDev) {
            static_assert(sizeof(C) == 4, "the half storage computes in single precision");
            o1 = dev_axis_offset(rho_ref);
            o0 = (C)4 * o1;
            o2 = (C)0.25 * o1;
            osum = (C)9 * o1;
        } else {
            o0 = o1 = o2 = osum = (C)0;
        }
        one = (_Float16)1;
        asm("" : "+v"(one));
    }
    __device__ C of(int i) const { return i == 0 ? o0 : (i < 5 ? o1 : o2); }
    // A stored value as the arithmetic type.  Half storage: off + h rounded
    // once, written as the fma h * 1 + off (the product is exact) with a
    // half-precision 1 the compiler cannot fold, so that it becomes a single
    // mixed-precision fma instead of a conversion and an add: the same value.
    __device__ C dec(S v, C off) const
    {
        if constexpr (P::kDev)
            return __builtin_fmaf((float)v, (float)one, off);
        else
            return v;
    }
    __device__ C ld(const S* p, C off) const { return dec(*p, off); }
};

// float -> half with stochastic rounding in hardware: the conversion adds
// random bits (the high bits of r) below the kept mantissa before
// truncating, so it rounds up with probability equal to the dropped
// fraction (unbiased), for normal and subnormal halves alike.
__device__ __forceinline__ _Float16 half_stochastic_hw(float v, uint32_t r)
{
    typedef _Float16 half2_t __attribute__((ext_vector_type(2)));
    const half2_t z = {};
    return __builtin_amdgcn_cvt_sr_f16_f32(z, v, r, false)[0];
}

// Store the nine post-collision populations of one site.  For the half
// storage the moving populations are rounded to nearest, and the rest
// population absorbs their rounding errors (so the stored populations of a
// site sum to its density up to a single rounding) and is itself rounded
// stochastically: at a uniform state every site would otherwise make the
// same rounding error at every step and the total mass would drift.  For
// the half storage q[0] is the density and q[1..8] are already the
// deviations f*_i - w_i rho_ref (site_collide<..., true>).
template <class P>
__device__ __forceinline__ void store_site(typename P::S* const* pd, int at,
                                           const typename P::C q[9],
                                           const Offs<P>& o, uint32_t rnd)
{
    if constexpr (P::kDev) {
        // The rest population is stored as what the rounded moving
        // populations leave of rho, so the nine decoded values sum to rho up
        // to the rounding of the rest itself.
#pragma clang fp contract(off)
        float resid = q[0] - o.osum;
#pragma unroll
        for (int i = 1; i < 9; ++i) {
            // Round the single-precision value, not the exact result of the
            // operation that formed it: the compiler may otherwise fuse that
            // fma with the conversion into one mixed-precision instruction
            // (a single rounding), in some kernels and not in others.
            float v = q[i];
            asm("" : "+v"(v));
            const _Float16 h = (_Float16)v;
            resid = __builtin_fmaf(-(float)h, (float)o.one, resid);  // exact product: resid - h
            pd[i][at] = h;
        }
        pd[0][at] = half_stochastic_hw(resid, rnd);
    } else {
#pragma unroll
        for (int i = 0; i < 9; ++i) P::st(pd[i] + at, q[i], o.of(i));
    }
}

// The element `bytes` after base: a uniform base plus a 32-bit lane offset needs
// no 64-bit vector arithmetic per access.
template <typename T>
__device__ __forceinline__ const T* at32(const T* base, uint32_t bytes)
{
    return reinterpret_cast<const T*>(reinterpret_cast<const char*>(base) + bytes);
}
template <typename T>
__device__ __forceinline__ T* at32(T* base, uint32_t bytes)
{
    return reinterpret_cast<T*>(reinterpret_cast<char*>(base) + bytes);
}

// Pull the nine populations arriving at (x, y): f_i(x, t) = stored_i(x - c_i).
// xm/xp are the periodic columns x-1 / x+1.
template <class P>
__device__ __forceinline__ void pull(const typename P::S* const* pl,
                                     const Geom& g, int x, int xm, int xp,
                                     int y, const Offs<P>& o,
                                     typename P::C f[9])
{
    const int ym = y == 0 ? g.ny - 1 : y - 1;
    const int yp = y == g.ny - 1 ? 0 : y + 1;
    // Offsets inside one plane fit in 32 bits (the host checks it).
    const int r0 = y * g.pitch, rm = ym * g.pitch, rp = yp * g.pitch;
    f[0] = o.ld(pl[0] + r0 + x, o.o0);
    f[1] = o.ld(pl[1] + r0 + xm, o.o1);  // c = ( 1, 0)
    f[2] = o.ld(pl[2] + rm + x, o.o1);   // c = ( 0, 1)
    f[3] = o.ld(pl[3] + r0 + xp, o.o1);  // c = (-1, 0)
    f[4] = o.ld(pl[4] + rp + x, o.o1);   // c = ( 0,-1)
    f[5] = o.ld(pl[5] + rm + xm, o.o2);  // c = ( 1, 1)
    f[6] = o.ld(pl[6] + rm + xp, o.o2);  // c = (-1, 1)
    f[7] = o.ld(pl[7] + rp + xp, o.o2);  // c = (-1,-1)
    f[8] = o.ld(pl[8] + rp + xm, o.o2);  // c = ( 1,-1)
}

template <typename C>
__device__ __forceinline__ C density(const C f[9])
{
    return ((f[0] + (f[1] + f[3])) + (f[2] + f[4])) + ((f[5] + f[7]) + (f[6] + f[8]));
}

__device__ __forceinline__ double wave_sum(double v)
{
#pragma unroll
    for (int m = 32; m >= 1; m >>= 1) v += __shfl_xor(v, m, 64);
    return v;
}

// ---------------------------------------------------------------------------
// The fused step.  Threads = tile_x = NT; LDS ring of 6 psi rows of NT + 4.
// ---------------------------------------------------------------------------

// D2Q9 speed components, population order (0,0) (1,0) (0,1) (-1,0) (0,-1)
// (1,1) (-1,1) (-1,-1) (1,-1), packed two bits per population as c + 1 so a
// lane can look up its own population's speed without a memory table.
constexpr int kQCx[9] = {0, 1, 0, -1, 0, 1, -1, -1, 1};
constexpr int kQCy[9] = {0, 0, 1, 0, -1, 1, 1, -1, -1};
constexpr unsigned pack_speeds(const int* c)
{
    unsigned v = 0;
    for (int i = 0; i < 9; ++i) v |= (unsigned)(c[i] + 1) << (2 * i);
    return v;
}
constexpr unsigned kCxPack = pack_speeds(kQCx);
constexpr unsigned kCyPack = pack_speeds(kQCy);
__device__ __forceinline__ int q_cx(int i) { return (int)((kCxPack >> (2 * i)) & 3u) - 1; }
__device__ __forceinline__ int q_cy(int i) { return (int)((kCyPack >> (2 * i)) & 3u) - 1; }
static_assert(((kCxPack >> 0) & 3u) == 1u && ((kCxPack >> 6) & 3u) == 0u &&
                  ((kCyPack >> 8) & 3u) == 0u && ((kCyPack >> 10) & 3u) == 2u,
              "speed packing");

// psi at the 25 sites of the force stencil around one site, read from five
// rows of a psi ring (rows y-2 .. y+2, LDS column c of the site), named by
// direction: e1 = psi(x+1, y), ne = psi(x+1, y+1), e2n = psi(x+2, y+1), ...
template <typename C>
struct Stencil {
    C p, e1, w1, n1, s1v, ne, nw, sw, se, e2, w2, n2, s2v, e2n, e2s, w2n, w2s, n2e, n2w, s2e, s2w,
        ne2, nw2, sw2, se2;
    __device__ __forceinline__ Stencil(const C* rm2, const C* rm1, const C* rc, const C* rp1,
                                       const C* rp2, int c)
        : p(rc[c]), e1(rc[c + 1]), w1(rc[c - 1]), n1(rp1[c]), s1v(rm1[c]), ne(rp1[c + 1]),
          nw(rp1[c - 1]), sw(rm1[c - 1]), se(rm1[c + 1]), e2(rc[c + 2]), w2(rc[c - 2]),
          n2(rp2[c]), s2v(rm2[c]), e2n(rp1[c + 2]), e2s(rm1[c + 2]), w2n(rp1[c - 2]),
          w2s(rm1[c - 2]), n2e(rp2[c + 1]), n2w(rp2[c - 1]), s2e(rm2[c + 1]), s2w(rm2[c - 1]),
          ne2(rp2[c + 2]), nw2(rp2[c - 2]), sw2(rm2[c - 2]), se2(rm2[c + 2])
    {
    }
};

// Density and momentum of one site's populations.
template <typename C>
struct Moments {
    C rho, jx, jy;
};
template <typename C>
__device__ __forceinline__ Moments<C> moments(const C (&R)[9])
{
#pragma clang fp contract(off)
    return {density(R), (R[1] - R[3]) + ((R[5] - R[7]) + (R[8] - R[6])),
            (R[2] - R[4]) + ((R[5] - R[7]) + (R[6] - R[8]))};
}

// Force of eq. (FORCE) and the velocity-shift BGK collision at one site: R
// the pre-collision populations, m their moments if the caller has them (R is
// then unread at kOm = 1; taken here, after the force, they occupy registers for
// less long), st the psi stencil around the site, Q the
// post-collision populations; with kTape also the tape entry.  For the half
// storage (kDev) Q[0] is the density and Q[1..8] the deviations
// f*_i - w_i rho_ref from the offsets o1 (axis) and o2 (diagonal), which at
// tau = 1 come out of one fma each.  kOm = 1 or 0 states that tau is 1, or
// is not, for a caller that has branched on it already; -1 tests k.omega.
// With mirror the stencil's rows come in the order y+2 .. y-2: every sum of
// the force is then the same value (x) or its exact negative (y).
// Every kernel that updates a site calls this, so all of them round
// identically.
template <bool kTape, bool kDev, int kOm = -1, typename C>
__device__ __forceinline__ void site_collide(const C (&R)[9], const Moments<C>* m, const Stencil<C>& st,
                                             const CoefT<C>& k, C (&Q)[9], C* tp, C o1 = (C)0, C o2 = (C)0,
                                             bool mirror = false)
{
#pragma clang fp contract(off)
    // Multiply-adds are written out as fma and nothing else is contracted,
    // so every kernel variant (launch shape, batched or not, one or two
    // steps per launch, one or two sites per lane) rounds each site's update
    // identically.
    const C p = st.p;
    // eq. (FORCE): F = -psi(x) sum_k K_k psi(x + c_k) c_k, links paired with
    // their opposites.  The differences of opposite links off the axes
    // (|c|^2 = 2, 5, 8) enter both components, so they are formed once.
    const C d2a = st.ne - st.sw, d2b = st.se - st.nw;      // (1, 1), (1,-1)
    const C d8a = st.ne2 - st.sw2, d8b = st.se2 - st.nw2;  // (2, 2), (2,-2)
    const C d5a = st.e2n - st.w2s, d5b = st.e2s - st.w2n;  // (2, 1), (2,-1)
    const C d5c = st.n2e - st.s2w, d5d = st.n2w - st.s2e;  // (1, 2), (-1, 2)
    const C sumx =
        fma_c(k.K1, st.e1 - st.w1,
              fma_c(k.K2, d2a + d2b,
                    fma_c(k.K4x2, st.e2 - st.w2,
                          fma_c(k.K5, fma_c((C)2, d5a + d5b, d5c - d5d), k.K8x2 * (d8a + d8b)))));
    const C sumy =
        fma_c(k.K1, st.n1 - st.s1v,
              fma_c(k.K2, d2a - d2b,
                    fma_c(k.K4x2, st.n2 - st.s2v,
                          fma_c(k.K5, fma_c((C)2, d5c + d5d, d5a - d5b), k.K8x2 * (d8a - d8b)))));
    const C Fx = -p * sumx;
    const C Fy = (mirror ? p : -p) * sumy;

    // BGK collision at u_eq = (j + tau F) / rho.
    const Moments<C> mo = m ? *m : moments(R);
    const C rho = mo.rho, jx = mo.jx, jy = mo.jy;
    if (kTape) {
        tp[0] = rho;
        tp[1] = jx;
        tp[2] = jy;
        tp[3] = p;
    }
    const C inv = rcp_c(rho);
    const C ux = fma_c(k.tau, Fx, jx) * inv;
    const C uy = fma_c(k.tau, Fy, jy) * inv;
    // 1 - 1.5 u^2, and f_eq = w rho (1 - 1.5 u^2 + cu (3 + 4.5 cu)).
    const C base = fma_c((C)-1.5, fma_c(ux, ux, uy * uy), (C)1);
    const C r1 = rho * ((C)1 / (C)9);
    const C r2 = rho * ((C)1 / (C)36);
    auto poly = [&](C cu) { return fma_c(cu, fma_c((C)4.5, cu, (C)3), base); };
    const C pr[9] = {(C)0,        poly(ux),       poly(uy),        poly(-ux), poly(-uy),
                     poly(ux + uy), poly(uy - ux), poly(-ux - uy), poly(ux - uy)};
    auto wr = [&](int i) { return i < 5 ? r1 : r2; };
    auto off = [&](int i) { return i < 5 ? o1 : o2; };
    // f* = f + (f_eq - f) / tau; at tau = 1 (every run of the paper) that is
    // f_eq itself.  The branch is uniform.
    if (kOm == 0 || (kOm < 0 && k.omega != (C)1)) {
        const C om = k.omega;
#pragma unroll
        for (int i = 1; i < 9; ++i) {
            Q[i] = fma_c(om, wr(i) * pr[i] - R[i], R[i]);
            if (kDev) Q[i] = Q[i] - off(i);
        }
    } else {
#pragma unroll
        for (int i = 1; i < 9; ++i) Q[i] = kDev ? fma_c(wr(i), pr[i], -off(i)) : wr(i) * pr[i];
    }
    // The collision conserves mass exactly; the rest population is taken
    // from that, so rounding cannot drift the mass.  The half storage forms
    // it when it rounds the moving populations: there Q[0] carries rho.
    if (kDev)
        Q[0] = rho;
    else
        Q[0] = rho - (((Q[1] + Q[3]) + (Q[2] + Q[4])) + ((Q[5] + Q[7]) + (Q[6] + Q[8])));
}

}  // namespace
}  // namespace lbk
