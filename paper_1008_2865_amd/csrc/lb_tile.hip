// Several time steps of a small lattice in one launch.
//
// A workgroup owns tx x ty sites and advances them `steps` time levels on
// chip.  It pulls the populations of its tile with a halo of 3 steps - 1
// sites from memory, and each step then consumes three sites of halo (two
// for the psi stencil, one for the streaming).  Per step:
//   the densities' psi of every site in reach into LDS | barrier | force and
//   collision of the sites two in from the edge, their post-collision
//   populations into LDS (the last step: to memory) | barrier.
// A thread holds the populations of its sites in registers between the two
// halves, so the LDS planes are overwritten in place.  Every site goes
// through the psi_of, density and site_collide of the one-step kernel, and
// half storage rounds into LDS as a store to memory would, so the fields are
// the same bits for any tile and any number of steps per launch.
//
// What bounds it: on small lattices the launch and the latency of its loads
// (about 4 us, which the steps of a launch share) and the issue of the halo's
// arithmetic, about 1.2 us a step in single and 2 us in double precision; on
// lattices of several tiles per CU the arithmetic, 180 (255) vector
// instructions per site and step, 1.2 to 1.4 times the sites for the halo.  A
// row walk of one step per launch spends 4.6 to 7 us on any small lattice.
// us/step before and after: FP32 64^2 4.4 -> 2.0, 256^2 5.6 -> 2.5, 512^2
// 7.5 -> 4.4, 997x701 12.8 -> 9.2; FP64 64^2 6.4 -> 2.7, 512^2 13.5 -> 7.0,
// 1200^2 44 -> 33, 2048^2 128 -> 95.
#include "lb_site.h"

#include <type_traits>

namespace lbk {
namespace {

// Tile lb of a lattice.  kOm as in site_collide; at 1 a site waits for its
// collision as its three moments instead of its nine populations.
template <class P, int NT, int kPitch, int kRows, bool kTape, int kOm>
__device__ __forceinline__ void
tile_steps(const typename P::S* __restrict__ src, typename P::S* __restrict__ dst, const TileGeom& g, const int steps,
           const CoefT<typename P::C>& k, typename P::C* __restrict__ tape, const int lb)
{
    using S = typename P::S;
    using C = typename P::C;
    constexpr int R = (kPitch * kRows + NT - 1) / NT;  // sites per thread
    constexpr int kPostPitch = kPitch - 4;             // post-collision planes: 2 sites in
    constexpr int kPostPlane = kPostPitch * (kRows - 4);
    extern __shared__ double lds[];
    C* const psi = reinterpret_cast<C*>(lds);
    S* const post = reinterpret_cast<S*>(psi + kPitch * kRows);

    const int tid = threadIdx.x;
    const int sy = lb / g.tiles_x;
    const int x0 = (lb - sy * g.tiles_x) * g.tx, y0 = sy * g.ty;
    const int nx = g.nx, ny = g.ny;
    const Offs<P> o(k.rho_ref);
    const S* pl[9];
    S* pd[9];
    S* lp[9];
#pragma unroll
    for (int i = 0; i < 9; ++i) {
        pl[i] = src + (int64_t)i * g.plane;
        pd[i] = dst + (int64_t)i * g.plane;
        lp[i] = post + i * kPostPlane;
    }

#pragma unroll 1
    for (int j = 0; j < steps; ++j) {
        // Sites in reach of this step: the tile and `halo` more on each side,
        // 3 j in from the first step's region.
        const int halo = 3 * (steps - 1 - j) + 2, in = 3 * j;
        const int w = g.tx + 2 * halo, h = g.ty + 2 * halo, ns = w * h;
        const uint32_t magic = g.magic[steps - 1 - j];
        // Site i of this thread; past the end the last site again (the same
        // values written twice), so that no load is conditional.
        auto site = [&](int i, int& x, int& y) {
            const int s = min(tid + i * NT, ns - 1);
            y = (int)__umulhi((uint32_t)s, magic);
            x = s - y * w;
        };
        C F[R][9];
        Moments<C> M[R];
        if (j == 0) {
#pragma unroll
            for (int i = 0; i < R; ++i) {
                if (i * NT >= ns) break;
                int x, y;
                site(i, x, y);
                const int gx = wrapi(x0 - halo + x, nx), gy = wrapi(y0 - halo + y, ny);
                const int xs[3] = {gx == nx - 1 ? 0 : gx + 1, gx, gx == 0 ? nx - 1 : gx - 1};
                const int r = gy * g.pitch;
                const int ys[3] = {gy == ny - 1 ? 0 : r + g.pitch, r, gy == 0 ? (ny - 1) * g.pitch : r - g.pitch};
#pragma unroll
                for (int q = 0; q < 9; ++q)
                    F[i][q] = o.ld(at32(pl[q], (uint32_t)(ys[1 + kQCy[q]] + xs[1 + kQCx[q]]) * (uint32_t)sizeof(S)), o.of(q));
            }
        } else {
#pragma unroll
            for (int i = 0; i < R; ++i) {
                if (i * NT >= ns) break;
                int x, y;
                site(i, x, y);
                const int at = (y + in - 2) * kPostPitch + x + in - 2;
#pragma unroll
                for (int q = 0; q < 9; ++q) F[i][q] = o.ld(lp[q] + at - kQCy[q] * kPostPitch - kQCx[q], o.of(q));
            }
        }
#pragma unroll
        for (int i = 0; i < R; ++i) {
            if (i * NT >= ns) break;
            int x, y;
            site(i, x, y);
            if (kOm == 1) M[i] = moments(F[i]);
            psi[(y + in) * kPitch + x + in] = psi_of(kOm == 1 ? M[i].rho : density(F[i]), k);
        }
        __syncthreads();

        const bool last = j + 1 == steps;
#pragma unroll
        for (int i = 0; i < R; ++i) {
            if (i * NT >= ns) break;
            int x, y;
            site(i, x, y);
            if (tid + i * NT >= ns || x < 2 || x >= w - 2 || y < 2 || y >= h - 2) continue;
            const int c = (y + in) * kPitch + x + in;
            const Stencil<C> st(psi - 2 * kPitch, psi - kPitch, psi, psi + kPitch, psi + 2 * kPitch, c);
            C q[9], tp[4];
            site_collide<kTape, P::kDev, kOm>(F[i], kOm == 1 ? &M[i] : nullptr, st, k, q, tp, o.o1, o.o2);
            const int ux = x0 - halo + x, uy = y0 - halo + y;  // before the periodic wrap
            const bool own = ux >= x0 && ux < min(x0 + g.tx, nx) && uy >= y0 && uy < min(y0 + g.ty, ny);
            const uint32_t rnd = P::kDev ? site_hash(wrapi(ux, nx), wrapi(uy, ny), k.step + j) : 0u;
            if (!last)
                store_site<P>(lp, (y + in - 2) * kPostPitch + x + in - 2, q, o, rnd);
            else if (own)
                store_site<P>(pd, uy * g.pitch + ux, q, o, rnd);
            if (kTape && own) {
                const int64_t N = (int64_t)nx * ny, at = (int64_t)uy * nx + ux;
#pragma unroll
                for (int v = 0; v < 4; ++v) tape[(4 * j + v) * N + at] = tp[v];
            }
        }
        if (!last) __syncthreads();
    }
}

// Two waves per SIMD in 256 threads: two workgroups fit a CU's LDS.  With one,
// FP64 1200^2 takes 51 us/step instead of 34.
template <class P, int NT, int kPitch, int kRows, bool kTape, int kOm>
__global__ void __launch_bounds__(NT, NT == 256 ? 2 : 1)
k_tile(const typename P::S* __restrict__ src, typename P::S* __restrict__ dst, TileGeom g,
       CoefT<typename P::C> k, typename P::C* __restrict__ tape)
{
    tile_steps<P, NT, kPitch, kRows, kTape, kOm>(src, dst, g, g.steps, k, tape, xcd_remap(blockIdx.x, gridDim.x));
}

// The same for every lattice of a batch: the tiles of all lattices are
// numbered consecutively, tile_lattice gives a tile's lattice.
template <class P, int NT, int kPitch, int kRows, int kOm>
__global__ void __launch_bounds__(NT, NT == 256 ? 2 : 1)
k_tile_batch(const BatchLattice* __restrict__ desc, const int32_t* __restrict__ tile_lattice, int parity,
             uint32_t step, int steps)
{
    using S = typename P::S;
    const int gl = xcd_remap(blockIdx.x, gridDim.x);
    const BatchLattice& d = desc[tile_lattice[gl]];
    CoefT<typename P::C> k;
    if constexpr (sizeof(typename P::C) == 4) {
        const float* c = d.coef_f;
        k = CoefT<float>{c[0], c[1], c[2], c[3], c[4], c[5], c[6], c[7], c[8], c[9], c[10], c[11], c[12], step};
    } else {
        k = convert<double>(d.coef);
        k.step = step;
    }
    tile_steps<P, NT, kPitch, kRows, false, kOm>(static_cast<const S*>(d.buf[parity]),
                                            static_cast<S*>(d.buf[parity ^ 1]), d.tile, steps, k, nullptr,
                                            gl - d.tile_begin3);
}

// LDS of a launch: psi, and with more than one step the post-collision planes.
template <class P, int kPitch, int kRows>
size_t tile_lds(int steps)
{
    constexpr size_t psi = sizeof(typename P::C) * kPitch * kRows;
    constexpr size_t post = sizeof(typename P::S) * 9 * (kPitch - 4) * (kRows - 4);
    return psi + (steps > 1 ? post : 0);
}

// Whether tau = 1 has a kernel of its own.  us/step with one and without: FP32
// 512^2 4.50 and 4.62, 997x701 9.27 and 9.53, half storage 512^2 4.35 and 4.42,
// FP64 in 256 threads 1200^2 33.3 and 34.7, 2048^2 95.0 and 97.8; in 1024 threads,
// which have no register to spare for the moments, FP64 64^2 3.05 and 2.78.
template <typename C, int NT>
constexpr bool kTau1Kernel = sizeof(C) == 4 || NT < 1024;

template <class P, int NT, int kPitch, int kRows, int kOm>
hipError_t tile_nt(const void* src, void* dst, const TileGeom& g, const Coef& c, void* tape, hipStream_t s)
{
    using S = typename P::S;
    using C = typename P::C;
    const auto k = convert<C>(c);
    const S* a = static_cast<const S*>(src);
    S* b = static_cast<S*>(dst);
    const size_t lds = tile_lds<P, kPitch, kRows>(g.steps);
    if (tape) {
        if constexpr (P::kDev)
            return hipErrorInvalidValue;
        else
            hipLaunchKernelGGL((k_tile<P, NT, kPitch, kRows, true, kOm>), dim3(g.tiles), dim3(NT), lds, s, a, b, g, k,
                               static_cast<C*>(tape));
    } else {
        hipLaunchKernelGGL((k_tile<P, NT, kPitch, kRows, false, kOm>), dim3(g.tiles), dim3(NT), lds, s, a, b, g, k,
                           static_cast<C*>(nullptr));
    }
    return hipGetLastError();
}

template <class P, int NT, int kPitch, int kRows>
hipError_t batch_nt(const TileBatch& b, hipStream_t s)
{
    // tau1: tau is 1 in every lattice; else each tile's collision tests its own.
    constexpr int kOm = kTau1Kernel<typename P::C, NT> ? 1 : -1;
    const auto kernel = b.tau1 ? k_tile_batch<P, NT, kPitch, kRows, kOm> : k_tile_batch<P, NT, kPitch, kRows, -1>;
    hipLaunchKernelGGL(kernel, dim3(b.tiles), dim3(NT), (tile_lds<P, kPitch, kRows>(b.steps)), s, b.desc,
                       b.tile_lattice, b.parity, b.step, b.steps);
    return hipGetLastError();
}

template <int W, int H>
struct Region {
    static constexpr int w = W, h = H;
};

// Calls fn with the threads and the region of tiles of tx x ty sites: 34 x 36
// sites keep two double-precision workgroups on a CU, 44 x 46 one.
template <class P, class Fn>
hipError_t with_shape(int threads, int tx, int ty, int steps, Fn&& fn)
{
    const int w = tx + 6 * steps - 2, h = ty + 6 * steps - 2;
    if (steps < 1 || steps > kTileMaxSteps || w > kTilePitch || h > kTileRows) return hipErrorInvalidValue;
    using Small = Region<34, 36>;
    using Large = Region<kTilePitch, kTileRows>;
    const bool small = w <= 34 && h <= 36;
    if (threads == 1024)
        return small ? fn(std::integral_constant<int, 1024>{}, Small{})
                     : fn(std::integral_constant<int, 1024>{}, Large{});
    if constexpr (sizeof(typename P::C) == 8) {
        if (threads == 256 && small) return fn(std::integral_constant<int, 256>{}, Small{});
    } else {
        if (threads == 512)
            return small ? fn(std::integral_constant<int, 512>{}, Small{})
                         : fn(std::integral_constant<int, 512>{}, Large{});
    }
    return hipErrorInvalidValue;
}

template <class P>
hipError_t tile_p(const void* src, void* dst, const TileGeom& g, const Coef& c, void* tape, hipStream_t s)
{
    return with_shape<P>(g.threads, g.tx, g.ty, g.steps, [&](auto nt, auto region) {
        using C = typename P::C;
        if constexpr (!kTau1Kernel<C, nt.value>)
            return tile_nt<P, nt.value, region.w, region.h, -1>(src, dst, g, c, tape, s);
        else
            return (C)c.omega == 1 ? tile_nt<P, nt.value, region.w, region.h, 1>(src, dst, g, c, tape, s)
                                   : tile_nt<P, nt.value, region.w, region.h, 0>(src, dst, g, c, tape, s);
    });
}

template <class P>
hipError_t batch_p(const TileBatch& b, hipStream_t s)
{
    return with_shape<P>(b.threads, b.tx, b.ty, b.steps, [&](auto nt, auto region) {
        return batch_nt<P, nt.value, region.w, region.h>(b, s);
    });
}

}  // namespace

hipError_t launch_tile(int storage, const void* src, void* dst, const TileGeom& g, const Coef& c, void* tape,
                       hipStream_t s)
{
    switch (storage) {
    case ST_F64: return tile_p<PF64>(src, dst, g, c, tape, s);
    case ST_F32: return tile_p<PF32>(src, dst, g, c, tape, s);
    case ST_F16DEV: return tile_p<PF16>(src, dst, g, c, tape, s);
    default: return hipErrorInvalidValue;
    }
}

hipError_t launch_tile_batch(int storage, const TileBatch& b, hipStream_t s)
{
    if (b.tiles <= 0) return hipErrorInvalidValue;
    switch (storage) {
    case ST_F64: return batch_p<PF64>(b, s);
    case ST_F32: return batch_p<PF32>(b, s);
    case ST_F16DEV: return batch_p<PF16>(b, s);
    default: return hipErrorInvalidValue;
    }
}

}  // namespace lbk
