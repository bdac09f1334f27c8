// HIP kernels of the two-belt Shan-Chen lattice Boltzmann step for gfx950.
//
// Plain steps run several per launch: on large lattices and in tiles of the
// caller's own two in k_step2 below, else in the tiles of lb_tile.hip.  k_step
// runs the logged steps, the steps left over, those asked for one per launch,
// tiles of the caller's own in double precision, and lattices whose tiles would
// hold few sites.  It performs one full time step of eq. (1) of the paper for a
// strip of the lattice in a single pass over HBM:
//   pull-stream (read each population once from its upstream site),
//   moments, psi(rho), the 24-link two-belt force of eq. (FORCE),
//   BGK collision at the force-shifted velocity, and a coalesced store.
// The psi values the force needs (a 5x5 neighbourhood) are staged in a ring
// of six LDS rows: each workgroup owns `tile_x` columns (one per lane) and
// walks down `tile_y` rows; for every row it pulls the populations two rows
// ahead, turns them into psi for its columns plus a 2-column halo, and then
// evaluates force and collision for the row whose +-2 neighbourhood is
// complete.  The populations of the two rows in between stay in registers,
// so every population is read from HBM once per step except for the
// 2-row/2-column halo, whose re-reads hit L2.
//
// The same kernel optionally accumulates the section V observables
// (mass, E_s, E_m, sum psi^2) of the pre-collision state in double:
// per-lane sums, a 64-lane xor-shuffle tree, a fixed-order sum over the
// waves of the workgroup, one partial per workgroup, and a single-workgroup
// fixed-order final reduction (k_final).  No floating-point atomics are
// used, so results are bit-reproducible for a given launch shape.
#include "lb_site.h"

#include <algorithm>
#include <map>
#include <mutex>
#include <tuple>
#include <type_traits>

namespace lbk {
namespace {

template <int J>
using Ic = std::integral_constant<int, J>;

// Lookahead of the row walk: the loads of a row are issued LEAD
// iterations before its psi is staged.  LEAD = 2 keeps two rows of loads in
// flight per wave (about 10 more registers in single precision, still 4
// waves per SIMD); its longer prologue only pays off on tall tiles.
constexpr int kLead2MinRows = 16;

// Plain steps of single-precision arithmetic with one row per stage have a
// LEAD = 2 variant.
template <class P, int RPI>
constexpr bool lead2_variant()
{
    return sizeof(typename P::C) == 4 && RPI == 1;
}

// One launch = one time step for a tile of NT columns (one lane each) by
// tile_y rows, walked RPI rows at a time.
template <class P, int NT, int MODE, int RPI, int LEAD>
__device__ __forceinline__ void
step_tile(const typename P::S* __restrict__ src, typename P::S* __restrict__ dst,
          const Geom& g, const CoefT<typename P::C>& k, double* __restrict__ partials,
          const int lb)
{
    using S = typename P::S;
    using C = typename P::C;
    constexpr bool kEnergy = MODE == MODE_STEP_ENERGY || MODE == MODE_ENERGY;
    constexpr bool kCollide = MODE != MODE_ENERGY;
    constexpr bool kTape = MODE == MODE_STEP_TAPE;
    constexpr int LW = NT + 4;
    constexpr int kWaves = NT / 64;
    constexpr int kHpw = 4 / kWaves;  // halo columns gathered per wave
    // psi ring: walk rows -2 .. RPI+1 around the rows being updated, plus
    // RPI rows being staged.  Population buffers: the RPI rows being
    // updated, the 2 rows after them (psi staged) and RPI lead rows whose
    // loads are in flight.
    constexpr int RS = 4 + 2 * RPI;
    constexpr int NB = 2 + RPI * (1 + LEAD);
    constexpr int U = NB / RPI;
    static_assert(NB % RPI == 0, "buffer rotation must be a whole number of iterations");
    static_assert(U <= 6, "the walk loop is unrolled at most 6 times");
    __shared__ C ring[RS][LW];

    const int tid = threadIdx.x;
    const int lane = tid & 63;
    const int wid = tid >> 6;
    const int sx = lb % g.tiles_x;
    const int sy = lb / g.tiles_x;
    const int x0 = sx * NT;
    const int y0 = sy * g.tile_y;
    const int y1 = min(y0 + g.tile_y, g.ny);
    // Vertically adjacent tiles walk in opposite directions, so the rows
    // at a shared tile boundary are pulled by both tiles at about the same
    // time (both at the start or both at the end of their walk) and the
    // second pull of those halo rows is served by L2.
    const int dir = (sy & 1) ? -1 : 1;
    const int ystart = dir > 0 ? y0 : y1 - 1;
    const int nrows = y1 - y0;
    const int nx = g.nx, ny = g.ny;
    // Lattice row of walk row r (r may run up to 2 rows past either end).
    auto wrow = [&](int r) { return wrapi(ystart + r * dir, ny); };

    const S* pl[9];
    S* pd[9];
#pragma unroll
    for (int i = 0; i < 9; ++i) {
        pl[i] = src + (int64_t)i * g.plane;
        pd[i] = dst + (int64_t)i * g.plane;
    }
    const Offs<P> o(k.rho_ref);

    // This lane's column, LDS column tid + 2.
    const bool own = x0 + tid < nx;
    const int xc = (x0 + tid) % nx;
    const int xcm = xc == 0 ? nx - 1 : xc - 1;
    const int xcp = xc == nx - 1 ? 0 : xc + 1;

    // Halo: the 4 columns x0-2, x0-1, x0+NT, x0+NT+1 (LDS 0, 1, NT+2, NT+3).
    // Each wave gathers kHpw of them with a single load instruction per row:
    // lane j < 9 kHpw fetches population j % 9 of halo column j / 9 (the
    // other lanes repeat the last address), and the nine values are then
    // summed across lanes.  No lane-divergent loads.
    const int hj = lane < 9 * kHpw ? lane : 9 * kHpw - 1;
    const int hi = hj % 9;
    const int hcol = wid * kHpw + hj / 9;
    const int hlds = hcol < 2 ? hcol : NT + hcol;
    int hgx = (x0 - 2 + hlds - q_cx(hi)) % nx;
    hgx = hgx < 0 ? hgx + nx : hgx;
    const S* hp = src + (int64_t)hi * g.plane + hgx;
    const int hcy = q_cy(hi);
    const C hoff = o.of(hi);
    const int mcol = wid * kHpw + (lane < kHpw ? lane : 0);
    const int mlds = mcol < 2 ? mcol : NT + mcol;
    const int gbase = 9 * (lane < kHpw ? lane : 0);

    auto halo_load = [&](int y) -> C {
        // Row y - c_y of this lane's population, from the three row offsets
        // every lane of the wave shares.
        const int ym = y == 0 ? ny - 1 : y - 1;
        const int yp = y == ny - 1 ? 0 : y + 1;
        const int r = (hcy > 0 ? ym : (hcy < 0 ? yp : y)) * g.pitch;
        return o.ld(hp + r, hoff);
    };
    auto halo_psi = [&](C hv, int slot) {
        C h[9];
#pragma unroll
        for (int m = 0; m < 9; ++m) h[m] = __shfl(hv, gbase + m, 64);
        const C ps = psi_of(density(h), k);
        if (lane < kHpw) ring[slot][mlds] = ps;
    };

    // Walk row r lives in buffer r % NB (its halo value in Hh[r % NB]).
    // Each loop iteration advances RPI rows and the loop body is unrolled
    // U = NB / RPI times, so every
    // buffer index below is a compile-time constant: the rotation is a
    // renaming, never a register copy (a copy of a register whose load may
    // still be outstanding would force a wait on the memory counter, which
    // on this target also counts the stores just issued).
    C Bf[NB][9] = {};
    C Hh[NB] = {};

    // Prologue: psi of walk rows -2 .. RPI+1 into ring slots 0 .. RPI+3, the
    // populations of rows 0 .. RPI+1 into Bf[0 .. RPI+1], and the loads of
    // the first LEAD-1 stages of lead rows.  All rows are requested before
    // any is used, so the prologue costs one latency.
    {
        C T0[9], T1[9], hv[RPI + 4];
        pull<P>(pl, g, xc, xcm, xcp, wrow(-2), o, T0);
        pull<P>(pl, g, xc, xcm, xcp, wrow(-1), o, T1);
#pragma unroll
        for (int r = 0; r < RPI + 2; ++r) pull<P>(pl, g, xc, xcm, xcp, wrow(r), o, Bf[r]);
#pragma unroll
        for (int r = -2; r < RPI + 2; ++r) hv[r + 2] = halo_load(wrow(r));
#pragma unroll
        for (int r = RPI + 2; r < 2 + RPI * LEAD; ++r) {
            const int yl = r < nrows + 2 ? wrow(r) : wrow(0);
            pull<P>(pl, g, xc, xcm, xcp, yl, o, Bf[r % NB]);
            Hh[r % NB] = halo_load(yl);
        }
        ring[0][tid + 2] = psi_of(density(T0), k);
        ring[1][tid + 2] = psi_of(density(T1), k);
#pragma unroll
        for (int r = 0; r < RPI + 2; ++r) ring[r + 2][tid + 2] = psi_of(density(Bf[r]), k);
#pragma unroll
        for (int r = 0; r < RPI + 4; ++r) halo_psi(hv[r], r);
    }

    double aM = 0.0, aEs = 0.0, aEm = 0.0, aS2 = 0.0;

    // Software pipeline, per iteration (rows b .. b+RPI-1 along the walk):
    //   issue the loads of the rows LEAD stages ahead, b+2+RPI*LEAD .. |
    //   barrier | force + collision of rows b .. b+RPI-1 | psi of rows
    //   b+RPI+2 .. b+2RPI+1 (loaded LEAD-1 iterations ago) into the ring
    //   slots of rows b-RPI-2 .. b-3 | stores.
    // The loads overlap LEAD barriers and rounds of arithmetic; the stores
    // overlap the next iteration's barrier and arithmetic.  The overwritten
    // slots were last read in the previous iteration, before this barrier.
    // Lead rows past the end of the walk re-read row b instead (an L2 hit),
    // so no load is conditional.
    auto group = [&](auto Jc, int it, int s0) {
        constexpr int J = decltype(Jc)::value;
        const int b = it * RPI;
#pragma unroll
        for (int m = 0; m < RPI; ++m) {
            const int r = b + 2 + RPI * LEAD + m;
            const int yl = r < nrows + 2 ? wrow(r) : wrow(b);
            pull<P>(pl, g, xc, xcm, xcp, yl, o, Bf[(J * RPI + 2 + RPI * LEAD + m) % NB]);
            Hh[(J * RPI + 2 + RPI * LEAD + m) % NB] = halo_load(yl);
        }
        __syncthreads();

        C q[RPI][9];
        C tp[RPI][4];  // tape entry (MODE_STEP_TAPE)
        C anchor = (C)0;
#pragma unroll
        for (int m = 0; m < RPI; ++m) {
            const C(&R)[9] = Bf[(J * RPI + m) % NB];
            if (m > 0 && b + m >= nrows) break;
            // Ring rows y-2 .. y+2 of lattice row y = walk row b+m.
            auto slot = [&](int dy) {
                int v = s0 + m + 2 + dy * dir;
                return v >= RS ? v - RS : v;
            };
            const C* rm2 = ring[slot(-2)];
            const C* rm1 = ring[slot(-1)];
            const C* rc = ring[slot(0)];
            const C* rp1 = ring[slot(1)];
            const C* rp2 = ring[slot(2)];
            const int c = tid + 2;

            const Stencil<C> st(rm2, rm1, rc, rp1, rp2, c);
            const C p = st.p;

            if (kEnergy && own) {
                // No contraction here: the energies must round identically
                // in every kernel variant that computes them (the step
                // that also logs, the energy-only pass, the batched kernel).
#pragma clang fp contract(off)
                const C S1 = (st.e1 + st.w1) + (st.n1 + st.s1v);
                const C S2 = (st.ne + st.sw) + (st.nw + st.se);
                const C S4 = (st.e2 + st.w2) + (st.n2 + st.s2v);
                const C S5 = ((st.e2n + st.w2s) + (st.e2s + st.w2n)) + ((st.n2e + st.s2w) + (st.n2w + st.s2e));
                const C S8 = (st.ne2 + st.sw2) + (st.nw2 + st.se2);
                const C es = (C)0.5 * p * (k.KE0 * p + k.K1 * S1 + k.K2 * S2);
                const C em = (C)0.5 * p * (k.K4 * S4 + k.K5 * S5 + k.K8 * S8);
                aM += (double)density(R);
                aEs += (double)es;
                aEm += (double)em;
                aS2 += (double)p * (double)p;
            }

            if (kCollide) {
                site_collide<kTape, P::kDev>(R, (const Moments<C>*)nullptr, st, k, q[m], tp[m], o.o1, o.o2);
                if (m == 0) anchor = q[m][1];
            } else if (m == 0) {
                anchor = p;
            }
        }

        // Stage psi of the lead rows (their loads have had the barrier and
        // the arithmetic above to arrive).  Rows past the end of the walk
        // write slots nobody reads any more.  The empty asm statements tie
        // the lead-row registers to the result of the arithmetic, so the
        // compiler cannot hoist this staging (and the wait for those loads)
        // above the arithmetic; the fence after it keeps the stores below,
        // so the wait does not also cover this iteration's stores.
#pragma unroll
        for (int m = 0; m < RPI; ++m) {
            C(&NF)[9] = Bf[(J * RPI + RPI + 2 + m) % NB];
            C& HF = Hh[(J * RPI + RPI + 2 + m) % NB];
#pragma unroll
            for (int i = 0; i < 9; ++i) asm volatile("" : "+v"(NF[i]) : "v"(anchor));
            asm volatile("" : "+v"(HF) : "v"(anchor));
            int sl = s0 + RPI + 4 + m;
            sl = sl >= RS ? sl - RS : sl;
            ring[sl][tid + 2] = psi_of(density(NF), k);
            halo_psi(HF, sl);
        }
        __builtin_amdgcn_sched_barrier(0);

        if (kCollide && own) {
#pragma unroll
            for (int m = 0; m < RPI; ++m) {
                if (m > 0 && b + m >= nrows) break;
                const int yw = wrow(b + m);
                const uint32_t rnd = P::kDev ? site_hash(xc, yw, k.step) : 0u;
                store_site<P>(pd, yw * g.pitch + xc, q[m], o, rnd);
                if (kTape) {
                    C* tape = reinterpret_cast<C*>(partials);
                    const int64_t N = (int64_t)nx * ny, si = (int64_t)yw * nx + xc;
#pragma unroll
                    for (int v = 0; v < 4; ++v) tape[v * N + si] = tp[m][v];
                }
            }
        }
    };

    auto step_slot = [](int s) { return s + RPI >= RS ? s + RPI - RS : s + RPI; };
    int s0 = 0;  // ring slot of walk row b - 2
#pragma unroll 1
    for (int it = 0;;) {
        group(Ic<0>{}, it, s0);
        s0 = step_slot(s0);
        if (++it * RPI >= nrows) break;
        group(Ic<1 % U>{}, it, s0);
        s0 = step_slot(s0);
        if (++it * RPI >= nrows) break;
        group(Ic<2 % U>{}, it, s0);
        s0 = step_slot(s0);
        if (++it * RPI >= nrows) break;
        if constexpr (U >= 4) {
            group(Ic<3 % U>{}, it, s0);
            s0 = step_slot(s0);
            if (++it * RPI >= nrows) break;
        }
        if constexpr (U >= 5) {
            group(Ic<4 % U>{}, it, s0);
            s0 = step_slot(s0);
            if (++it * RPI >= nrows) break;
        }
        if constexpr (U >= 6) {
            group(Ic<5 % U>{}, it, s0);
            s0 = step_slot(s0);
            if (++it * RPI >= nrows) break;
        }
    }

    if (kEnergy) {
        __shared__ double red[4][kWaves];
        double v[4] = {aM, aEs, aEm, aS2};
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            v[q] = wave_sum(v[q]);
            if (lane == 0) red[q][wid] = v[q];
        }
        __syncthreads();
        if (tid < 4) {
            double s = 0.0;
            for (int w = 0; w < kWaves; ++w) s += red[tid][w];
            partials[(int64_t)lb * 4 + tid] = s;
        }
    }
}

// ---------------------------------------------------------------------------
// Two time steps per launch (temporal blocking) for plain steps of the
// single-precision and half storages.  A tile of NT lanes produces NT - 6
// output columns x0 .. x0+W-1 of step t+2 for tile_y rows.  Level 1 is the one-step row walk above on the
// NT columns x0-3 .. x0+NT-4 and on rows -3 .. nrows+2 of the tile (walk
// order); its post-collision rows go to a 4-row LDS ring instead of memory.
// Level 2 trails it: at walk row p it pulls the pre-collision populations of
// row p-2 at t+1 from that ring (rows p-3 .. p-1, lanes l-1 .. l+1), stages
// their psi, and, after the row's barrier, applies the same force and
// collision (site_collide, so every site rounds as in two one-step
// launches) to row p-4, which it stores.  One barrier per walk row: every
// LDS row an iteration reads was written before the previous barrier, and
// the slots written between two barriers are not read between them (the
// rings are deep enough).  Global traffic per two steps is one read and one
// write of the populations, plus halo rows and columns that neighbouring
// tiles also read.
//
// Neighbouring tiles walk in opposite directions, so that they reach a shared
// halo together, and every tile turns round from one launch to the next: the
// rows a launch wrote last are read first while the memory-side cache holds them
// (FP32 3000^2 80.5 -> 73.7 us per step, 4096^2 141.5 -> 136.1; reversing the
// order of the tiles as well gains nothing).
//
// What bounds it: single precision, memory (2048^2 79 us per launch whether 6 or
// 3 workgroups are resident on a CU, 4.4 TB/s of fabric traffic); half storage,
// the vector ALU and the latency of a row.  So a row's loads are issued before
// all else and waited for after the row's arithmetic, slots are constants, only
// three moments of a waiting row are kept at tau = 1, addresses are a uniform
// base and a 32-bit lane offset, and a halo column's density is summed by lane
// shifts.  us per step before and after all of these and the turning: FP32
// 2048^2 40.0 -> 38.9, 3000^2 80.3 -> 72.7, 4096^2 141.2 -> 136.5; half storage
// 2048^2 31.2 -> 27.4, 4096^2 (tau 0.8) 116.5 -> 102, 8192^2 416 -> 362.
// ---------------------------------------------------------------------------
// LDS of a two-step workgroup, declared once per kernel so that the walks
// for tau = 1 and for other tau share it.  The rings are powers of two and
// the walk is unrolled by their length, so that every slot is a constant.  At
// 128 lanes in single precision that is 26880 bytes: six workgroups fit on a CU.
template <class P, int NT>
struct Step2Smem {
    static constexpr int U = 8, NF = 4;
    // fs lies between the rings: lanes -1 and NT of its first and last row,
    // which lanes 0 and NT - 1 read for values no output uses, are there.
    typename P::C ring[U][NT + 4];  // psi at t: level-1 row r in slot r + 5
    // Post-collision populations of step t+1, in the storage type and
    // rounded exactly as a one-step launch stores them: row r in slot r + 4.
    typename P::S fs[NF][9][NT];
    typename P::C ring2[U][NT + 4];  // psi at t+1: row r in slot r + 5
};

// Issue priority of a wave for one walk row.  Among waves of equal
// priority the arbiter picks the oldest, so the workgroups a CU receives
// first run ahead of the ones it receives last, which then finish alone
// (timed per workgroup at 2048^2: 61 us for the first resident slot, 74 us
// for the last, against an 82 us launch).  Drawing each row's priority from
// a hash of the row and the workgroup keeps any wave from holding the lead:
// launches 0.4% (2048^2) to 1.7% (half storage 8192^2) shorter.  The
// priority orders issue only; results are unaffected.
__device__ __forceinline__ void set_row_priority(int it)
{
    const uint32_t h = ((uint32_t)it * 0x9E3779B1u + blockIdx.x * 0x85EBCA77u) >> 30;
    switch (h) {
    case 0: __builtin_amdgcn_s_setprio(0); break;
    case 1: __builtin_amdgcn_s_setprio(1); break;
    case 2: __builtin_amdgcn_s_setprio(2); break;
    default: __builtin_amdgcn_s_setprio(3); break;
    }
}

// Rows a two-step walk loads ahead of the row it stages: in half storage, whose
// walk waits for latency and the vector ALU, two (8192^2: 372 us per step
// against 391 with one); in single precision, which is near the memory's rate,
// one (4096^2: 136.8 against 142.8).
template <class P>
constexpr int kStep2Lead = P::kDev ? 2 : 1;

// The value of another lane of the same 16: 0xB1 swaps the lanes of each
// pair, 0x100 + n takes it from n lanes up.
template <int kCtrl>
__device__ __forceinline__ float row_move(float v)
{
    return __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v), kCtrl, 0xf, 0xf, true));
}

template <class P, int NT, int kOm>
__device__ __forceinline__ void
step2_tile(const typename P::S* __restrict__ src, typename P::S* __restrict__ dst,
           const Geom& g, const CoefT<typename P::C>& k, const int lb, Step2Smem<P, NT>& sm)
{
    using S = typename P::S;
    using C = typename P::C;
    constexpr int W = NT - 6;           // output columns of the tile
    constexpr int LW = NT + 4;          // psi rings: lanes plus 2 columns each side
    constexpr int kWaves = NT / 64;
    constexpr int kHpw = 4 / kWaves;
    constexpr int U = Step2Smem<P, NT>::U, NF = Step2Smem<P, NT>::NF;
    C (&ring)[U][LW] = sm.ring;
    C (&ring2)[U][LW] = sm.ring2;
    S* const fs = &sm.fs[0][0][0];
    constexpr int FR = 9 * NT;          // one row of fs

    const int tid = threadIdx.x;
    const int lane = tid & 63;
    const int wid = tid >> 6;
    const int sx = lb % g.tiles_x;
    const int sy = lb / g.tiles_x;
    const int x0 = sx * W;              // first output column
    const int y0 = sy * g.tile_y;
    const int y1 = min(y0 + g.tile_y, g.ny);
    const int dir = ((sy + (int)(k.step >> 1)) & 1) ? -1 : 1;
    const int ystart = dir > 0 ? y0 : y1 - 1;
    const int nrows = y1 - y0;
    const int nx = g.nx, ny = g.ny;
    auto modn = [](int v, int n) { v %= n; return v < 0 ? v + n : v; };
    // Lattice row of walk row r.  r runs from -5 to nrows + 4, so
    // ystart + r dir lies in [y0 - 5, y1 + 4], within [-ny, 2 ny) for
    // ny >= 5: one conditional add or subtract wraps it (a modulo by a
    // value unknown at compile time costs a long scalar sequence per row).
    auto wrow = [&](int r) { return wrapi(ystart + r * dir, ny); };

    const S* pl[9];
    S* pd[9];
#pragma unroll
    for (int i = 0; i < 9; ++i) {
        pl[i] = src + (int64_t)i * g.plane;
        pd[i] = dst + (int64_t)i * g.plane;
    }
    const Offs<P> o(k.rho_ref);
    CoefT<C> k2 = k;
    k2.step = k.step + 1;

    // Level-1 column of this lane (LDS column tid + 2): x0 - 3 + tid.
    const int xb = x0 - 3;
    const int xc = modn(xb + tid, nx);
    const int xcm = xc == 0 ? nx - 1 : xc - 1;
    const int xcp = xc == nx - 1 ? 0 : xc + 1;
    // A uniform row base plus a 32-bit lane offset needs no 64-bit vector add.
    auto pull32 = [&](int rm, int r0, int rp, S (&f)[9]) {
        constexpr uint32_t kB = sizeof(S);
        const int rows[3] = {rp, r0, rm};
        uint32_t cols[3] = {xcp * kB, xc * kB, xcm * kB};
#pragma unroll
        for (int i = 0; i < 3; ++i) asm volatile("" : "+v"(cols[i]));
#pragma unroll
        for (int i = 0; i < 9; ++i)
            f[i] = *at32(pl[i] + rows[1 + kQCy[i]], cols[1 + kQCx[i]]);
    };
    auto decode = [&](const S (&v)[9], C (&f)[9]) {
#pragma unroll
        for (int i = 0; i < 9; ++i) f[i] = o.dec(v[i], o.of(i));
    };
    // Level-2 output: lanes 3 .. 3+W-1, column x0 + tid - 3.
    const bool own2 = tid >= 3 && tid < 3 + W && x0 + tid - 3 < nx;

    // Halo columns of level 1 (xb-2, xb-1, xb+NT, xb+NT+1): a column is held
    // by 16 lanes, its populations in the lanes' order 1 3 2 4 5 7 6 8 0, so
    // that the density's sum needs only shifts within the 16 lanes.
    const int hj = lane & 15;
    const int hi = hj < 8 ? (int)(0x86754231u >> (4 * hj)) & 15 : 0;
    const int hcol = wid * kHpw + (lane >> 4) % kHpw;
    const int hlds = hcol < 2 ? hcol : NT + hcol;
    const int hgx = modn(xb - 2 + hlds - q_cx(hi), nx);
    const S* hp = src + (int64_t)hi * g.plane + hgx;
    const int hcy = q_cy(hi);
    const C hoff = o.of(hi);
    const bool hown = hj == 0 && lane < 16 * kHpw;
    // rm, r0, rp: offsets of rows y - 1, y, y + 1 in a plane.
    auto halo_load = [&](int rm, int r0, int rp) -> S { return hp[hcy > 0 ? rm : (hcy < 0 ? rp : r0)]; };
    auto halo_psi = [&](S raw, int slot) {
        const C hv = o.dec(raw, hoff);
        const C pair = hv + row_move<0xB1>(hv);             // 1 + 3, 2 + 4, 5 + 7, 6 + 8
        const C diag = pair + row_move<0x102>(pair);        // lane 4: (5 + 7) + (6 + 8)
        const C axis = (row_move<0x108>(hv) + pair) + row_move<0x102>(pair);
        const C ps = psi_of(axis + row_move<0x104>(diag), k);
        if (hown) ring[slot][hlds] = ps;
    };
    auto load = [&](int y, S (&f)[9], S& hv) {
        const int r0 = y * g.pitch;
        const int rm = (y == 0 ? ny - 1 : y - 1) * g.pitch, rp = (y == ny - 1 ? 0 : y + 1) * g.pitch;
        pull32(rm, r0, rp, f);
        hv = halo_load(rm, r0, rp);
    };

    // Level-1 walk row p lives in Bf[(p + 3) % U] (p >= -3); the level-2
    // pre-collision row formed at iteration it in F2[(it + 2) % U].  The
    // loads of a row are written LEAD iterations before its psi is staged.
    // At tau = 1 the collision needs no more of a row than its moments, taken
    // where its psi is staged: three registers a row wait for it, not nine.
    constexpr int LEAD = kStep2Lead<P>;
    constexpr bool kMom = kOm == 1;
    S Raw[U][9] = {}, Hh[U] = {};
    C Bf[U][9] = {}, F2[U][9] = {};
    Moments<C> M1[U] = {}, M2[U] = {};

    // Prologue: psi at t of walk rows -5 .. -1 into ring slots 0 .. 4 and
    // the populations of rows -3 .. -1 into Bf[0 .. 2].
    {
        S T[5][9], hv[5];
#pragma unroll
        for (int r = 0; r < 5; ++r) load(wrow(r - 5), T[r], hv[r]);
#pragma unroll
        for (int r = 0; r < 5; ++r) {
            C f[9];
            decode(T[r], f);
            ring[r][tid + 2] = psi_of(density(f), k);
            if (r >= 2) {
                M1[r - 2] = moments(f);
                for (int i = 0; i < 9; ++i) Bf[r - 2][i] = f[i];
            }
        }
#pragma unroll
        for (int r = 0; r < 5; ++r) halo_psi(hv[r], r);
        // Rows 0 .. LEAD - 2: their loads stay in flight into the walk.
#pragma unroll
        for (int r = 0; r < LEAD - 1; ++r) load(wrow(r), Raw[3 + r], Hh[3 + r]);
    }
    __syncthreads();

    int yl = wrow(LEAD - 2);  // lattice row of the last loaded walk row
    // One iteration per level-1 row p = it - 3, it = 0 .. nrows + 6; it % U = J.
    // All of it but the last collision runs at every row: where a row's
    // neighbours are not there yet, or no longer needed, it forms values that
    // nothing reads, and without branches the phases interleave.
    auto group = [&](auto Jc, int it) {
        constexpr int J = decltype(Jc)::value;
        const int p = it - 3;
        set_row_priority(it);
        // Lead row p + 2 + LEAD (psi at t is needed up to row nrows + 4; past
        // it the last row again).
        yl = p + 2 + LEAD < nrows + 5 ? wrapi(yl + dir, ny) : yl;
        load(yl, Raw[(J + 2 + LEAD) % U], Hh[(J + 2 + LEAD) % U]);
        __builtin_amdgcn_sched_barrier(0);

        // Level 2, part 1: pre-collision populations at t+1 of row p - 2
        // (pulled from the ring rows p-3 .. p-1) and their psi.  Formed here,
        // collided two iterations later (which reads F2[J]).  Population i
        // comes from row y - c_y, which is walk row p - 2 - c_y dir, lane
        // l - c_x (lanes 0 and NT-1 form values no output uses).
        {
            C(&Fr)[9] = F2[(J + 2) % U];
            const S* const row[3] = {fs + (dir > 0 ? J % NF : (J + 2) % NF) * FR + tid, fs + (J + 3) % NF * FR + tid,
                                     fs + (dir > 0 ? (J + 2) % NF : J % NF) * FR + tid};
#pragma unroll
            for (int i = 0; i < 9; ++i) Fr[i] = o.dec(row[1 + kQCy[i]][i * NT - kQCx[i]], o.of(i));
            M2[(J + 2) % U] = moments(Fr);
            ring2[J % U][tid + 2] = psi_of(M2[(J + 2) % U].rho, k2);
        }

        // Level 1: force and collision of row p into the ring of t+1.  The
        // stencil's rows are taken in walk order.
        C anchor;
        {
            const Stencil<C> st(ring[J % U], ring[(J + 1) % U], ring[(J + 2) % U], ring[(J + 3) % U],
                                ring[(J + 4) % U], tid + 2);
            C q[9];
            site_collide<false, P::kDev, kOm>(Bf[J % U], kMom ? &M1[J % U] : nullptr, st, k, q, (C*)nullptr,
                                              o.o1, o.o2, dir < 0);
            S* lp[9];
#pragma unroll
            for (int i = 0; i < 9; ++i) lp[i] = fs + (J + 1) % NF * FR + i * NT;
            const uint32_t rnd = P::kDev ? site_hash(xc, wrow(p), k.step) : 0u;
            store_site<P>(lp, tid, q, o, rnd);
            anchor = q[1];
        }

        // Stage psi at t of row p + 3.
        {
            C(&NFr)[9] = Bf[(J + 3) % U];
            S(&raw)[9] = Raw[(J + 3) % U];
            S& HF = Hh[(J + 3) % U];
#pragma unroll
            for (int i = 0; i < 9; ++i) asm volatile("" : "+v"(raw[i]) : "v"(anchor));
            asm volatile("" : "+v"(HF) : "v"(anchor));
            decode(raw, NFr);
            M1[(J + 3) % U] = moments(NFr);
            ring[(J + 5) % U][tid + 2] = psi_of(M1[(J + 3) % U].rho, k);
            halo_psi(HF, (J + 5) % U);
        }
        __builtin_amdgcn_sched_barrier(0);
        __syncthreads();

        // Level 2, part 2: force and collision at t+1 of row q = p - 4, from
        // psi rows q-2 .. q+2 at t+1; store.
        const int qr = p - 4;
        if (qr >= 0 && qr < nrows) {
            const Stencil<C> st2(ring2[(J + 4) % U], ring2[(J + 5) % U], ring2[(J + 6) % U], ring2[(J + 7) % U],
                                 ring2[J % U], tid + 2);
            C q2[9];
            site_collide<false, P::kDev, kOm>(F2[J % U], kMom ? &M2[J % U] : nullptr, st2, k2, q2,
                                              (C*)nullptr, o.o1, o.o2, dir < 0);
            if (own2) {
                const int yq = wrow(qr);
                const int xq = x0 + tid - 3;
                uint32_t cq = (uint32_t)xq * (uint32_t)sizeof(S);
                asm volatile("" : "+v"(cq));
                const uint32_t rnd = P::kDev ? site_hash(xq, yq, k2.step) : 0u;
                S* row[9];
#pragma unroll
                for (int i = 0; i < 9; ++i) row[i] = at32(pd[i] + yq * g.pitch, cq);
                store_site<P>(row, 0, q2, o, rnd);
            }
        }
    };

    const int iters = nrows + 7;
#pragma unroll 1
    for (int it = 0;;) {
        group(Ic<0>{}, it);
        if (++it >= iters) break;
        group(Ic<1>{}, it);
        if (++it >= iters) break;
        group(Ic<2>{}, it);
        if (++it >= iters) break;
        group(Ic<3>{}, it);
        if (++it >= iters) break;
        group(Ic<4>{}, it);
        if (++it >= iters) break;
        group(Ic<5>{}, it);
        if (++it >= iters) break;
        group(Ic<6>{}, it);
        if (++it >= iters) break;
        group(Ic<7>{}, it);
        if (++it >= iters) break;
    }
}

// At least three waves per SIMD: without the bound the kernel for any tau
// takes 188 registers and two.  Four (128 registers, 8 bytes spilled) are slower
// at tau = 1: half storage 8192^2 387 us per step against 362.
template <class P, int NT, int kOm>
__global__ void __launch_bounds__(NT, 3)
k_step2(const typename P::S* __restrict__ src, typename P::S* __restrict__ dst, Geom g,
        CoefT<typename P::C> k)
{
    // tau = 1 (every run of the paper) and other tau as separate kernels: the
    // collision has no branch inside the loop, and the walk at tau = 1, which
    // keeps three moments of a waiting row instead of its nine populations,
    // is not given the registers of the other.
    __shared__ Step2Smem<P, NT> sm;
    step2_tile<P, NT, kOm>(src, dst, g, k, xcd_remap(blockIdx.x, gridDim.x), sm);
}

// One launch = one time step of one lattice: workgroup b updates logical
// tile xcd_remap(b).
template <class P, int NT, int MODE, int RPI, int LEAD>
__global__ void __launch_bounds__(NT)
k_step(const typename P::S* __restrict__ src, typename P::S* __restrict__ dst,
       Geom g, CoefT<typename P::C> k, double* __restrict__ partials)
{
    step_tile<P, NT, MODE, RPI, LEAD>(src, dst, g, k, partials, xcd_remap(blockIdx.x, gridDim.x));
}

// One launch = one time step of a batch of independent lattices.  The
// logical tiles of all lattices are numbered consecutively (lattice by
// lattice); tile_lattice maps a logical tile to its lattice, whose
// geometry, coefficients and buffers sit in desc.  Every lattice's tile is
// processed exactly as the single-lattice kernel processes it, so fields
// are bit-identical to single-lattice runs with the same tile shape.
template <class P, int NT, bool kTau1>
__global__ void __launch_bounds__(NT, 3)
k_step2_batch(const BatchLattice* __restrict__ desc, const int32_t* __restrict__ tile_lattice,
              int parity, uint32_t step)
{
    using S = typename P::S;
    const int gl = xcd_remap(blockIdx.x, gridDim.x);
    const int lat = tile_lattice[gl];
    const BatchLattice& d = desc[lat];
    static_assert(sizeof(typename P::C) == 4, "two-step kernels compute in single precision");
    const float* cf = d.coef_f;
    const CoefT<float> k{cf[0], cf[1], cf[2],  cf[3],  cf[4],  cf[5], cf[6],
                         cf[7], cf[8], cf[9], cf[10], cf[11], cf[12], step};
    // kTau1 states that tau is 1 in every lattice; else the walks for tau = 1 and
    // for other tau share the kernel and its registers.
    __shared__ Step2Smem<P, NT> sm;
    if (kTau1 || k.omega == 1.0f)
        step2_tile<P, NT, 1>(static_cast<const S*>(d.buf[parity]), static_cast<S*>(d.buf[parity ^ 1]),
                             d.geom2, k, gl - d.tile_begin2, sm);
    else
        step2_tile<P, NT, 0>(static_cast<const S*>(d.buf[parity]), static_cast<S*>(d.buf[parity ^ 1]),
                             d.geom2, k, gl - d.tile_begin2, sm);
}

template <class P, int NT, int MODE, int RPI, int LEAD>
__global__ void __launch_bounds__(NT)
k_step_batch(const BatchLattice* __restrict__ desc, const int32_t* __restrict__ tile_lattice,
             int parity, uint32_t step, double* __restrict__ partials)
{
    using S = typename P::S;
    const int gl = xcd_remap(blockIdx.x, gridDim.x);
    const int lat = tile_lattice[gl];
    const BatchLattice& d = desc[lat];
    CoefT<typename P::C> k = convert<typename P::C>(d.coef);
    k.step = step;
    step_tile<P, NT, MODE, RPI, LEAD>(static_cast<const S*>(d.buf[parity]),
                                static_cast<S*>(d.buf[parity ^ 1]), d.geom, k,
                                partials + (int64_t)d.tile_begin * 4, gl - d.tile_begin);
}

// Fixed-order reduction of the per-workgroup partials into one trace row
// {t, M, E_s, E_m, sum psi^2, E_bulk} (one workgroup of 256 threads).
__device__ __forceinline__ void final_row(const double* __restrict__ partials, int blocks,
                                          double t, double half_A1, double* __restrict__ out)
{
    __shared__ double sm[4][256];
    const int tid = threadIdx.x;
#pragma unroll
    for (int q = 0; q < 4; ++q) {
        double s = 0.0;
        for (int b = tid; b < blocks; b += 256) s += partials[(int64_t)b * 4 + q];
        sm[q][tid] = s;
    }
    __syncthreads();
    for (int w = 128; w > 0; w >>= 1) {
        if (tid < w) {
#pragma unroll
            for (int q = 0; q < 4; ++q) sm[q][tid] += sm[q][tid + w];
        }
        __syncthreads();
    }
    if (tid == 0) {
        out[0] = t;
        out[1] = sm[0][0];
        out[2] = sm[1][0];
        out[3] = sm[2][0];
        out[4] = sm[3][0];
        out[5] = half_A1 * sm[3][0];
    }
}

__global__ void __launch_bounds__(256)
k_final(const double* __restrict__ partials, int blocks, double t, double half_A1,
        double* __restrict__ out)
{
    final_row(partials, blocks, t, half_A1, out);
}

// One workgroup per lattice of a batch: row `row` of each lattice's trace.
__global__ void __launch_bounds__(256)
k_final_batch(const BatchLattice* __restrict__ desc, const double* __restrict__ partials,
              double t, int64_t row)
{
    const BatchLattice& d = desc[blockIdx.x];
    final_row(partials + (int64_t)d.tile_begin * 4, d.geom.blocks, t, d.half_A1,
              d.trace + row * 6);
}

// Sets *flag to 1 if some value is not finite or, with positive, not > 0.  The
// flag is only ever set, so no order of the stores matters.
__global__ void __launch_bounds__(256)
k_check(const double* __restrict__ v, int64_t n, bool positive, int* __restrict__ flag)
{
    bool bad = false;
    for (int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x; i < n; i += (int64_t)gridDim.x * 256) {
        const double x = v[i];
        bad = bad || !(fabs(x) <= 1.7976931348623157e308) || (positive && !(x > 0.0));
    }
    if (bad) *flag = 1;
}

__global__ void k_clear(int* __restrict__ flag) { *flag = 0; }

// rho and u = j / rho of the pre-collision state, dense [ny][nx] doubles.
template <class P>
__global__ void __launch_bounds__(256)
k_moments(const typename P::S* __restrict__ src, Geom g, typename P::C rho_ref,
          double* __restrict__ rho, double* __restrict__ ux, double* __restrict__ uy)
{
    using C = typename P::C;
    const int x = blockIdx.x * 256 + threadIdx.x;
    const int y = blockIdx.y;
    if (x >= g.nx) return;
    const typename P::S* pl[9];
#pragma unroll
    for (int i = 0; i < 9; ++i) pl[i] = src + (int64_t)i * g.plane;
    const Offs<P> o(rho_ref);
    C f[9];
    pull<P>(pl, g, x, x == 0 ? g.nx - 1 : x - 1, x == g.nx - 1 ? 0 : x + 1, y, o, f);
    const C r = density(f);
    const C jx = (f[1] - f[3]) + ((f[5] - f[7]) + (f[8] - f[6]));
    const C jy = (f[2] - f[4]) + ((f[5] - f[7]) + (f[6] - f[8]));
    const int64_t at = (int64_t)y * g.nx + x;
    if (rho) rho[at] = (double)r;
    if (ux) ux[at] = (double)jx / (double)r;
    if (uy) uy[at] = (double)jy / (double)r;
}

// Equilibrium populations f_i^eq(rho, u) of each site, stored upstream at
// x - c_i so that the next pull delivers them to x.
template <class P>
__global__ void __launch_bounds__(256)
k_init(const double* __restrict__ rho, const double* __restrict__ ux,
       const double* __restrict__ uy, typename P::S* __restrict__ dst, Geom g,
       typename P::C rho_ref)
{
    using C = typename P::C;
    const int x = blockIdx.x * 256 + threadIdx.x;
    const int y = blockIdx.y;
    if (x >= g.nx) return;
    const int64_t at = (int64_t)y * g.nx + x;
    const C r = (C)rho[at];
    const C u = ux ? (C)ux[at] : (C)0;
    const C v = uy ? (C)uy[at] : (C)0;
    const C usq = (C)1.5 * (u * u + v * v);
    const Offs<P> o(rho_ref);
    const int cx[9] = {0, 1, 0, -1, 0, 1, -1, -1, 1};
    const int cy[9] = {0, 0, 1, 0, -1, 1, 1, -1, -1};
#pragma unroll
    for (int i = 0; i < 9; ++i) {
        const C w = i == 0 ? (C)4 / (C)9 : (i < 5 ? (C)1 / (C)9 : (C)1 / (C)36);
        const C cu = (C)cx[i] * u + (C)cy[i] * v;
        const C feq = w * r * ((C)1 + (C)3 * cu + (C)4.5 * cu * cu - usq);
        const int xs = wrapi(x - cx[i], g.nx);
        const int ys = wrapi(y - cy[i], g.ny);
        P::st(dst + (int64_t)i * g.plane + (int64_t)ys * g.pitch + xs, feq, o.of(i));
    }
}

// Raw population words between the pitched upstream layout and a dense
// [9][ny][nx] array of pre-collision populations (an exact permutation).
template <typename W, bool kGet>
__global__ void __launch_bounds__(256)
k_state(const W* __restrict__ in, W* __restrict__ out, Geom g)
{
    const int x = blockIdx.x * 256 + threadIdx.x;
    const int y = blockIdx.y;
    const int i = blockIdx.z;
    if (x >= g.nx) return;
    const int cx[9] = {0, 1, 0, -1, 0, 1, -1, -1, 1};
    const int cy[9] = {0, 0, 1, 0, -1, 1, 1, -1, -1};
    const int64_t d = ((int64_t)i * g.ny + y) * g.nx + x;
    const int64_t s = (int64_t)i * g.plane + (int64_t)wrapi(y - cy[i], g.ny) * g.pitch +
                      wrapi(x - cx[i], g.nx);
    if (kGet)
        out[d] = in[s];
    else
        out[s] = in[d];
}

template <class P, int NT, int RPI>
hipError_t step_nt(int mode, const void* src, void* dst, const Geom& g,
                   const Coef& c, double* partials, hipStream_t s)
{
    using S = typename P::S;
    const auto k = convert<typename P::C>(c);
    const dim3 grid(g.blocks), block(NT);
    const S* a = static_cast<const S*>(src);
    S* b = static_cast<S*>(dst);
    if (mode == MODE_STEP) {
        if constexpr (lead2_variant<P, RPI>()) {
            if (g.tile_y >= kLead2MinRows) {
                hipLaunchKernelGGL((k_step<P, NT, MODE_STEP, RPI, 2>), grid, block, 0, s, a, b, g, k, partials);
                return hipGetLastError();
            }
        }
        hipLaunchKernelGGL((k_step<P, NT, MODE_STEP, RPI, 1>), grid, block, 0, s, a, b, g, k, partials);
    } else if (mode == MODE_STEP_ENERGY)
        hipLaunchKernelGGL((k_step<P, NT, MODE_STEP_ENERGY, RPI, 1>), grid, block, 0, s, a, b, g, k, partials);
    else if (mode == MODE_STEP_TAPE) {
        if constexpr (P::kDev)
            return hipErrorInvalidValue;
        else
            hipLaunchKernelGGL((k_step<P, NT, MODE_STEP_TAPE, RPI, 1>), grid, block, 0, s, a, b, g, k, partials);
    } else
        hipLaunchKernelGGL((k_step<P, NT, MODE_ENERGY, RPI, 1>), grid, block, 0, s, a, b, g, k, partials);
    return hipGetLastError();
}

template <class P, int NT>
hipError_t step2_nt(const void* src, void* dst, const Geom& g, const Coef& c, hipStream_t s)
{
    using S = typename P::S;
    const auto k = convert<typename P::C>(c);
    if (k.omega == 1)
        hipLaunchKernelGGL((k_step2<P, NT, 1>), dim3(g.blocks), dim3(NT), 0, s, static_cast<const S*>(src),
                           static_cast<S*>(dst), g, k);
    else
        hipLaunchKernelGGL((k_step2<P, NT, 0>), dim3(g.blocks), dim3(NT), 0, s, static_cast<const S*>(src),
                           static_cast<S*>(dst), g, k);
    return hipGetLastError();
}

template <class P, int NT>
hipError_t step_rpi(int mode, const void* src, void* dst, const Geom& g,
                    const Coef& c, double* partials, hipStream_t s)
{
    return g.rows_per_iter == 2 ? step_nt<P, NT, 2>(mode, src, dst, g, c, partials, s)
                                : step_nt<P, NT, 1>(mode, src, dst, g, c, partials, s);
}

template <class P>
hipError_t step_p(int mode, const void* src, void* dst, const Geom& g,
                  const Coef& c, double* partials, hipStream_t s)
{
    switch (g.tile_x) {
    case 64: return step_rpi<P, 64>(mode, src, dst, g, c, partials, s);
    case 128: return step_rpi<P, 128>(mode, src, dst, g, c, partials, s);
    case 256: return step_rpi<P, 256>(mode, src, dst, g, c, partials, s);
    default: return hipErrorInvalidValue;
    }
}

struct BatchLaunch {
    const BatchLattice* desc;
    const int32_t* tile_lattice;
    int tiles;
    int parity;
    uint32_t step;
    double* partials;
    int min_tile_y;  // smallest tile_y of the batch's lattices
};

template <class P, int NT, int RPI>
hipError_t batch_nt(int mode, const BatchLaunch& a, hipStream_t s)
{
    const dim3 grid(a.tiles), block(NT);
    if (mode == MODE_STEP) {
        if constexpr (lead2_variant<P, RPI>()) {
            if (a.min_tile_y >= kLead2MinRows) {
                hipLaunchKernelGGL((k_step_batch<P, NT, MODE_STEP, RPI, 2>), grid, block, 0, s, a.desc,
                                   a.tile_lattice, a.parity, a.step, a.partials);
                return hipGetLastError();
            }
        }
        hipLaunchKernelGGL((k_step_batch<P, NT, MODE_STEP, RPI, 1>), grid, block, 0, s, a.desc,
                           a.tile_lattice, a.parity, a.step, a.partials);
    } else if (mode == MODE_STEP_ENERGY)
        hipLaunchKernelGGL((k_step_batch<P, NT, MODE_STEP_ENERGY, RPI, 1>), grid, block, 0, s, a.desc,
                           a.tile_lattice, a.parity, a.step, a.partials);
    else
        hipLaunchKernelGGL((k_step_batch<P, NT, MODE_ENERGY, RPI, 1>), grid, block, 0, s, a.desc,
                           a.tile_lattice, a.parity, a.step, a.partials);
    return hipGetLastError();
}

template <class P>
hipError_t batch_p(int mode, int tile_x, int rpi, const BatchLaunch& a, hipStream_t s)
{
    const bool two = rpi == 2;
    switch (tile_x) {
    case 64: return two ? batch_nt<P, 64, 2>(mode, a, s) : batch_nt<P, 64, 1>(mode, a, s);
    case 128: return two ? batch_nt<P, 128, 2>(mode, a, s) : batch_nt<P, 128, 1>(mode, a, s);
    case 256: return two ? batch_nt<P, 256, 2>(mode, a, s) : batch_nt<P, 256, 1>(mode, a, s);
    default: return hipErrorInvalidValue;
    }
}

}  // namespace

template <class P>
hipError_t step2_p(const void* src, void* dst, const Geom& g, const Coef& c, hipStream_t s)
{
    switch (g.tile_x) {
    case 64: return step2_nt<P, 64>(src, dst, g, c, s);
    case 128: return step2_nt<P, 128>(src, dst, g, c, s);
    case 256: return step2_nt<P, 256>(src, dst, g, c, s);
    default: return hipErrorInvalidValue;
    }
}

template <class P>
static hipError_t step2_batch_p(bool tau1, const BatchLattice* desc, const int32_t* tile_lattice, int tiles, int parity,
                                uint32_t step, hipStream_t s)
{
    const auto kernel = tau1 ? k_step2_batch<P, kBatchLanes2, true> : k_step2_batch<P, kBatchLanes2, false>;
    hipLaunchKernelGGL(kernel, dim3(tiles), dim3(kBatchLanes2), 0, s, desc, tile_lattice, parity, step);
    return hipGetLastError();
}

hipError_t launch_step2_batch(int storage, bool tau1, const BatchLattice* desc, const int32_t* tile_lattice, int tiles,
                              int parity, uint32_t step, hipStream_t s)
{
    if (tiles <= 0) return hipErrorInvalidValue;
    switch (storage) {
    case ST_F32: return step2_batch_p<PF32>(tau1, desc, tile_lattice, tiles, parity, step, s);
    case ST_F16DEV: return step2_batch_p<PF16>(tau1, desc, tile_lattice, tiles, parity, step, s);
    default: return hipErrorInvalidValue;
    }
}

hipError_t launch_step2(int storage, const void* src, void* dst, const Geom& g, const Coef& c,
                        hipStream_t s)
{
    switch (storage) {
    case ST_F32: return step2_p<PF32>(src, dst, g, c, s);
    case ST_F16DEV: return step2_p<PF16>(src, dst, g, c, s);
    default: return hipErrorInvalidValue;
    }
}

namespace {
template <class P>
const void* step2_kernel(int tile_x)
{
    switch (tile_x) {
    case 64: return reinterpret_cast<const void*>(k_step2<P, 64, 0>);
    case 128: return reinterpret_cast<const void*>(k_step2<P, 128, 0>);
    case 256: return reinterpret_cast<const void*>(k_step2<P, 256, 0>);
    default: return nullptr;
    }
}
}  // namespace

int step2_resident(int storage, int tile_x)
{
    static std::mutex mu;
    static std::map<std::tuple<int, int, int>, int> cache;
    int dev = 0;
    if (hipGetDevice(&dev) != hipSuccess) return -1;
    const auto key = std::make_tuple(dev, storage, tile_x);
    std::lock_guard<std::mutex> lk(mu);
    auto it = cache.find(key);
    if (it != cache.end()) return it->second;
    const void* fn = storage == ST_F32 ? step2_kernel<PF32>(tile_x)
                   : storage == ST_F16DEV ? step2_kernel<PF16>(tile_x) : nullptr;
    int cus = 0, per_cu = 0;
    if (!fn || hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess ||
        hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, fn, tile_x, 0) != hipSuccess) {
        (void)hipGetLastError();
        return -1;
    }
    const int r = cus > 0 && per_cu > 0 ? cus * per_cu : -1;
    cache.emplace(key, r);
    return r;
}

hipError_t launch_step_batch(int storage, int mode, int tile_x, int rows_per_iter, int min_tile_y,
                             const BatchLattice* desc, const int32_t* tile_lattice, int tiles,
                             int parity, uint32_t step, double* partials, hipStream_t s)
{
    const BatchLaunch a{desc, tile_lattice, tiles, parity, step, partials, min_tile_y};
    switch (storage) {
    case ST_F64: return batch_p<PF64>(mode, tile_x, rows_per_iter, a, s);
    case ST_F32: return batch_p<PF32>(mode, tile_x, rows_per_iter, a, s);
    case ST_F16DEV: return batch_p<PF16>(mode, tile_x, rows_per_iter, a, s);
    default: return hipErrorInvalidValue;
    }
}

hipError_t launch_final_batch(const BatchLattice* desc, int count, const double* partials,
                              double t, int64_t row, hipStream_t s)
{
    hipLaunchKernelGGL(k_final_batch, dim3(count), dim3(256), 0, s, desc, partials, t, row);
    return hipGetLastError();
}

hipError_t launch_step(int storage, int mode, const void* src, void* dst,
                       const Geom& g, const Coef& c, double* partials,
                       hipStream_t s)
{
    switch (storage) {
    case ST_F64: return step_p<PF64>(mode, src, dst, g, c, partials, s);
    case ST_F32: return step_p<PF32>(mode, src, dst, g, c, partials, s);
    case ST_F16DEV: return step_p<PF16>(mode, src, dst, g, c, partials, s);
    default: return hipErrorInvalidValue;
    }
}

hipError_t launch_final(const double* partials, int blocks, double t,
                        double half_A1, double* out_row, hipStream_t s)
{
    hipLaunchKernelGGL(k_final, dim3(1), dim3(256), 0, s, partials, blocks, t, half_A1, out_row);
    return hipGetLastError();
}

hipError_t launch_check(const double* v, int64_t n, bool positive, int* flag, hipStream_t s)
{
    const int blocks = (int)std::min<int64_t>(2048, (n + 255) / 256);
    hipLaunchKernelGGL(k_check, dim3(blocks), dim3(256), 0, s, v, n, positive, flag);
    return hipGetLastError();
}

hipError_t launch_clear(int* flag, hipStream_t s)
{
    hipLaunchKernelGGL(k_clear, dim3(1), dim3(1), 0, s, flag);
    return hipGetLastError();
}

hipError_t launch_moments(int storage, const void* src, const Geom& g,
                          const Coef& c, double* rho, double* ux, double* uy,
                          hipStream_t s)
{
    const dim3 grid((g.nx + 255) / 256, g.ny), block(256);
    switch (storage) {
    case ST_F64:
        hipLaunchKernelGGL(k_moments<PF64>, grid, block, 0, s, static_cast<const double*>(src), g,
                           c.rho_ref, rho, ux, uy);
        break;
    case ST_F32:
        hipLaunchKernelGGL(k_moments<PF32>, grid, block, 0, s, static_cast<const float*>(src), g,
                           (float)c.rho_ref, rho, ux, uy);
        break;
    case ST_F16DEV:
        hipLaunchKernelGGL(k_moments<PF16>, grid, block, 0, s, static_cast<const _Float16*>(src), g,
                           (float)c.rho_ref, rho, ux, uy);
        break;
    default: return hipErrorInvalidValue;
    }
    return hipGetLastError();
}

hipError_t launch_init(int storage, const double* rho, const double* ux,
                       const double* uy, void* dst, const Geom& g,
                       const Coef& c, hipStream_t s)
{
    const dim3 grid((g.nx + 255) / 256, g.ny), block(256);
    switch (storage) {
    case ST_F64:
        hipLaunchKernelGGL(k_init<PF64>, grid, block, 0, s, rho, ux, uy, static_cast<double*>(dst), g,
                           c.rho_ref);
        break;
    case ST_F32:
        hipLaunchKernelGGL(k_init<PF32>, grid, block, 0, s, rho, ux, uy, static_cast<float*>(dst), g,
                           (float)c.rho_ref);
        break;
    case ST_F16DEV:
        hipLaunchKernelGGL(k_init<PF16>, grid, block, 0, s, rho, ux, uy, static_cast<_Float16*>(dst), g,
                           (float)c.rho_ref);
        break;
    default: return hipErrorInvalidValue;
    }
    return hipGetLastError();
}

template <bool kGet>
static hipError_t state_copy(int storage, const void* in, void* out, const Geom& g, hipStream_t s)
{
    const dim3 grid((g.nx + 255) / 256, g.ny, 9), block(256);
    switch (storage_bytes(storage)) {
    case 8:
        hipLaunchKernelGGL((k_state<uint64_t, kGet>), grid, block, 0, s,
                           static_cast<const uint64_t*>(in), static_cast<uint64_t*>(out), g);
        break;
    case 4:
        hipLaunchKernelGGL((k_state<uint32_t, kGet>), grid, block, 0, s,
                           static_cast<const uint32_t*>(in), static_cast<uint32_t*>(out), g);
        break;
    case 2:
        hipLaunchKernelGGL((k_state<uint16_t, kGet>), grid, block, 0, s,
                           static_cast<const uint16_t*>(in), static_cast<uint16_t*>(out), g);
        break;
    default: return hipErrorInvalidValue;
    }
    return hipGetLastError();
}

hipError_t launch_get_state(int storage, const void* src, void* dense, const Geom& g, hipStream_t s)
{
    return state_copy<true>(storage, src, dense, g, s);
}

hipError_t launch_set_state(int storage, const void* dense, void* dst, const Geom& g, hipStream_t s)
{
    return state_copy<false>(storage, dense, dst, g, s);
}

void coef_to_f32(const Coef& c, float out[13])
{
    const CoefT<float> k = convert<float>(c);
    const float v[13] = {k.K1, k.K2, k.K4, k.K5, k.K8, k.KE0, k.tau, k.omega,
                         k.sqrt_rho0, k.inv_rho0, k.rho_ref, k.K4x2, k.K8x2};
    for (int i = 0; i < 13; ++i) out[i] = v[i];
}

}  // namespace lbk
