// Host side of liblb.so: the C ABI declared in include/lb.h.
//
// Validates every argument before any launch that uses it (host values here,
// device values by a copy or a kernel that looks them over), carves the
// caller's device workspace, keeps the time step, the ping-pong buffer
// index and the trace bookkeeping, and issues the kernels of
// lb_kernels.hip on the caller's stream.
#include "lb.h"
#include "lb_internal.h"

#include <hip/hip_runtime.h>

#include <algorithm>
#include <cmath>
#include <cstdarg>
#include <cstdio>
#include <cstring>
#include <functional>
#include <map>
#include <mutex>
#include <set>
#include <utility>
#include <string>
#include <vector>

using lbk::Coef;
using lbk::Geom;

namespace {

thread_local std::string g_err;

int fail(int code, const char* fmt, ...)
{
    char buf[512];
    va_list ap;
    va_start(ap, fmt);
    std::vsnprintf(buf, sizeof buf, fmt, ap);
    va_end(ap);
    g_err = buf;
    return code;
}

int hip_fail(hipError_t e, const char* what)
{
    return fail(LB_ERR_HIP, "%s: %s", what, hipGetErrorString(e));
}

constexpr size_t kAlign = 256;
size_t align_up(size_t v) { return (v + kAlign - 1) / kAlign * kAlign; }

// Table 1 weights p(|c|^2), the D2Q9 weights w and the first-belt rest
// weight p_s0 = 1 - sum_k p_k = 247/420 implied by eq. (weights_1).
constexpr double kP1 = 4.0 / 63.0, kP2 = 4.0 / 135.0, kP4 = 1.0 / 180.0,
                 kP5 = 2.0 / 945.0, kP8 = 1.0 / 15120.0;
constexpr double kW0 = 4.0 / 9.0, kW1 = 1.0 / 9.0, kW2 = 1.0 / 36.0;
constexpr double kPS0 = 247.0 / 420.0;

// Link order: first belt in D2Q9 order, then |c|^2 = 4, 5, 8, each
// counter-clockwise from +x.
constexpr int kLX[24] = {1, 0, -1, 0, 1, -1, -1, 1, 2, 0, -2, 0,
                         2, 1, -1, -2, -2, -1, 1, 2, 2, -2, -2, 2};
constexpr int kLY[24] = {0, 1, 0, -1, 1, 1, -1, -1, 0, 2, 0, -2,
                         1, 2, 2, 1, -1, -2, -2, -1, 2, 2, -2, -2};

double coupling(int k, double G1, double G2)
{
    const int c2 = kLX[k] * kLX[k] + kLY[k] * kLY[k];
    const double p = c2 == 1 ? kP1 : c2 == 2 ? kP2 : c2 == 4 ? kP4 : c2 == 5 ? kP5 : kP8;
    if (k < 8) return G1 * (c2 == 1 ? kW1 : kW2) + G2 * p;
    return G2 * p;
}

Coef make_coef(const lb_params& p)
{
    Coef c;
    c.K1 = coupling(0, p.G1, p.G2);
    c.K2 = coupling(4, p.G1, p.G2);
    c.K4 = coupling(8, p.G1, p.G2);
    c.K5 = coupling(12, p.G1, p.G2);
    c.K8 = coupling(20, p.G1, p.G2);
    c.KE0 = p.G1 * kW0 + p.G2 * kPS0;
    c.tau = p.tau;
    c.omega = 1.0 / p.tau;
    c.sqrt_rho0 = std::sqrt(p.rho0);
    c.inv_rho0 = 1.0 / p.rho0;
    c.rho_ref = p.storage == LB_F16DEV ? p.rho_ref : 0.0;
    c.step = 0;
    return c;
}

int check_params(const lb_params* p)
{
    if (!p) return fail(LB_ERR_INVALID, "params is NULL");
    if (p->nx < 5 || p->ny < 5)
        return fail(LB_ERR_INVALID, "nx, ny must be >= 5 (got %d x %d)", p->nx, p->ny);
    // One population plane, padded rows included, must be indexable with
    // 32-bit offsets.
    if (((int64_t)p->nx + 192) * p->ny >= (int64_t(1) << 31))
        return fail(LB_ERR_INVALID, "(nx + 192) * ny must be < 2^31");
    // The moments, initialisation and state kernels put rows on the grid's
    // second dimension.
    if (p->ny > 65535) return fail(LB_ERR_INVALID, "ny must be <= 65535 (got %d)", p->ny);
    if (p->storage != LB_F64 && p->storage != LB_F32 && p->storage != LB_F16DEV)
        return fail(LB_ERR_INVALID, "unknown storage %d", p->storage);
    if (p->log_every < 0) return fail(LB_ERR_INVALID, "log_every must be >= 0");
    if (p->trace_cap < 0) return fail(LB_ERR_INVALID, "trace_cap must be >= 0");
    if (p->tile_x != 0 && p->tile_x != 64 && p->tile_x != 128 && p->tile_x != 256)
        return fail(LB_ERR_INVALID, "tile_x must be 0, 64, 128 or 256 (got %d)", p->tile_x);
    if (p->tile_y < 0 || p->tile_y > 4096)
        return fail(LB_ERR_INVALID, "tile_y must be in [0, 4096] (got %d)", p->tile_y);
    if (p->tile_rows < 0 || p->tile_rows > 2)
        return fail(LB_ERR_INVALID, "tile_rows must be 0, 1 or 2 (got %d)", p->tile_rows);
    if (p->steps_per_launch < 0 || p->steps_per_launch > 2)
        return fail(LB_ERR_INVALID, "steps_per_launch must be 0, 1 or 2 (got %d)", p->steps_per_launch);
    if (!std::isfinite(p->tau) || !(p->tau > 0.5))
        return fail(LB_ERR_INVALID, "tau must be finite and > 0.5");
    if (!std::isfinite(p->rho0) || !(p->rho0 > 0.0))
        return fail(LB_ERR_INVALID, "rho0 must be finite and > 0");
    if (!std::isfinite(p->G1) || !std::isfinite(p->G2))
        return fail(LB_ERR_INVALID, "G1, G2 must be finite");
    if (p->storage == LB_F16DEV && (!std::isfinite(p->rho_ref) || !(p->rho_ref > 0.0)))
        return fail(LB_ERR_INVALID, "rho_ref must be finite and > 0 for LB_F16DEV");
    return LB_OK;
}

// Launch shape and layout.  Defaults: the widest column strip (256, 128 or
// 64 columns) that the lattice fills, and the tallest tile of 32, 16, 8, 4
// or 2 rows that still gives at least 512 workgroups.
Geom make_geom(const lb_params& p)
{
    Geom g;
    g.nx = p.nx;
    g.ny = p.ny;
    // Row pitch: a multiple of 64 elements whose count of 64-element blocks
    // is odd, so consecutive rows (and the rows that concurrently running
    // workgroups touch) do not sit at power-of-two strides, which would
    // pile their accesses onto the same HBM channels.
    g.pitch = (p.nx + 63) / 64 * 64;
    if ((g.pitch / 64) % 2 == 0) g.pitch += 64;  // pitch <= nx + 127
    g.plane = (int64_t)p.ny * g.pitch;
    g.tile_x = p.tile_x ? p.tile_x : (p.nx >= 256 ? 256 : p.nx >= 128 ? 128 : 64);
    g.tiles_x = (p.nx + g.tile_x - 1) / g.tile_x;
    if (p.tile_y) {
        g.tile_y = p.tile_y;
    } else {
        // The tallest tile of 32, 16, 8, 4 or 2 rows that still gives at
        // least 512 workgroups (two per CU): tall tiles re-read fewer halo
        // rows, but a lattice of a few hundred rows would otherwise leave
        // most of the 256 CUs idle.
        g.tile_y = 32;
        while (g.tile_y > 2 && (int64_t)g.tiles_x * ((p.ny + g.tile_y - 1) / g.tile_y) < 512)
            g.tile_y /= 2;
    }
    if (g.tile_y > p.ny) g.tile_y = p.ny;
    g.rows_per_iter = p.tile_rows ? p.tile_rows : 1;
    g.blocks = g.tiles_x * ((p.ny + g.tile_y - 1) / g.tile_y);
    return g;
}

// Geometry of the two-step launches: tiles of tile_x lanes that produce
// tile_x - 6 columns (the first step also covers 3 columns each side).
// Explicit tile_x / tile_y apply to both kernels; the library's choice
// follows.
// Workgroups of the two-step kernel resident at once: the runtime's
// occupancy query on the current device (registers and LDS of the kernel for
// any tau as built; the one for tau = 1 needs fewer registers, but a fourth wave
// per SIMD gains nothing) times its compute units.  Without a device to ask, the value for
// the MI355X as the kernel is built today: 3 waves per SIMD, i.e. 6
// workgroups of 128 lanes or 3 of 256 lanes per CU, on 256 CUs (a GPU test
// holds this to the occupancy query).
int64_t step2_slots_fallback(int tile_x) { return 256 * (tile_x == 256 ? 3 : 6); }
int64_t step2_slots(int storage, int tile_x)
{
    const int r = lbk::step2_resident(storage == LB_F16DEV ? LB_F16DEV : LB_F32, tile_x);
    return r > 0 ? r : step2_slots_fallback(tile_x);
}

// Two-step launch shape.  A workgroup walks its rows one after the other,
// so while every tile is resident at once (one round), shorter tiles finish
// sooner: the default takes the shortest tiles (128 lanes, else 256) that
// all fit in one round, up to 48 rows.  Past that, a launch of more than
// one round pays for a last round left partly empty, and a taller tile for
// fewer recomputed halo rows:
//   - single precision: 256-lane tiles filling one round when they are at
//     most 96 rows tall, else tiles of about 48 rows, a few rows shorter
//     when that fills the last round, or, when the last round would be
//     under half full, the height that fills one round fewer (at most 56);
//   - half storage, whose two-step kernel is not bound by memory: the
//     tallest 256-lane tiles of at most 128 rows whose last round is full.
// Measured on MI355X (FP32, us/step; one step per launch in brackets):
//   1200^2 128x8 14.1 (19.6);  1800^2 128x18 23.9, 128x24 24.4 (42.6);
//   2048^2 128x23 38.5, 128x24 39.2, 256x46 45.2 (57.6);  2500^2 128x35 54.0,
//   128x40 55.1, 128x48 56.1 (115);  3000^2 256x47 72.4, 256x48 68.8, 128x48
//   94.1 (152);  3500^2 256x65 108, 256x47 131 (203);  4096^2 256x92 137,
//   128x92 131, 256x46 138 (245);  5120^2 256x47 225, 256x71 228, 256x143 227
//   (390);  6144^2 256x51 320, 256x48 337 (549);  8192^2 256x45 587, 256x48
//   606, 256x90 594, 256x179 576, 128x48 609 (1037).
// Half storage: 4096^2 256x92 98, 256x46 105, 256x56 113 (142);  6144^2 256x101
//   217, 256x48 238 (306);  8192^2 256x119 381 (three rounds), 256x90 388,
//   256x179 377, 256x357 370, 256x56 404 (6.3 rounds), 256x104 405 (3.4),
//   256x164 423 (2.1) (568).
Geom make_geom2(const lb_params& p, const Geom& g)
{
    Geom g2 = g;
    auto strips = [&](int tx) { return (int64_t)(p.nx + tx - 7) / (tx - 6); };
    auto rows = [&](int ty) { return (int64_t)(p.ny + ty - 1) / ty; };
    // Height of the tiles of tx lanes that fill nr rounds (their count is at
    // most nr rounds' worth, and just under it).
    auto fill = [&](int tx, int64_t nr) -> int64_t {
        const int64_t per_strip = nr * step2_slots(p.storage, tx) / strips(tx);
        return per_strip > 0 ? (p.ny + per_strip - 1) / per_strip : (int64_t)p.ny;
    };
    int tx = p.tile_x, ty = p.tile_y;
    if (!tx || !ty) {
        int one_x = 0, one_y = 0;
        for (int c : {128, 256}) {
            if (tx && tx != c) continue;
            const int64_t per_strip = step2_slots(p.storage, c) / strips(c);
            if (per_strip < 1) continue;
            const int64_t h = (p.ny + per_strip - 1) / per_strip;
            if (h <= 48) {
                one_x = c;
                one_y = (int)h;
                break;
            }
        }
        if (one_x) {
            if (!tx) tx = one_x;
            if (!ty) ty = one_y;
        } else {
            if (!tx) tx = 256;
            if (!ty) {
                if (p.storage == LB_F16DEV) {
                    int64_t nr = 1;
                    while (fill(tx, nr) > 128) ++nr;
                    ty = (int)fill(tx, nr);
                } else if (fill(tx, 1) <= 96) {
                    ty = (int)fill(tx, 1);
                } else {
                    ty = 48;
                    const int64_t slots = step2_slots(p.storage, tx);
                    const int64_t tiles = strips(tx) * rows(48);
                    const int64_t rounds = (tiles + slots - 1) / slots;
                    const int64_t fit = fill(tx, rounds);
                    if (fit >= 44 && fit < 48)
                        ty = (int)fit;
                    else if (rounds > 1 && 2 * (tiles - (rounds - 1) * slots) < slots &&
                             fill(tx, rounds - 1) <= 56)
                        ty = (int)fill(tx, rounds - 1);
                }
            }
        }
    }
    g2.tile_x = tx;
    g2.tile_y = ty > p.ny ? p.ny : ty;
    const int w = g2.tile_x - 6;
    g2.tiles_x = (p.nx + w - 1) / w;
    g2.blocks = g2.tiles_x * ((p.ny + g2.tile_y - 1) / g2.tile_y);
    g2.rows_per_iter = 1;
    return g2;
}

// Tiles of at most w x h sites that cover an nx x ny lattice, rounded up to
// whole rounds of `slots` resident workgroups.
int64_t round_tiles(int nx, int ny, int w, int h, int64_t slots)
{
    const int64_t fewest = (int64_t)((nx + w - 1) / w) * ((ny + h - 1) / h);
    return (fewest + slots - 1) / slots * slots;
}

struct TileSplit {
    int tx, ty;
};

// The split into at most round_tiles tiles of at most w x h (and, unless the
// lattice itself is narrower, at least `least`) sites whose region, `halo`
// sites larger in both directions, is smallest.
TileSplit split_tiles(int nx, int ny, int w, int h, int least, int64_t slots, int halo)
{
    TileSplit s{};
    const int64_t tiles = round_tiles(nx, ny, w, h, slots);
    const int first = (nx + w - 1) / w;
    int64_t best = 0;
    for (int a = first; a <= tiles; ++a) {
        const int tx = (nx + a - 1) / a;
        if (tx < least && a > first) break;
        const int64_t rows = tiles / a;
        const int ty = (int)std::max<int64_t>(std::min(least, h), (ny + rows - 1) / rows);
        if (ty > h) break;
        const int64_t region = (int64_t)(tx + halo) * (ty + halo);
        if (best && region >= best) continue;
        best = region;
        s = TileSplit{tx, ty};
    }
    return s;
}

// Threads of the tiles of N sites, workgroups resident at once, most steps per
// launch, and the widest and tallest tile for k steps.
struct TileClass {
    bool large;  // double precision: two workgroups of 256 threads per CU
    int threads, steps;
    int64_t slots;
    TileClass(int64_t N, bool f64)
    {
        const bool round = N <= 256 * 34 * 36;  // one tile per CU
        const int64_t area = (N + 255) / 256;
        large = f64 && N > 1050000;
        threads = large ? 256 : f64 || round ? 1024 : 512;
        slots = !large && (f64 || round) ? 256 : 512;
        steps = area <= 24 ? 5 : area <= 112 ? 4 : large ? 2 : 3;
    }
    int width(int k) const { return large ? 24 : lbk::kTilePitch - 6 * k + 2; }
    int height(int k) const { return large ? 26 : lbk::kTileRows - 6 * k + 2; }
};

// The geometry of tiles of tx x ty sites (steps left open).
lbk::TileGeom tile_geom(const lb_params& p, const Geom& g, int tx, int ty, int threads)
{
    lbk::TileGeom t{};
    t.nx = p.nx;
    t.ny = p.ny;
    t.pitch = g.pitch;
    t.plane = g.plane;
    t.tx = tx;
    t.ty = ty;
    t.tiles_x = (p.nx + tx - 1) / tx;
    t.tiles = t.tiles_x * ((p.ny + ty - 1) / ty);
    t.threads = threads;
    for (int j = 0; j < lbk::kTileMaxSteps; ++j) {
        const uint32_t w = tx + 6 * j + 4;
        t.magic[j] = (uint32_t)(((uint64_t(1) << 32) + w - 1) / w);
    }
    return t;
}

// Whether 32-bit byte offsets reach all of a plane.
bool plane_fits(const lb_params& p, const Geom& g)
{
    return (uint64_t)g.plane * lbk::storage_bytes(p.storage) < (uint64_t(1) << 32);
}

// us per step of the row walk at one step per launch, and of the tiles, fitted to
// 488 timings of lattices and batches.  In both a wave takes about 0.35 ns per row or per
// site slot in single and 0.6 ns in double precision, once the launch's own time
// is taken off; a walk's waves also take four rows beyond its tile, and a round of
// tiles takes all the waves of its workgroups, however few sites they have.  A
// walk takes at least 0.85 (1.2) us for each row after the second, and neither
// kernel beats the memory, 4.9 TB/s: 9 values in and 9 out a site, and a part of
// the halo again, all of it where an XCD's run of the walk's tiles does not reach
// a tile's vertical neighbour.
struct WalkCost {
    bool f64;
    double waves = 0.0, bytes = 0.0;
    int rows = 0;
    explicit WalkCost(int storage) : f64(storage == LB_F64) {}
    void add(const Geom& g, int storage, bool alone)
    {
        waves += (double)g.blocks * (g.tile_x / 64) * (g.tile_y + 4);
        rows = std::max(rows, g.tile_y);
        const double again = alone && g.blocks < 16 * g.tiles_x ? 1.0 : 0.35;
        bytes += 9.0 * (2.0 + again * 4.0 / g.tile_y) * lbk::storage_bytes(storage) * g.nx * (double)g.ny;
    }
    double us() const
    {
        const double launch = f64 ? 6.0 : 4.0;
        return std::max({launch + (f64 ? 0.6e-3 : 0.35e-3) * waves, launch + (f64 ? 1.2 : 0.85) * (rows - 2), bytes / 4.9e6});
    }
};

// Launches of k steps on `tiles` tiles of at most tx x ty sites.
double tile_us(int storage, int64_t sites, int64_t tiles, int tx, int ty, int threads, int64_t slots, int k)
{
    int64_t site_slots = 0;  // of a thread, over the steps
    for (int j = 0; j < k; ++j) site_slots += ((tx + 6 * j + 4) * (ty + 6 * j + 4) + threads - 1) / threads;
    const double round = (storage == LB_F64 ? 0.9 : 0.6) + (storage == LB_F64 ? 0.6e-3 : 0.35e-3) * (double)(site_slots * slots * (threads / 64));
    const double launch = 3.5 + round * (double)((tiles + slots - 1) / slots);
    const double halo = (double)((tx + 6 * k - 2) * (ty + 6 * k - 2)) / (tx * ty) - 1.0;
    const double bytes = 9.0 * (2.0 + 0.5 * halo) * lbk::storage_bytes(storage) * (double)sites;
    return std::max(launch, bytes / 4.9e6) / k;
}

// Which launches of up to k steps the tiles take over from the walk: all while one
// round holds them; else those of several steps unless the estimate is 1.1 times
// the walk's, and those of one step, which share no launch and no load, where it
// is `one` of it: 0.93 in a batch (FP64 two of 900^2 51 on tiles and 61 in the walk,
// two of 1200^2 115 and 101, 900 of 32^2 70 and 62), for a lattice 0.95, or 0.85 from
// 850 000 sites on (FP32 900^2 14.1 and 15.1, 948^2 15.8 and 14.9, 100 x 9000 19.0
// and 27.8).  us/step of several per launch on tiles and in the walk: 60000 x 5 in
// FP32 27.4 and 11.3, FP64 60000 x 11 40.5 and 30.2, 20000 x 30 in FP32 10.6 and
// 13.9; batches in FP32, 1000 lattices of 8^2 26.6 and 12.0, 500 of 16^2 13.9 and
// 12.2, 300 of 24^2 9.8 and 11.4 (13.7 and 11.3 at one step per call).
struct TileUse {
    int steps = 0;
    bool single = false;
    TileUse(int storage, int64_t sites, int64_t tiles, int tx, int ty, const TileClass& c, int k, const WalkCost& walk,
            double one)
    {
        auto gain = [&](int j, double most) {
            return tiles <= c.slots || tile_us(storage, sites, tiles, tx, ty, c.threads, c.slots, j) <= most * walk.us();
        };
        single = gain(1, one);
        steps = k > 1 ? (gain(k, 1.1) ? k : 0) : single;
    }
};

// Plain steps of several levels per launch (lb_tile.hip), for lattices that
// do not run two per launch in the row walk.
struct TilePlan {
    lbk::TileGeom g;
    int steps;       // most steps of a launch; 0: not used
    bool single;     // also where one step is left
};

// The tile: about one per CU (256) while that keeps it within the region a
// workgroup can hold, else a whole number of rounds of the workgroups that
// are resident at once, so that no round runs partly empty.  Steps per launch
// by the tile's area: the halo of a step costs three sites on every side, so
// small tiles, whose time is the launch's, take more steps than large ones.
// Measured us/step (tile, steps): FP32 64^2 4x4 5 steps 1.96, 4 2.04; 128^2
// 8x8 4 2.19, 3 2.30; 256^2 16x16 3 2.53, 4 2.60; 448^2 28x28 3 3.82, 2
// 4.20; 512^2 32x32 2 4.50, 24x24 3 5.16; 768^2 34x35 2 in two rounds' worth
// 7.91, 24x24 in four 7.92; 1100^2 34x36 2 13.6, two per launch in the row
// walk 15.9; 1200^2 16.3 against 15.8, 1300^2 18.1 against 17.2.
// FP64 above about 1000^2 takes tiles of up to 24 x 26 and 256 threads, two
// workgroups per CU, whose loads overlap each other's arithmetic: 1200^2 24x24
// (4.9 rounds) 33.4 and 24x26 (4.6) 36.1 against 35.4 for 34x34 tiles, 2048^2
// 98 against 111 (one step per launch 44 and 128).
TilePlan make_tile(const lb_params& p, const Geom& g)
{
    TilePlan t{};
    const int64_t N = (int64_t)p.nx * p.ny;
    if (p.steps_per_launch != 0 || p.tile_x || p.tile_y || p.tile_rows || !plane_fits(p, g)) return t;
    const TileClass c(N, p.storage == LB_F64);
    for (int k = c.steps; k >= 1; --k) {
        const int w = std::min(c.width(k), p.nx - 3 * k + 2), h = std::min(c.height(k), p.ny - 3 * k + 2);
        if (w < 4 || h < 4) continue;
        if (k == 3 && !c.large &&
            round_tiles(p.nx, p.ny, w, h, c.slots) > round_tiles(p.nx, p.ny, c.width(2), c.height(2), c.slots))
            continue;  // three steps only where they need no more rounds than two
        const TileSplit s = split_tiles(p.nx, p.ny, w, h, 4, c.slots, 6 * k - 2);
        if (!s.tx) continue;
        t.g = tile_geom(p, g, s.tx, s.ty, c.threads);
        WalkCost walk(p.storage);
        walk.add(g, p.storage, true);
        const TileUse use(p.storage, N, t.g.tiles, s.tx, s.ty, c, k, walk, N <= 850000 ? 0.95 : 0.85);
        t.steps = use.steps;
        t.single = use.single;
        return t;
    }
    return t;
}

// Whether plain steps run two per launch: FP32 or half storage when asked
// for (steps_per_launch = 2), and by default on lattices large enough for tiles of
// 8 rows or more, if a tile shape is given (512^2 in tiles of 128 x 32: 24.1
// us/step, one per launch 27.5), if the lattice does not run on lb_tile.hip's tiles
// (100000 x 8: 12.8, on tiles 24.6) or if there are 1.2 million sites.  Below that
// the tiles are about as fast or faster (us/step against two per launch: 900^2
// 11.1 and 12.0 in FP32, 12.3 and 12.6 in half storage; 1040^2 13.4 and 13.1, 13.6
// and 13.9), above it slower (1120^2 14.5 and 14.2, 15.7 and 14.5; 1140^2 16.1 and
// 14.2, 16.3 and 14.5).
bool use_two(const lb_params& p, const Geom& g, const Geom& g2)
{
    if (p.storage != LB_F32 && p.storage != LB_F16DEV) return false;
    if (p.steps_per_launch == 2) return true;
    return p.steps_per_launch == 0 && g2.tile_y >= 8 &&
           ((int64_t)p.nx * p.ny >= 1200000 || !make_tile(p, g).steps);
}

// The tile geometry of a launch of `steps` <= t.steps steps.
lbk::TileGeom tile_launch(const TilePlan& t, int steps)
{
    lbk::TileGeom g = t.g;
    g.steps = steps;
    return g;
}

// Steps of the next launch of a run of n: as few launches as `most` steps
// each allow, evenly.
int even_steps(int64_t n, int most)
{
    const int64_t launches = (n + most - 1) / most;
    return (int)((n + launches - 1) / launches);
}

// Steps of the next launch of a run of n plain steps on tiles; 0: one step in
// the row walk.
int tile_steps(const TilePlan& t, int64_t n)
{
    if (!t.steps || n < 1) return 0;
    const int k = even_steps(n, t.steps);
    return k > 1 || t.single ? k : 0;
}

// Workspace layout, each region 256-byte aligned.
struct Layout {
    size_t buf[2], partials, trace, scalars, staging, total;
};

Layout make_layout(const lb_params& p, const Geom& g)
{
    Layout L;
    const size_t pop = align_up((size_t)9 * g.plane * lbk::storage_bytes(p.storage));
    size_t off = 0;
    L.buf[0] = off; off += pop;
    L.buf[1] = off; off += pop;
    L.partials = off; off += align_up((size_t)g.blocks * 4 * sizeof(double));
    L.trace = off; off += align_up((size_t)p.trace_cap * 6 * sizeof(double));
    L.scalars = off; off += align_up(8 * sizeof(double));
    L.staging = off; off += align_up((size_t)3 * p.nx * p.ny * sizeof(double));
    L.total = off;
    return L;
}

}  // namespace

struct lb_ctx {
    lb_params p;
    Geom g;
    Geom g2;     // two-step launches: tile_x lanes make tile_x - 6 columns
    bool two;    // plain steps run two per launch where they can
    TilePlan tile;  // else several per launch on tiles, where that is faster
    Coef coef;
    int device;
    hipStream_t stream;
    char* ws;
    void* buf[2];
    int cur;
    double* partials;
    double* trace;
    double* scalars;
    double* staging;
    int64_t t;
    int64_t trace_rows;
    int64_t last_logged;
    lb_batch* batch;  // non-NULL for a lattice owned by a batch
};

struct lb_batch {
    std::vector<lb_ctx*> members;
    lbk::BatchLattice* desc;   // device
    int32_t* tile_lattice;     // device
    int32_t* tile_lattice2;    // device, two-step tiles (when two)
    lbk::TileBatch tile;       // tiles of several steps per launch
    int tile_steps;            // most of their steps; 0: not used
    bool tile_single;          // also for one step
    double* partials;          // device, 4 per tile
    int tiles, tiles2;
    bool two;                  // plain steps run two per launch
    bool two_may;              // or would with a height of the caller's
    bool tau1;                 // tau is 1 in every lattice
    int tile_y2;
    int storage, tile_x, rows_per_iter, min_tile_y;
    int device;
    hipStream_t stream;
    int parity;
    int64_t t, log_every, trace_cap, trace_rows, last_logged;
    bool use_graphs;
    std::map<std::pair<int64_t, int>, hipGraphExec_t> graphs;
    std::vector<lb_params> params;           // per lattice, as given to lb_batch_init
    std::vector<lbk::BatchLattice> host_desc;  // host copy of desc
    int tiles2_cap;                          // capacity of tile_lattice2
};

namespace {

std::mutex g_mu;
std::set<lb_ctx*> g_live;

int check_ctx(lb_ctx* c)
{
    std::lock_guard<std::mutex> lk(g_mu);
    if (!c || !g_live.count(c)) return fail(LB_ERR_STATE, "unknown or destroyed context");
    return LB_OK;
}

// Makes the context's device current for the duration of a call.
struct DeviceGuard {
    int prev = -1;
    hipError_t err = hipSuccess;
    explicit DeviceGuard(int dev)
    {
        err = hipGetDevice(&prev);
        if (err == hipSuccess && prev != dev) err = hipSetDevice(dev);
    }
    ~DeviceGuard()
    {
        int now = -1;
        if (prev >= 0 && hipGetDevice(&now) == hipSuccess && now != prev) (void)hipSetDevice(prev);
    }
};

int field_check_host(const double* v, int64_t n, bool positive, const char* name)
{
    for (int64_t i = 0; i < n; ++i) {
        if (!std::isfinite(v[i]) || (positive && !(v[i] > 0.0)))
            return fail(LB_ERR_INVALID, "%s[%lld] = %g is not %s", name, (long long)i, v[i],
                        positive ? "finite and > 0" : "finite");
    }
    return LB_OK;
}

// The same for device memory, through a copy: names the first bad value.
int field_check_device(const double* v, int64_t n, bool positive, const char* name, hipStream_t st)
{
    std::vector<double> host(n);
    hipError_t e = hipMemcpyAsync(host.data(), v, n * sizeof(double), hipMemcpyDeviceToHost, st);
    if (!e) e = hipStreamSynchronize(st);
    if (e) return hip_fail(e, "copy field");
    return field_check_host(host.data(), n, positive, name);
}

// The device's address of a caller's host memory if it is mapped (pinned), so
// that a kernel can store a result there; NULL for pageable memory.
double* mapped(double* host)
{
    void* d = nullptr;
    if (hipHostGetDevicePointer(&d, host, 0) == hipSuccess) return static_cast<double*>(d);
    (void)hipGetLastError();
    return nullptr;
}

int energy_row(lb_ctx* c, int mode, const void* src, void* dst, double* row)
{
    c->coef.step = (uint32_t)c->t;
    hipError_t e = lbk::launch_step(c->p.storage, mode, src, dst, c->g, c->coef, c->partials, c->stream);
    if (e != hipSuccess) return hip_fail(e, "step kernel launch");
    e = lbk::launch_final(c->partials, c->g.blocks, (double)c->t, 0.5 * (c->p.G1 + c->p.G2), row,
                          c->stream);
    if (e != hipSuccess) return hip_fail(e, "final reduction launch");
    return LB_OK;
}

bool rows_finite(const double* r, int64_t n)
{
    for (int64_t i = 0; i < n * 6; ++i)
        if (!std::isfinite(r[i])) return false;
    return true;
}

}  // namespace

extern "C" {

const char* lb_last_error(void) { return g_err.c_str(); }

int lb_validate(const lb_params* p) { return check_params(p); }

size_t lb_workspace_bytes(const lb_params* p)
{
    if (check_params(p) != LB_OK) return 0;
    const Geom g = make_geom(*p);
    return make_layout(*p, g).total;
}

int lb_launch_shape(const lb_params* p, int32_t* tile_x, int32_t* tile_y, int32_t* tile_rows,
                    int32_t* blocks)
{
    int rc = check_params(p);
    if (rc) return rc;
    const Geom g = make_geom(*p);
    if (tile_x) *tile_x = g.tile_x;
    if (tile_y) *tile_y = g.tile_y;
    if (tile_rows) *tile_rows = g.rows_per_iter;
    if (blocks) *blocks = g.blocks;
    return LB_OK;
}

int lb_two_step_shape(const lb_params* p, int32_t* tile_x, int32_t* tile_y, int32_t* blocks)
{
    int rc = check_params(p);
    if (rc) return rc;
    const Geom g = make_geom(*p), g2 = make_geom2(*p, g);
    const bool on = use_two(*p, g, g2);
    if (tile_x) *tile_x = on ? g2.tile_x : 0;
    if (tile_y) *tile_y = on ? g2.tile_y : 0;
    if (blocks) *blocks = on ? g2.blocks : 0;
    return LB_OK;
}

int lb_tables(const lb_params* p, int8_t cx[24], int8_t cy[24], double K[24], double KE[25])
{
    if (!p) return fail(LB_ERR_INVALID, "params is NULL");
    if (!cx || !cy || !K || !KE) return fail(LB_ERR_INVALID, "NULL output table");
    for (int k = 0; k < 24; ++k) {
        cx[k] = (int8_t)kLX[k];
        cy[k] = (int8_t)kLY[k];
        K[k] = coupling(k, p->G1, p->G2);
        KE[1 + k] = K[k];
    }
    KE[0] = p->G1 * kW0 + p->G2 * kPS0;
    return LB_OK;
}

int lb_init(lb_ctx** out, const lb_params* p, void* workspace, size_t bytes,
            const double* rho_init, const double* ux_init, const double* uy_init,
            int inputs_on_device, void* hip_stream)
{
    if (!out) return fail(LB_ERR_INVALID, "out is NULL");
    *out = nullptr;
    int rc = check_params(p);
    if (rc) return rc;
    if (!workspace) return fail(LB_ERR_INVALID, "workspace is NULL");
    if (reinterpret_cast<uintptr_t>(workspace) % kAlign)
        return fail(LB_ERR_INVALID, "workspace must be %zu-byte aligned", kAlign);
    if (!rho_init) return fail(LB_ERR_INVALID, "rho_init is NULL");
    const Geom g = make_geom(*p);
    const Layout L = make_layout(*p, g);
    if (bytes < L.total)
        return fail(LB_ERR_INVALID, "workspace too small: %zu < %zu bytes", bytes, L.total);
    const int64_t N = (int64_t)p->nx * p->ny;

    // Host inputs are validated right here; device inputs on the device.
    if (!inputs_on_device) {
        if ((rc = field_check_host(rho_init, N, true, "rho_init"))) return rc;
        if (ux_init && (rc = field_check_host(ux_init, N, false, "ux_init"))) return rc;
        if (uy_init && (rc = field_check_host(uy_init, N, false, "uy_init"))) return rc;
    }

    int ndev = 0;
    hipError_t e = hipGetDeviceCount(&ndev);
    if (e != hipSuccess || ndev <= 0) return fail(LB_ERR_HIP, "no HIP device available");
    int dev = 0;
    if ((e = hipGetDevice(&dev)) != hipSuccess) return hip_fail(e, "hipGetDevice");
    hipStream_t st = static_cast<hipStream_t>(hip_stream);

    if (inputs_on_device) {
        // Up to 20 000 sites a copy costs less than the check's launches (64^2 28.6
        // us for the whole call against 41, 128^2 38.6 and 40.9, 181^2 51.6 and 41.4).
        int bad = N <= 20000;
        if (!bad) {
            int* flag = reinterpret_cast<int*>(static_cast<char*>(workspace) + L.scalars);
            if ((e = lbk::launch_clear(flag, st)) || (e = lbk::launch_check(rho_init, N, true, flag, st)) ||
                (ux_init && (e = lbk::launch_check(ux_init, N, false, flag, st))) ||
                (uy_init && (e = lbk::launch_check(uy_init, N, false, flag, st))) ||
                (e = hipMemcpyAsync(&bad, flag, sizeof bad, hipMemcpyDeviceToHost, st)) ||
                (e = hipStreamSynchronize(st)))
                return hip_fail(e, "check initial fields");
        }
        if (bad && ((rc = field_check_device(rho_init, N, true, "rho_init", st)) ||
                    (ux_init && (rc = field_check_device(ux_init, N, false, "ux_init", st))) ||
                    (uy_init && (rc = field_check_device(uy_init, N, false, "uy_init", st)))))
            return rc;
    }

    lb_ctx* c = new lb_ctx();
    c->p = *p;
    c->g = g;
    c->g2 = make_geom2(*p, g);
    c->two = use_two(*p, g, c->g2);
    c->tile = c->two ? TilePlan{} : make_tile(*p, g);
    c->coef = make_coef(*p);
    c->device = dev;
    c->stream = st;
    c->ws = static_cast<char*>(workspace);
    c->buf[0] = c->ws + L.buf[0];
    c->buf[1] = c->ws + L.buf[1];
    c->cur = 0;
    c->partials = reinterpret_cast<double*>(c->ws + L.partials);
    c->trace = reinterpret_cast<double*>(c->ws + L.trace);
    c->scalars = reinterpret_cast<double*>(c->ws + L.scalars);
    c->staging = reinterpret_cast<double*>(c->ws + L.staging);
    c->t = 0;
    c->trace_rows = 0;
    c->last_logged = -1;
    c->batch = nullptr;

    const double *r = rho_init, *u = ux_init, *v = uy_init;
    if (!inputs_on_device) {
        double* sr = c->staging;
        double* su = c->staging + N;
        double* sv = c->staging + 2 * N;
        e = hipMemcpyAsync(sr, rho_init, N * sizeof(double), hipMemcpyHostToDevice, st);
        if (!e && ux_init) e = hipMemcpyAsync(su, ux_init, N * sizeof(double), hipMemcpyHostToDevice, st);
        if (!e && uy_init) e = hipMemcpyAsync(sv, uy_init, N * sizeof(double), hipMemcpyHostToDevice, st);
        if (e) {
            delete c;
            return hip_fail(e, "copy initial fields");
        }
        r = sr;
        u = ux_init ? su : nullptr;
        v = uy_init ? sv : nullptr;
    }
    if ((e = lbk::launch_init(p->storage, r, u, v, c->buf[0], g, c->coef, st)) ||
        (e = hipStreamSynchronize(st))) {
        delete c;
        return hip_fail(e, "init kernel");
    }
    {
        std::lock_guard<std::mutex> lk(g_mu);
        g_live.insert(c);
    }
    *out = c;
    return LB_OK;
}

int lb_step(lb_ctx* c, int64_t n)
{
    int rc = check_ctx(c);
    if (rc) return rc;
    if (c->batch) return fail(LB_ERR_STATE, "this lattice belongs to a batch: step it with lb_batch_step");
    if (n < 0) return fail(LB_ERR_INVALID, "n must be >= 0");
    if (n == 0) return LB_OK;
    const int64_t le = c->p.log_every;
    // Rows this call appends: log points in [t, t+n) not recorded yet.  The
    // state at t+n itself is recorded by the step that leaves it (or by
    // lb_trace), so that logging always rides on a step.
    int64_t need = 0;
    if (le > 0) {
        const int64_t first = (c->t + le - 1) / le * le;
        if (first < c->t + n) need = (c->t + n - 1 - first) / le + 1;
        if (c->last_logged == c->t && c->t % le == 0) --need;
    }
    if (c->trace_rows + need > c->p.trace_cap)
        return fail(LB_ERR_STATE, "trace full: %lld rows recorded, %lld more needed, capacity %lld",
                    (long long)c->trace_rows, (long long)need, (long long)c->p.trace_cap);
    DeviceGuard dg(c->device);
    if (dg.err) return hip_fail(dg.err, "select device");

    for (int64_t s = 0; s < n; ++s) {
        const void* src = c->buf[c->cur];
        void* dst = c->buf[c->cur ^ 1];
        const bool log = le > 0 && c->t % le == 0 && c->last_logged != c->t;
        if (!log && c->tile.steps) {
            int64_t run = n - s;  // plain steps up to the next logged one
            if (le > 0) run = std::min(run, le - c->t % le);
            if (const int k = tile_steps(c->tile, run)) {
                c->coef.step = (uint32_t)c->t;
                hipError_t e = lbk::launch_tile(c->p.storage, src, dst, tile_launch(c->tile, k), c->coef, nullptr,
                                                c->stream);
                if (e) return hip_fail(e, "tile kernel launch");
                c->cur ^= 1;
                c->t += k;
                s += k - 1;
                continue;
            }
        }
        // Two plain steps in one launch when neither state is logged.
        if (c->two && !log && s + 1 < n && !(le > 0 && (c->t + 1) % le == 0)) {
            c->coef.step = (uint32_t)c->t;
            hipError_t e = lbk::launch_step2(c->p.storage, src, dst, c->g2, c->coef, c->stream);
            if (e) return hip_fail(e, "two-step kernel launch");
            c->cur ^= 1;
            c->t += 2;
            ++s;
            continue;
        }
        if (log) {
            // The logged step, then the reduction of its partials into the
            // trace row.  If only the reduction fails to launch, the step
            // itself was issued: the context follows it, without the row.
            c->coef.step = (uint32_t)c->t;
            hipError_t e = lbk::launch_step(c->p.storage, lbk::MODE_STEP_ENERGY, src, dst, c->g,
                                            c->coef, c->partials, c->stream);
            if (e) return hip_fail(e, "step kernel launch");
            c->cur ^= 1;
            ++c->t;
            e = lbk::launch_final(c->partials, c->g.blocks, (double)(c->t - 1),
                                  0.5 * (c->p.G1 + c->p.G2), c->trace + c->trace_rows * 6, c->stream);
            if (e) return hip_fail(e, "final reduction launch");
            c->last_logged = c->t - 1;
            ++c->trace_rows;
            continue;
        } else {
            c->coef.step = (uint32_t)c->t;
            hipError_t e = lbk::launch_step(c->p.storage, lbk::MODE_STEP, src, dst, c->g, c->coef,
                                            c->partials, c->stream);
            if (e) return hip_fail(e, "step kernel launch");
        }
        c->cur ^= 1;
        ++c->t;
    }
    return LB_OK;
}

int lb_time(lb_ctx* c, int64_t* t)
{
    int rc = check_ctx(c);
    if (rc) return rc;
    if (!t) return fail(LB_ERR_INVALID, "t is NULL");
    *t = c->t;
    return LB_OK;
}

int lb_moments(lb_ctx* c, double* rho, double* ux, double* uy, int on_device)
{
    int rc = check_ctx(c);
    if (rc) return rc;
    DeviceGuard dg(c->device);
    if (dg.err) return hip_fail(dg.err, "select device");
    const int64_t N = (int64_t)c->p.nx * c->p.ny;
    hipError_t e;
    if (on_device) {
        if ((e = lbk::launch_moments(c->p.storage, c->buf[c->cur], c->g, c->coef, rho, ux, uy, c->stream)))
            return hip_fail(e, "moments kernel");
        return LB_OK;
    }
    double* s = c->staging;
    if ((e = lbk::launch_moments(c->p.storage, c->buf[c->cur], c->g, c->coef, rho ? s : nullptr,
                                 ux ? s + N : nullptr, uy ? s + 2 * N : nullptr, c->stream)))
        return hip_fail(e, "moments kernel");
    double* outs[3] = {rho, ux, uy};
    for (int q = 0; q < 3; ++q) {
        if (!outs[q]) continue;
        if ((e = hipMemcpyAsync(outs[q], s + q * N, N * sizeof(double), hipMemcpyDeviceToHost, c->stream)))
            return hip_fail(e, "copy moments");
    }
    if ((e = hipStreamSynchronize(c->stream))) return hip_fail(e, "synchronise");
    return LB_OK;
}

int lb_pseudo_energy(lb_ctx* c, double out[6])
{
    int rc = check_ctx(c);
    if (rc) return rc;
    if (!out) return fail(LB_ERR_INVALID, "out is NULL");
    DeviceGuard dg(c->device);
    if (dg.err) return hip_fail(dg.err, "select device");
    // Pinned output: the last kernel stores the row there, with no copy (one
    // step and the energies of a 96x80 lattice 33.6 -> 25.0 us).
    double* const row = mapped(out);
    if ((rc = energy_row(c, lbk::MODE_ENERGY, c->buf[c->cur], c->buf[c->cur ^ 1], row ? row : c->scalars)))
        return rc;
    hipError_t e = hipSuccess;
    if (!row) e = hipMemcpyAsync(out, c->scalars, 6 * sizeof(double), hipMemcpyDeviceToHost, c->stream);
    if (!e) e = hipStreamSynchronize(c->stream);
    if (e) return hip_fail(e, "copy energies");
    if (!rows_finite(out, 1)) return fail(LB_ERR_NONFINITE, "non-finite mass or energy at t = %lld", (long long)c->t);
    return LB_OK;
}

int lb_trace(lb_ctx* c, double* out, int64_t cap, int64_t* n_rows)
{
    int rc = check_ctx(c);
    if (rc) return rc;
    if (cap < 0 || (cap > 0 && !out)) return fail(LB_ERR_INVALID, "bad output buffer");
    DeviceGuard dg(c->device);
    if (dg.err) return hip_fail(dg.err, "select device");
    // Record the current state first if it is a log point not yet recorded
    // and the trace has room.
    const int64_t le = c->p.log_every;
    if (!c->batch && le > 0 && c->t % le == 0 && c->last_logged != c->t &&
        c->trace_rows < c->p.trace_cap) {
        if ((rc = energy_row(c, lbk::MODE_ENERGY, c->buf[c->cur], c->buf[c->cur ^ 1],
                             c->trace + c->trace_rows * 6)))
            return rc;
        c->last_logged = c->t;
        ++c->trace_rows;
    }
    const int64_t rows = cap < c->trace_rows ? cap : c->trace_rows;
    hipError_t e = hipSuccess;
    if (rows > 0)
        e = hipMemcpyAsync(out, c->trace, rows * 6 * sizeof(double), hipMemcpyDeviceToHost, c->stream);
    if (!e) e = hipStreamSynchronize(c->stream);
    if (e) return hip_fail(e, "copy trace");
    if (n_rows) *n_rows = c->trace_rows;
    if (!rows_finite(out, rows)) return fail(LB_ERR_NONFINITE, "non-finite value in the trace");
    return LB_OK;
}

int lb_get_state(lb_ctx* c, void* dst, int on_device)
{
    int rc = check_ctx(c);
    if (rc) return rc;
    if (!dst) return fail(LB_ERR_INVALID, "dst is NULL");
    DeviceGuard dg(c->device);
    if (dg.err) return hip_fail(dg.err, "select device");
    const size_t bytes = (size_t)9 * c->p.nx * c->p.ny * lbk::storage_bytes(c->p.storage);
    void* spare = c->buf[c->cur ^ 1];
    hipError_t e = lbk::launch_get_state(c->p.storage, c->buf[c->cur], on_device ? dst : spare, c->g, c->stream);
    if (e) return hip_fail(e, "state kernel");
    if (!on_device) {
        if ((e = hipMemcpyAsync(dst, spare, bytes, hipMemcpyDeviceToHost, c->stream)) ||
            (e = hipStreamSynchronize(c->stream)))
            return hip_fail(e, "copy state");
    }
    return LB_OK;
}

int lb_set_state(lb_ctx* c, const void* src, int on_device, int64_t t)
{
    int rc = check_ctx(c);
    if (rc) return rc;
    if (c->batch) return fail(LB_ERR_STATE, "this lattice belongs to a batch");
    if (!src) return fail(LB_ERR_INVALID, "src is NULL");
    if (t < 0) return fail(LB_ERR_INVALID, "t must be >= 0");
    DeviceGuard dg(c->device);
    if (dg.err) return hip_fail(dg.err, "select device");
    const size_t bytes = (size_t)9 * c->p.nx * c->p.ny * lbk::storage_bytes(c->p.storage);
    void* spare = c->buf[c->cur ^ 1];
    hipError_t e = hipSuccess;
    const void* in = src;
    if (!on_device) {
        if ((e = hipMemcpyAsync(spare, src, bytes, hipMemcpyHostToDevice, c->stream)))
            return hip_fail(e, "copy state");
        in = spare;
    }
    // The permutation must not read and write one buffer: when the input was
    // staged in the spare buffer, write into the current one, else either.
    if ((e = lbk::launch_set_state(c->p.storage, in, c->buf[c->cur], c->g, c->stream)) ||
        (e = hipStreamSynchronize(c->stream)))
        return hip_fail(e, "state kernel");
    c->t = t;
    c->last_logged = -1;
    return LB_OK;
}

int lb_pseudo_energy_state(const lb_params* p, const void* state, double t, double out[6],
                           void* hip_stream)
{
    int rc = check_params(p);
    if (rc) return rc;
    if (!state) return fail(LB_ERR_INVALID, "state is NULL");
    if (!out) return fail(LB_ERR_INVALID, "out is NULL");
    if (!std::isfinite(t)) return fail(LB_ERR_INVALID, "t must be finite");
    int ndev = 0;
    hipError_t e = hipGetDeviceCount(&ndev);
    if (e != hipSuccess || ndev <= 0) return fail(LB_ERR_HIP, "no HIP device available");
    e = lbk::noalloc_energy(p->storage, state, p->nx, p->ny, make_coef(*p), t, 0.5 * (p->G1 + p->G2),
                            out, static_cast<hipStream_t>(hip_stream));
    if (e) return hip_fail(e, "energy of a population array");
    if (!rows_finite(out, 1)) return fail(LB_ERR_NONFINITE, "non-finite mass or energy");
    return LB_OK;
}

int lb_destroy(lb_ctx* c)
{
    {
        std::lock_guard<std::mutex> lk(g_mu);
        if (!c || !g_live.count(c)) return fail(LB_ERR_STATE, "unknown or destroyed context");
        if (c->batch) return fail(LB_ERR_STATE, "this lattice belongs to a batch: use lb_batch_destroy");
        g_live.erase(c);
    }
    DeviceGuard dg(c->device);
    hipError_t e = hipStreamSynchronize(c->stream);
    delete c;
    if (e) return hip_fail(e, "synchronise");
    return LB_OK;
}

// ---------------------------------------------------------------------------
// Batches of independent lattices.
// ---------------------------------------------------------------------------
namespace {

std::set<lb_batch*> g_batches;

int check_batch(lb_batch* b)
{
    std::lock_guard<std::mutex> lk(g_mu);
    if (!b || !g_batches.count(b)) return fail(LB_ERR_STATE, "unknown or destroyed batch");
    return LB_OK;
}

// Tiles of several steps per launch for a batch that does not run two in the
// row walk: the smallest tile, shared by the lattices as far as their own
// sizes allow, whose count fills no more rounds than the largest would.
struct BatchTiles {
    int steps, tx, ty, threads, tiles;
    bool single;  // also for one step
    std::vector<lbk::TileGeom> geom;
};

void batch_tiles(const lb_params* ps, int32_t count, BatchTiles& t)
{
    int64_t N = 0;
    int least = INT32_MAX;
    WalkCost walk(ps[0].storage);
    for (int32_t i = 0; i < count; ++i) {
        const Geom g = make_geom(ps[i]);
        N += (int64_t)ps[i].nx * ps[i].ny;
        least = std::min({least, ps[i].nx, ps[i].ny});
        if (!plane_fits(ps[i], g)) return;
        walk.add(g, ps[i].storage, count == 1);
    }
    const TileClass c(N, ps[0].storage == LB_F64);
    auto tiles = [&](int k, int w, int h) {
        int64_t n = 0;
        for (int32_t i = 0; i < count; ++i) {
            const int a = std::min(w, ps[i].nx - 3 * k + 2), b = std::min(h, ps[i].ny - 3 * k + 2);
            n += (int64_t)((ps[i].nx + a - 1) / a) * ((ps[i].ny + b - 1) / b);
        }
        return n;
    };
    auto rounds = [&](int64_t n) { return (n + c.slots - 1) / c.slots; };
    for (int k = c.steps; k >= 1; --k) {
        if (least - 3 * k + 2 < 4) continue;
        const int w = c.width(k), h = c.height(k);
        const int64_t most = rounds(tiles(k, w, h));
        if (k == 3 && !c.large && most > rounds(tiles(2, c.width(2), c.height(2)))) continue;
        int side = w;
        while (side > 4 && rounds(tiles(k, side - 1, std::min(h, side - 1))) <= most) --side;
        if (tiles(k, side, std::min(h, side)) >= (int64_t(1) << 30)) return;
        t.steps = k;
        t.threads = c.threads;
        for (int32_t i = 0; i < count; ++i) {
            const int a = std::min(side, ps[i].nx - 3 * k + 2), b = std::min({side, h, ps[i].ny - 3 * k + 2});
            const int na = (ps[i].nx + a - 1) / a, nb = (ps[i].ny + b - 1) / b;
            t.geom.push_back(tile_geom(ps[i], make_geom(ps[i]), (ps[i].nx + na - 1) / na, (ps[i].ny + nb - 1) / nb,
                                       c.threads));
            t.tiles += t.geom.back().tiles;
            t.tx = std::max(t.tx, t.geom.back().tx);
            t.ty = std::max(t.ty, t.geom.back().ty);
        }
        const TileUse use(ps[0].storage, N, t.tiles, t.tx, t.ty, c, k, walk, 0.93);
        if (!use.steps) t = BatchTiles{};
        t.single = use.single;
        return;
    }
}

// Workspace of a batch: descriptor table, tile -> lattice table, partials,
// then one single-lattice workspace per member.
struct BatchLayout {
    size_t desc, tile_lattice, tile_lattice2, tile_lattice3, partials;
    BatchTiles tile;
    std::vector<size_t> member, member_bytes;
    size_t total;
    int tiles, tiles2, tiles2_cap, tile_y2;
    bool two;      // plain steps run two per launch
    bool two_may;  // or would with a height of the caller's
    std::vector<Geom> geom2;
};

// Smallest two-step tile height of a batch: the two-step tile table is
// sized for it, so the height can change after initialisation.
constexpr int kBatchMinTile2 = 8;
constexpr int kBatchMaxTile2 = 64;

// Two-step geometry of a batch member: tiles of kBatchLanes2 lanes and a tile
// height shared by the batch.
Geom batch_geom2(const lb_params& p, int tile_y2)
{
    lb_params q = p;
    q.tile_x = lbk::kBatchLanes2;
    q.tile_y = std::min(tile_y2, p.ny);
    return make_geom2(q, make_geom(q));
}

// Height of the two-step tiles of a batch.  A workgroup walks its height and 7
// rows more; a round of resident workgroups takes about as long per row whether
// it is full or half empty (full: 1.1 times in single precision, 1.05 in half
// storage).  So the height is the one of least rounds x rows: the model ranks
// heights as measured, though their times differ by less than half of what it
// says, for the memory's share.  In single precision up to 48 rows: taller tiles
// are faster for a batch alone, slower for several at once.  Measured us/step
// (alone; three batches on three streams): 20 lattices of 9.1 million sites in
// FP32 16 rows (3.3 rounds of 1536) 101, 89.2; 20 (2.7) 97.0, 86.7; 28 (1.9) 94.1,
// 85.5; 48 (1.1) 110, 86.0; 56 (0.98) 86.4, 87.2; 64 (0.86) 90.6, 86.8; half storage
// 28 68.6, 65.6; 48 88.8, 62.6; 56 62.5, 61.4; 64 68.5, 60.8.  13 lattices of 4.8
// million: FP32 24 (1.1) 58.0, 44.4; 28 (0.96) 45.1, 44.6; 48 50.7, 44.7; half
// storage 51.5, 35.8; 36.3, 34.0; 44.8, 32.9.
int batch_height2(const lb_params* ps, int32_t count)
{
    const int64_t slots = step2_slots(ps[0].storage, lbk::kBatchLanes2);
    const double full = ps[0].storage == LB_F32 ? 1.1 : 1.05;
    const int most = ps[0].storage == LB_F32 ? 48 : kBatchMaxTile2;
    std::vector<std::pair<int, int>> strips(count);  // a lattice's strips and rows
    for (int32_t i = 0; i < count; ++i) strips[i] = {batch_geom2(ps[i], kBatchMinTile2).tiles_x, ps[i].ny};
    int best = kBatchMinTile2;
    double least = 0.0;
    for (int h = kBatchMinTile2; h <= most; ++h) {
        int64_t tiles = 0;
        for (const auto& [across, ny] : strips) tiles += (int64_t)across * ((ny + h - 1) / h);
        const int64_t rounds = tiles / slots, rest = tiles % slots;
        const double cost = (h + 7) * (full * (double)rounds +
                                       (rest ? std::max(1.0, full * (double)rest / (double)slots) : 0.0));
        if (h == kBatchMinTile2 || cost < least) {
            least = cost;
            best = h;
        }
    }
    return best;
}

int batch_layout(const lb_params* ps, int32_t count, BatchLayout* L)
{
    L->tile = BatchTiles{};
    if (!ps) return fail(LB_ERR_INVALID, "params is NULL");
    if (count < 1 || count > 65536) return fail(LB_ERR_INVALID, "count must be in [1, 65536]");
    int rc;
    L->tiles = 0;
    Geom g0{};
    for (int32_t i = 0; i < count; ++i) {
        if ((rc = check_params(&ps[i]))) {
            return fail(rc, "lattice %d: %s", i, g_err.c_str());
        }
        const Geom g = make_geom(ps[i]);
        if (i == 0) g0 = g;
        if (ps[i].storage != ps[0].storage || g.tile_x != g0.tile_x ||
            g.rows_per_iter != g0.rows_per_iter || ps[i].log_every != ps[0].log_every ||
            ps[i].trace_cap != ps[0].trace_cap)
            return fail(LB_ERR_INVALID,
                        "lattice %d: storage, tile_x, tile_rows, log_every and trace_cap must "
                        "match lattice 0", i);
        if (ps[i].steps_per_launch != ps[0].steps_per_launch)
            return fail(LB_ERR_INVALID, "lattice %d: steps_per_launch must match lattice 0", i);
        if ((int64_t)L->tiles + g.blocks >= (int64_t(1) << 30))
            return fail(LB_ERR_INVALID, "too many tiles in the batch");
        L->tiles += g.blocks;
    }
    // Two steps per launch in the row walk: FP32 or half storage, by default
    // for a million sites and more.  Below that the tiles of batch_tiles are
    // faster: us/step, 0.61 million sites 10.6 against 12.2 in FP32, 11.4 against
    // 12.9 in half storage; 0.72 million 10.9 against 12.9, 12.1 against 13.8;
    // 1.2 million 16.8 against 15.6, 17.6 against 16.8.
    const int spl = ps[0].steps_per_launch;
    const int st = ps[0].storage;
    int64_t sites = 0;
    for (int32_t i = 0; i < count; ++i) sites += (int64_t)ps[i].nx * ps[i].ny;
    L->two = (st == LB_F32 || st == LB_F16DEV) && (spl == 2 || (spl == 0 && sites >= 1000000));
    // Batches of many lattices that fill 1400 workgroups of 16 rows take a height
    // too, and two steps per launch with it, though tiles are faster.
    L->two_may = L->two;
    if (spl == 0 && st != LB_F64 && !L->two) {
        int64_t low = 0;
        for (int32_t i = 0; i < count; ++i) low += batch_geom2(ps[i], 16).blocks;
        L->two_may = low >= 1400;
    }
    L->tile_y2 = L->two ? batch_height2(ps, count) : 0;
    L->tiles2 = 0;
    L->tiles2_cap = 0;
    L->geom2.assign(count, Geom{});
    for (int32_t i = 0; i < count; ++i) {
        if (L->two) {
            L->geom2[i] = batch_geom2(ps[i], L->tile_y2);
            L->tiles2 += L->geom2[i].blocks;
        }
        if (L->two_may) L->tiles2_cap += batch_geom2(ps[i], kBatchMinTile2).blocks;
    }
    if ((int64_t)L->tiles2_cap >= (int64_t(1) << 30))
        return fail(LB_ERR_INVALID, "too many two-step tiles in the batch");
    size_t off = 0;
    L->desc = off;
    off += align_up(sizeof(lbk::BatchLattice) * count);
    L->tile_lattice = off;
    off += align_up(sizeof(int32_t) * L->tiles);
    L->tile_lattice2 = off;
    off += align_up(sizeof(int32_t) * L->tiles2_cap);
    if (spl == 0 && !L->two) batch_tiles(ps, count, L->tile);
    L->tile_lattice3 = off;
    off += align_up(sizeof(int32_t) * L->tile.tiles);
    L->partials = off;
    off += align_up(sizeof(double) * 4 * L->tiles);
    L->member.resize(count);
    L->member_bytes.resize(count);
    for (int32_t i = 0; i < count; ++i) {
        L->member[i] = off;
        L->member_bytes[i] = make_layout(ps[i], make_geom(ps[i])).total;
        off += L->member_bytes[i];
    }
    L->total = off;
    return LB_OK;
}

// One step of every lattice from buf[parity]; t is the step's time level
// (it seeds the half storage's stochastic rounding).
hipError_t batch_launch(lb_batch* b, int mode, int parity, int64_t t)
{
    return lbk::launch_step_batch(b->storage, mode, b->tile_x, b->rows_per_iter, b->min_tile_y, b->desc,
                                  b->tile_lattice, b->tiles, parity, (uint32_t)t, b->partials,
                                  b->stream);
}

// Steps of the next launch of a run of n plain steps.
int batch_steps(const lb_batch* b, int64_t n)
{
    if (b->tile_steps) return even_steps(n, b->tile_steps);
    return b->two && n > 1 ? 2 : 1;
}

// Buffer flips of the first m steps of a run of n plain steps: one per launch.
int batch_flips(const lb_batch* b, int64_t n, int64_t m)
{
    int flips = 0;
    for (int64_t j = 0; j < m; ++flips) j += batch_steps(b, n - j);
    return flips & 1;
}

// n plain steps from buf[parity] at time t, launch by launch: on tiles, or
// pairs in the two-step kernel and then any odd step, or one by one.  *done
// counts the steps whose launch was issued (all n unless one fails).
hipError_t batch_run(lb_batch* b, int64_t n, int parity, int64_t t, int64_t* done)
{
    for (*done = 0; *done < n; parity ^= 1) {
        const int k = batch_steps(b, n - *done);
        const int64_t now = t + *done;
        hipError_t e;
        if (b->tile_steps && (k > 1 || b->tile_single)) {
            lbk::TileBatch launch = b->tile;
            launch.parity = parity;
            launch.steps = k;
            launch.step = (uint32_t)now;
            e = lbk::launch_tile_batch(b->storage, launch, b->stream);
        } else if (k == 2) {
            e = lbk::launch_step2_batch(b->storage, b->tau1, b->desc, b->tile_lattice2, b->tiles2, parity,
                                        (uint32_t)now, b->stream);
        } else {
            e = batch_launch(b, lbk::MODE_STEP, parity, now);
        }
        if (e != hipSuccess) return e;
        *done += k;
    }
    return hipSuccess;
}

// n plain steps starting from the current parity, as one replay of a
// captured graph when the stream allows capture, else launch by launch.
// A graph keeps the time levels it was captured with, so batches whose
// rounding depends on them (half storage) never use graphs.  *done counts
// the steps issued.
hipError_t batch_plain(lb_batch* b, int64_t n, int64_t* done)
{
    *done = 0;
    if (b->use_graphs && n >= 2) {
        const auto key = std::make_pair(n, b->parity);
        auto it = b->graphs.find(key);
        if (it == b->graphs.end()) {
            hipGraph_t graph = nullptr;
            hipGraphExec_t exec = nullptr;
            hipError_t e = hipStreamBeginCapture(b->stream, hipStreamCaptureModeThreadLocal);
            if (e == hipSuccess) {
                int64_t captured = 0;
                const hipError_t le = batch_run(b, n, b->parity, b->t, &captured);
                e = hipStreamEndCapture(b->stream, &graph);
                if (e == hipSuccess && le != hipSuccess) e = le;
            }
            if (e == hipSuccess) e = hipGraphInstantiate(&exec, graph, nullptr, nullptr, 0);
            if (graph) (void)hipGraphDestroy(graph);
            if (e != hipSuccess) {
                // This stream cannot be captured: run launch by launch from now on.
                (void)hipGetLastError();
                b->use_graphs = false;
                return batch_plain(b, n, done);
            }
            it = b->graphs.emplace(key, exec).first;
        }
        const hipError_t e = hipGraphLaunch(it->second, b->stream);
        if (e == hipSuccess) *done = n;
        return e;
    }
    return batch_run(b, n, b->parity, b->t, done);
}

int batch_log(lb_batch* b, int mode)
{
    hipError_t e = batch_launch(b, mode, b->parity, b->t);
    if (!e)
        e = lbk::launch_final_batch(b->desc, (int)b->members.size(), b->partials, (double)b->t,
                                    b->trace_rows, b->stream);
    if (e) return hip_fail(e, "batched energy launch");
    b->last_logged = b->t;
    ++b->trace_rows;
    return LB_OK;
}

// n steps of the batch, logging where due; the batch's time level and
// parity follow every launch that was issued.
int batch_advance(lb_batch* b, int64_t n)
{
    const int64_t le = b->log_every;
    int rc;
    int64_t done = 0;
    while (done < n) {
        if (le > 0 && b->t % le == 0 && b->last_logged != b->t) {
            hipError_t e = batch_launch(b, lbk::MODE_STEP_ENERGY, b->parity, b->t);
            if (e) return hip_fail(e, "batched energy launch");
            b->parity ^= 1;
            ++b->t;
            ++done;
            e = lbk::launch_final_batch(b->desc, (int)b->members.size(), b->partials,
                                        (double)(b->t - 1), b->trace_rows, b->stream);
            if (e) return hip_fail(e, "batched energy reduction launch");
            b->last_logged = b->t - 1;
            ++b->trace_rows;
            continue;
        }
        int64_t run = n - done;
        if (le > 0) {
            const int64_t next = (b->t / le + 1) * le;
            if (next - b->t < run) run = next - b->t;
        }
        int64_t issued = 0;
        hipError_t e = batch_plain(b, run, &issued);
        b->parity ^= batch_flips(b, run, issued);
        b->t += issued;
        done += issued;
        if (e) return hip_fail(e, "batched step launch");
    }
    if (le > 0 && b->t % le == 0 && b->last_logged != b->t)
        if ((rc = batch_log(b, lbk::MODE_ENERGY))) return rc;
    return LB_OK;
}

void batch_sync_members(lb_batch* b)
{
    for (lb_ctx* c : b->members) {
        c->t = b->t;
        c->cur = b->parity;
        c->trace_rows = b->trace_rows;
        c->last_logged = b->last_logged;
    }
}

}  // namespace

size_t lb_batch_workspace_bytes(const lb_params* ps, int32_t count)
{
    BatchLayout L;
    if (batch_layout(ps, count, &L) != LB_OK) return 0;
    return L.total;
}

int lb_batch_init(lb_batch** out, const lb_params* ps, int32_t count, void* workspace,
                  size_t bytes, const double* const* rho_init, int inputs_on_device,
                  void* hip_stream)
{
    if (!out) return fail(LB_ERR_INVALID, "out is NULL");
    *out = nullptr;
    BatchLayout L;
    int rc = batch_layout(ps, count, &L);
    if (rc) return rc;
    if (!workspace) return fail(LB_ERR_INVALID, "workspace is NULL");
    if (reinterpret_cast<uintptr_t>(workspace) % kAlign)
        return fail(LB_ERR_INVALID, "workspace must be %zu-byte aligned", kAlign);
    if (bytes < L.total) return fail(LB_ERR_INVALID, "workspace too small: %zu < %zu bytes", bytes, L.total);
    if (!rho_init) return fail(LB_ERR_INVALID, "rho_init is NULL");
    for (int32_t i = 0; i < count; ++i)
        if (!rho_init[i]) return fail(LB_ERR_INVALID, "rho_init[%d] is NULL", i);

    char* ws = static_cast<char*>(workspace);
    lb_batch* b = new lb_batch();
    b->stream = static_cast<hipStream_t>(hip_stream);
    std::vector<lbk::BatchLattice> desc(count);
    std::vector<int32_t> tl(L.tiles), tl2(L.tiles2), tl3;
    tl3.reserve(L.tile.tiles);
    int tile = 0, tile2 = 0;
    for (int32_t i = 0; i < count; ++i) {
        lb_ctx* c = nullptr;
        rc = lb_init(&c, &ps[i], ws + L.member[i], L.member_bytes[i], rho_init[i], nullptr, nullptr,
                     inputs_on_device, hip_stream);
        if (rc) {
            std::string msg = g_err;
            for (lb_ctx* m : b->members) {
                m->batch = nullptr;
                lb_destroy(m);
            }
            delete b;
            return fail(rc, "lattice %d: %s", i, msg.c_str());
        }
        c->batch = b;
        b->members.push_back(c);
        lbk::BatchLattice& d = desc[i];
        std::memset(static_cast<void*>(&d), 0, sizeof d);
        d.geom = c->g;
        d.coef = c->coef;
        lbk::coef_to_f32(c->coef, d.coef_f);
        d.buf[0] = c->buf[0];
        d.buf[1] = c->buf[1];
        d.trace = c->trace;
        d.half_A1 = 0.5 * (ps[i].G1 + ps[i].G2);
        d.tile_begin = tile;
        for (int j = 0; j < c->g.blocks; ++j) tl[tile + j] = i;
        tile += c->g.blocks;
        if (L.two) {
            d.geom2 = L.geom2[i];
            d.tile_begin2 = tile2;
            for (int j = 0; j < d.geom2.blocks; ++j) tl2[tile2 + j] = i;
            tile2 += d.geom2.blocks;
        }
        if (L.tile.steps) {
            d.tile = L.tile.geom[i];
            d.tile_begin3 = (int32_t)tl3.size();
            tl3.insert(tl3.end(), d.tile.tiles, i);
        }
    }
    lb_ctx* c0 = b->members[0];
    b->desc = reinterpret_cast<lbk::BatchLattice*>(ws + L.desc);
    b->tile_lattice = reinterpret_cast<int32_t*>(ws + L.tile_lattice);
    b->tile_lattice2 = reinterpret_cast<int32_t*>(ws + L.tile_lattice2);
    b->tile = lbk::TileBatch{};
    b->tile.desc = b->desc;
    b->tile.tile_lattice = reinterpret_cast<int32_t*>(ws + L.tile_lattice3);
    b->tile.tiles = L.tile.tiles;
    b->tile.tx = L.tile.tx;
    b->tile.ty = L.tile.ty;
    b->tile.threads = L.tile.threads;
    b->tile.tau1 = std::all_of(ps, ps + count, [](const lb_params& p) { return 1.0 / p.tau == 1.0; });
    b->tile_steps = L.tile.steps;
    b->tile_single = L.tile.single;
    b->partials = reinterpret_cast<double*>(ws + L.partials);
    b->tiles = L.tiles;
    b->tiles2 = L.tiles2;
    b->two = L.two;
    b->two_may = L.two_may;
    b->tau1 = b->tile.tau1;
    b->tile_y2 = L.tile_y2;
    b->storage = ps[0].storage;
    b->tile_x = c0->g.tile_x;
    b->min_tile_y = c0->g.tile_y;
    for (lb_ctx* m : b->members) b->min_tile_y = std::min(b->min_tile_y, m->g.tile_y);
    b->rows_per_iter = c0->g.rows_per_iter;
    b->device = c0->device;
    b->parity = 0;
    b->t = 0;
    b->log_every = ps[0].log_every;
    b->trace_cap = ps[0].trace_cap;
    b->trace_rows = 0;
    b->last_logged = -1;
    b->use_graphs = b->stream != nullptr && b->storage != LB_F16DEV;
    b->params.assign(ps, ps + count);
    b->host_desc = desc;
    b->tiles2_cap = L.tiles2_cap;
    hipError_t e = hipMemcpyAsync(b->desc, desc.data(), sizeof(lbk::BatchLattice) * count,
                                  hipMemcpyHostToDevice, b->stream);
    if (!e) e = hipMemcpyAsync(b->tile_lattice, tl.data(), sizeof(int32_t) * L.tiles,
                               hipMemcpyHostToDevice, b->stream);
    if (!e && L.tiles2)
        e = hipMemcpyAsync(b->tile_lattice2, tl2.data(), sizeof(int32_t) * L.tiles2,
                           hipMemcpyHostToDevice, b->stream);
    if (!e && !tl3.empty())
        e = hipMemcpyAsync(ws + L.tile_lattice3, tl3.data(), sizeof(int32_t) * tl3.size(), hipMemcpyHostToDevice,
                           b->stream);
    if (!e) e = hipStreamSynchronize(b->stream);
    if (e) {
        for (lb_ctx* m : b->members) {
            m->batch = nullptr;
            lb_destroy(m);
        }
        delete b;
        return hip_fail(e, "copy batch tables");
    }
    {
        std::lock_guard<std::mutex> lk(g_mu);
        g_batches.insert(b);
    }
    *out = b;
    return LB_OK;
}

int lb_batch_step(lb_batch* b, int64_t n)
{
    int rc = check_batch(b);
    if (rc) return rc;
    if (n < 0) return fail(LB_ERR_INVALID, "n must be >= 0");
    const int64_t le = b->log_every;
    // Rows this call appends: log points in [t, t+n] not recorded yet (the
    // state reached at t+n is recorded too).
    int64_t need = 0;
    if (le > 0) {
        const int64_t first = (b->t + le - 1) / le * le;
        if (first <= b->t + n) need = (b->t + n - first) / le + 1;
        if (b->last_logged == b->t && b->t % le == 0) --need;
    }
    if (b->trace_rows + need > b->trace_cap)
        return fail(LB_ERR_STATE, "trace full: %lld rows recorded, %lld more needed, capacity %lld",
                    (long long)b->trace_rows, (long long)need, (long long)b->trace_cap);
    DeviceGuard dg(b->device);
    if (dg.err) return hip_fail(dg.err, "select device");
    // On a launch failure the steps issued before it stand: the batch and
    // its member contexts are left at the time level they reached.
    rc = batch_advance(b, n);
    batch_sync_members(b);
    return rc;
}

int lb_batch_use_graphs(lb_batch* b, int enable)
{
    int rc = check_batch(b);
    if (rc) return rc;
    if (enable && !b->stream)
        return fail(LB_ERR_INVALID, "the null stream cannot be captured into a graph");
    if (enable && b->storage == LB_F16DEV)
        return fail(LB_ERR_INVALID, "half-storage batches seed their rounding with the time "
                                    "level and cannot replay captured graphs");
    b->use_graphs = enable != 0;
    return LB_OK;
}

int lb_batch_two_step_shape(lb_batch* b, int32_t* tile_x, int32_t* tile_y, int32_t* blocks)
{
    int rc = check_batch(b);
    if (rc) return rc;
    if (tile_x) *tile_x = b->two ? lbk::kBatchLanes2 : 0;
    if (tile_y) *tile_y = b->two ? b->tile_y2 : 0;
    if (blocks) *blocks = b->two ? b->tiles2 : 0;
    return LB_OK;
}

int lb_batch_two_step_tile(lb_batch* b, int32_t tile_y)
{
    int rc = check_batch(b);
    if (rc) return rc;
    if (!b->two_may) return fail(LB_ERR_STATE, "this batch does not run two steps per launch");
    if (tile_y != 0 && (tile_y < kBatchMinTile2 || tile_y > kBatchMaxTile2))
        return fail(LB_ERR_INVALID, "tile_y must be 0 or in [%d, %d] (got %d)", kBatchMinTile2,
                    kBatchMaxTile2, tile_y);
    const int count = (int)b->members.size();
    BatchLayout L;
    if ((rc = batch_layout(b->params.data(), count, &L))) return rc;
    const int ty = tile_y ? tile_y : L.tile_y2;  // 0: back to the tiles
    std::vector<lbk::BatchLattice> desc = b->host_desc;
    std::vector<int32_t> tl2;
    tl2.reserve(b->tiles2_cap);
    for (int i = 0; ty && i < count; ++i) {
        desc[i].geom2 = batch_geom2(b->params[i], ty);
        desc[i].tile_begin2 = (int32_t)tl2.size();
        tl2.insert(tl2.end(), desc[i].geom2.blocks, i);
    }
    if ((int)tl2.size() > b->tiles2_cap) return fail(LB_ERR_INVALID, "two-step tile table too small");
    DeviceGuard dg(b->device);
    if (dg.err) return hip_fail(dg.err, "select device");
    // Work already issued reads the tables: let it finish before rewriting them.
    hipError_t e = hipStreamSynchronize(b->stream);
    if (!e) e = hipMemcpyAsync(b->desc, desc.data(), sizeof(lbk::BatchLattice) * count,
                               hipMemcpyHostToDevice, b->stream);
    if (!e && !tl2.empty())
        e = hipMemcpyAsync(b->tile_lattice2, tl2.data(), sizeof(int32_t) * tl2.size(),
                           hipMemcpyHostToDevice, b->stream);
    if (!e) e = hipStreamSynchronize(b->stream);
    if (e) return hip_fail(e, "copy batch tables");
    for (auto& kv : b->graphs) (void)hipGraphExecDestroy(kv.second);
    b->graphs.clear();  // captured launches carry the old grid
    b->host_desc = desc;
    b->tile_y2 = ty;
    b->tiles2 = (int)tl2.size();
    b->two = ty > 0;
    b->tile_steps = ty ? 0 : L.tile.steps;
    return LB_OK;
}

int lb_batch_member(lb_batch* b, int32_t i, lb_ctx** member)
{
    int rc = check_batch(b);
    if (rc) return rc;
    if (!member) return fail(LB_ERR_INVALID, "member is NULL");
    if (i < 0 || i >= (int32_t)b->members.size())
        return fail(LB_ERR_INVALID, "lattice index %d out of range", i);
    *member = b->members[i];
    return LB_OK;
}

int lb_batch_destroy(lb_batch* b)
{
    {
        std::lock_guard<std::mutex> lk(g_mu);
        if (!b || !g_batches.count(b)) return fail(LB_ERR_STATE, "unknown or destroyed batch");
        g_batches.erase(b);
    }
    DeviceGuard dg(b->device);
    hipError_t e = hipStreamSynchronize(b->stream);
    for (auto& kv : b->graphs) (void)hipGraphExecDestroy(kv.second);
    for (lb_ctx* c : b->members) {
        std::lock_guard<std::mutex> lk(g_mu);
        g_live.erase(c);
        delete c;
    }
    delete b;
    if (e) return hip_fail(e, "synchronise");
    return LB_OK;
}


// ---------------------------------------------------------------------------
// Adjoint of a run: gradients of L = (E(T) - E*)^2 + beta A(T).
// ---------------------------------------------------------------------------
namespace {

// Tiles of the adjoint steps, and the most steps of a launch.
struct AdjPlan {
    lbk::AdjTile g;
    int steps;
};

// About one tile per CU, as for the plain steps (make_tile), then whole rounds
// of the workgroups resident at once.  A step's halo is two sites wider than a
// plain step's, so launches take three steps up to 16 x 16 tiles and two
// beyond.  Double precision keeps 512 threads, whose registers hold a site's
// adjoint without spilling.  Measured us/step, backward pass of a run in one
// segment: FP32 96x80 6x5 tiles 3 steps 4.8, 4 4.9; 256^2 16x16 3 5.9, 2 6.1;
// 512^2 32x32 2 8.2, 1 10.7, 24x24 3 12.1, 32x16 2 8.8; 1024^2 32x32 2 with
// 512 threads 28.6, with 1024 33.3; FP64 96x80 6x5 3 5.8, 2 6.0; 256^2 16x16 2
// 7.0, 3 7.4; 512^2 32x32 2 12.8.
AdjPlan adj_plan(int nx, int ny, bool f64)
{
    AdjPlan t{};
    const int64_t N = (int64_t)nx * ny, area = (N + 255) / 256;
    const bool round = area <= lbk::kAdjTileMax * lbk::kAdjTileMax;
    const int64_t slots = f64 || round ? 256 : 512;
    t.g.threads = f64 || !round ? 512 : 1024;
    for (int k = area <= (f64 ? 144 : 256) ? 3 : 2; k >= 1; --k) {
        const int top = k == 3 ? 24 : lbk::kAdjTileMax;  // the halo fits a second round of the threads
        const int w = std::min(top, nx - 3 * k), h = std::min(top, ny - 3 * k);
        if (w < 2 || h < 2) continue;
        const TileSplit s = split_tiles(nx, ny, w, h, 4, slots, 6 * k + 2);
        if (!s.tx) continue;
        t.steps = k;
        t.g.tx = s.tx;
        t.g.ty = s.ty;
        t.g.tiles_x = (nx + s.tx - 1) / s.tx;
        t.g.tiles = t.g.tiles_x * ((ny + s.ty - 1) / s.ty);
        return t;
    }
    return t;
}

int adj_waves(const AdjPlan& t) { return t.g.tiles * (t.g.threads / 64); }

// The tile geometry of a launch of `steps` <= t.steps adjoint steps.
lbk::AdjTile adj_launch(const AdjPlan& t, int steps)
{
    lbk::AdjTile g = t.g;
    auto magic = [](uint32_t d) { return (uint32_t)(((uint64_t(1) << 32) + d - 1) / d); };
    g.steps = steps;
    g.magic_tx = magic(g.tx);
    for (int j = 0; j < steps; ++j) {
        const int r = 3 * (steps - 1 - j) + 2;
        g.magic_w[j] = magic(g.tx + 2 * r);
        g.magic_2r[j] = magic(2 * r);
        g.magic_e[j] = magic(g.tx + 2 * r + 4);
    }
    return g;
}

}  // namespace

struct lb_adj {
    lb_ctx* fwd;          // the forward lattice (never handed out)
    lbk::AdjParams ap;
    int64_t T;
    int32_t every, nseg;
    size_t ckpt_bytes;    // one raw population buffer
    char* ckpt;           // nseg checkpoints, at t = 0, every, 2 every, ...
    char* tapes[2];       // two regions of `every` tape entries of 4 N values
    char* tapeT;          // tape entry of the state at T
    char* lam[2];         // 9 N values each
    char* dir;            // 2 N values
    double* part;         // adj_waves(tile) x 2: dL/dG from the steps
    double* partE;        // adj_blocks x 2: dE/dG at T
    double* partA;        // adj_blocks: interface measure
    double* host;         // pinned: kernels store the reduced values here
    double* red;          // its device address: a row of observables, A, dL/dG, dE/dG, a flag
    double* drho;         // N doubles
    int blocks;
    AdjPlan tile;         // the adjoint steps' tiles
    int32_t tape_of[2];   // segment whose tape each region holds, or -1
    bool have_forward;
    double E, A, E_target, beta, eps;
    // The backward pass re-steps segment s - 1 (taping it into region
    // (s - 1) & 1) on `side` while the adjoint steps of segment s run on
    // the context's stream; ev_r[b] marks region b taped, ev_a[b] region b
    // read.  Without a stream of its own (the null stream) both run in turn
    // on the context's stream.
    hipStream_t side;
    bool own_side;
    hipEvent_t ev_r[2], ev_a[2];
    // Full segments replay captured graphs: the taped re-step keyed by its
    // region, the adjoint steps by region and the parity of the adjoint
    // buffers at their start; valid for the couplings they were captured
    // with.
    std::map<int, hipGraphExec_t> tape_graphs, adj_graphs;
    double graph_G1, graph_G2;
    bool use_graphs;
};

namespace {

std::set<lb_adj*> g_adjs;

// n steps of the forward lattice on stream st, each also recording the tape
// entry of the state it leaves (entry j = state t + j) in `tape`.
hipError_t adj_tape_steps(lb_adj* a, int64_t n, char* tape, hipStream_t st)
{
    lb_ctx* c = a->fwd;
    const size_t entry = (size_t)4 * c->p.nx * c->p.ny * (a->ap.f64 ? 8 : 4);
    for (int64_t j = 0; j < n;) {
        c->coef.step = (uint32_t)c->t;
        const void* src = c->buf[c->cur];
        void* dst = c->buf[c->cur ^ 1];
        const int k = std::max(1, tile_steps(c->tile, n - j));
        hipError_t e;
        if (k > 1 || (c->tile.steps && c->tile.single))
            e = lbk::launch_tile(c->p.storage, src, dst, tile_launch(c->tile, k), c->coef, tape + j * entry, st);
        else
            e = lbk::launch_step(c->p.storage, lbk::MODE_STEP_TAPE, src, dst, c->g, c->coef,
                                 reinterpret_cast<double*>(tape + j * entry), st);
        if (e) return e;
        c->cur ^= 1;
        c->t += k;
        j += k;
    }
    return hipSuccess;
}

// Buffer flips of n taped forward steps (the launches of adj_tape_steps).
int adj_tape_flips(const lb_adj* a, int64_t n)
{
    int flips = 0;
    for (; n > 0; ++flips) n -= std::max(1, tile_steps(a->fwd->tile, n));
    return flips & 1;
}

// n adjoint steps on stream st, from tape entry n - 1 down to 0, starting
// from adjoint buffer `cur`.
hipError_t adj_back_steps(lb_adj* a, int64_t n, const char* tape, int cur, hipStream_t st)
{
    const size_t entry = (size_t)4 * a->ap.nx * a->ap.ny * (a->ap.f64 ? 8 : 4);
    while (n > 0) {
        const int k = even_steps(n, a->tile.steps);
        hipError_t e = lbk::adj_steps(a->ap, adj_launch(a->tile, k), a->lam[cur], tape + (n - 1) * entry,
                                      a->lam[cur ^ 1], a->part, st);
        if (e) return e;
        cur ^= 1;
        n -= k;
    }
    return hipSuccess;
}

// Adjoint buffer flips of n steps.
int adj_flips(const lb_adj* a, int64_t n) { return (int)((n + a->tile.steps - 1) / a->tile.steps & 1); }

void adj_drop_graphs(lb_adj* a)
{
    for (auto& kv : a->tape_graphs) (void)hipGraphExecDestroy(kv.second);
    for (auto& kv : a->adj_graphs) (void)hipGraphExecDestroy(kv.second);
    a->tape_graphs.clear();
    a->adj_graphs.clear();
}

// Launch `work` on st, as one replay of a graph captured under `key` in
// `graphs` when graphs are in use (captured on first use), else directly.
hipError_t adj_replay(lb_adj* a, std::map<int, hipGraphExec_t>& graphs, int key, hipStream_t st,
                      const std::function<hipError_t()>& work)
{
    if (!a->use_graphs) return work();
    auto it = graphs.find(key);
    if (it == graphs.end()) {
        hipGraph_t graph = nullptr;
        hipGraphExec_t exec = nullptr;
        hipError_t e = hipStreamBeginCapture(st, hipStreamCaptureModeThreadLocal);
        if (e == hipSuccess) {
            const hipError_t le = work();
            e = hipStreamEndCapture(st, &graph);
            if (e == hipSuccess && le != hipSuccess) e = le;
        }
        if (e == hipSuccess) e = hipGraphInstantiate(&exec, graph, nullptr, nullptr, 0);
        if (graph) (void)hipGraphDestroy(graph);
        if (e != hipSuccess) {
            // This stream cannot be captured: launch by launch from now on.
            (void)hipGetLastError();
            a->use_graphs = false;
            adj_drop_graphs(a);
            return work();
        }
        it = graphs.emplace(key, exec).first;
    }
    return hipGraphLaunch(it->second, st);
}

// Tape segment s into region s & 1 on the side stream (unless the region
// holds it already), once the adjoint steps that last read that region are
// done; marks the region taped.
hipError_t adj_restep(lb_adj* a, int32_t s)
{
    lb_ctx* c = a->fwd;
    const int b = s & 1;
    hipStream_t st = a->side;
    hipError_t e;
    if (a->tape_of[b] != s) {
        a->tape_of[b] = -1;
        const int64_t t0 = (int64_t)s * a->every;
        const int64_t n = a->T - t0 < a->every ? a->T - t0 : a->every;
        if ((e = hipStreamWaitEvent(st, a->ev_a[b], 0)) ||
            (e = hipMemcpyAsync(c->buf[0], a->ckpt + (size_t)s * align_up(a->ckpt_bytes), a->ckpt_bytes,
                                hipMemcpyDeviceToDevice, st)))
            return e;
        // From the checkpoint each time: adj_replay runs this again where a
        // capture of it came to nothing.
        auto work = [&] {
            c->cur = 0;
            c->t = t0;
            return adj_tape_steps(a, n, a->tapes[b], st);
        };
        if (n == a->every) {
            e = adj_replay(a, a->tape_graphs, b, st, work);
            c->cur = adj_tape_flips(a, n);
            c->t = t0 + n;
        } else {
            e = work();
        }
        if (e) return e;
        a->tape_of[b] = s;
    }
    return hipEventRecord(a->ev_r[b], st);
}

// The adjoint steps of segment s on the context's stream, once its tape is
// in place; marks its region read.
hipError_t adj_backseg(lb_adj* a, int32_t s, int cur)
{
    const int b = s & 1;
    hipStream_t st = a->fwd->stream;
    const int64_t t0 = (int64_t)s * a->every;
    const int64_t n = a->T - t0 < a->every ? a->T - t0 : a->every;
    hipError_t e;
    if ((e = hipStreamWaitEvent(st, a->ev_r[b], 0))) return e;
    auto work = [&] { return adj_back_steps(a, n, a->tapes[b], cur, st); };
    e = n == a->every ? adj_replay(a, a->adj_graphs, b * 2 + cur, st, work) : work();
    if (e) return e;
    return hipEventRecord(a->ev_a[b], st);
}

int check_adj(lb_adj* a)
{
    std::lock_guard<std::mutex> lk(g_mu);
    if (!a || !g_adjs.count(a)) return fail(LB_ERR_STATE, "unknown or destroyed adjoint context");
    return LB_OK;
}

struct AdjLayout {
    lb_params fp;         // forward parameters: no trace
    size_t fwd, fwd_bytes, ckpt, ckpt_bytes, tape[2], tapeT, lam[2], dir, part, partE, partA,
        drho, total;
    int32_t nseg;
    int blocks;
    AdjPlan tile;
};

int adj_layout(const lb_params* p, int64_t nsteps, int32_t every, AdjLayout* L)
{
    int rc = check_params(p);
    if (rc) return rc;
    if (p->storage != LB_F64 && p->storage != LB_F32)
        return fail(LB_ERR_INVALID, "the adjoint needs LB_F64 or LB_F32 storage");
    if (nsteps < 0) return fail(LB_ERR_INVALID, "nsteps must be >= 0");
    if (every < 1) return fail(LB_ERR_INVALID, "checkpoint_every must be >= 1");
    // The adjoint kernels address their dense per-site arrays with 32-bit
    // byte offsets from a per-array base (8-byte values).
    if ((int64_t)p->nx * p->ny > (int64_t(1) << 29))
        return fail(LB_ERR_INVALID, "the adjoint supports at most 2^29 sites (got %lld)",
                    (long long)p->nx * p->ny);
    L->fp = *p;
    L->fp.log_every = 0;
    L->fp.trace_cap = 0;
    const Geom g = make_geom(L->fp);
    const Layout F = make_layout(L->fp, g);
    const int64_t N = (int64_t)p->nx * p->ny;
    const size_t es = p->storage == LB_F64 ? 8 : 4;
    const int64_t nseg = (nsteps + every - 1) / every;
    if (nseg > INT32_MAX) return fail(LB_ERR_INVALID, "too many checkpoints");
    L->nseg = (int32_t)nseg;
    L->blocks = lbk::adj_blocks(N);
    const int64_t seg_len = nsteps < every ? nsteps : every;
    size_t off = 0;
    L->fwd = off; L->fwd_bytes = F.total; off += align_up(F.total);
    L->ckpt_bytes = (size_t)9 * g.plane * es;
    L->ckpt = off; off += (size_t)nseg * align_up(L->ckpt_bytes);
    // Segment s is taped into region s & 1; a run of one segment keeps its
    // whole tape from the forward pass and needs only region 0.
    L->tape[0] = off; off += align_up((size_t)seg_len * 4 * N * es);
    L->tape[1] = L->tape[0];
    if (nseg > 1) { L->tape[1] = off; off += align_up((size_t)seg_len * 4 * N * es); }
    L->tapeT = off; off += align_up((size_t)4 * N * es);
    for (int q = 0; q < 2; ++q) { L->lam[q] = off; off += align_up((size_t)9 * N * es); }
    L->dir = off; off += align_up((size_t)2 * N * es);
    L->tile = adj_plan(p->nx, p->ny, p->storage == LB_F64);
    L->part = off; off += align_up((size_t)adj_waves(L->tile) * 2 * sizeof(double));
    L->partE = off; off += align_up((size_t)L->blocks * 2 * sizeof(double));
    L->partA = off; off += align_up((size_t)L->blocks * sizeof(double));
    L->drho = off; off += align_up((size_t)N * sizeof(double));
    L->total = off;
    return LB_OK;
}

}  // namespace

size_t lb_adj_workspace_bytes(const lb_params* p, int64_t nsteps, int32_t checkpoint_every)
{
    AdjLayout L;
    return adj_layout(p, nsteps, checkpoint_every, &L) ? 0 : L.total;
}

int lb_adj_init(lb_adj** out, const lb_params* p, int64_t nsteps, int32_t checkpoint_every,
                void* workspace, size_t bytes, void* hip_stream)
{
    if (!out) return fail(LB_ERR_INVALID, "out is NULL");
    *out = nullptr;
    AdjLayout L;
    int rc = adj_layout(p, nsteps, checkpoint_every, &L);
    if (rc) return rc;
    if (!workspace) return fail(LB_ERR_INVALID, "workspace is NULL");
    if (reinterpret_cast<uintptr_t>(workspace) % kAlign)
        return fail(LB_ERR_INVALID, "workspace must be %zu-byte aligned", kAlign);
    if (bytes < L.total) return fail(LB_ERR_INVALID, "workspace too small: %zu < %zu bytes", bytes, L.total);
    char* ws = static_cast<char*>(workspace);
    const std::vector<double> ones((size_t)p->nx * p->ny, 1.0);
    lb_ctx* c = nullptr;
    if ((rc = lb_init(&c, &L.fp, ws + L.fwd, L.fwd_bytes, ones.data(), nullptr, nullptr, 0, hip_stream)))
        return rc;
    lb_adj* a = new lb_adj();
    a->fwd = c;
    a->ap.nx = p->nx;
    a->ap.ny = p->ny;
    a->ap.f64 = p->storage == LB_F64;
    a->ap.G1 = p->G1;
    a->ap.G2 = p->G2;
    a->ap.tau = p->tau;
    a->ap.sqrt_rho0 = std::sqrt(p->rho0);
    a->ap.inv_rho0 = 1.0 / p->rho0;
    a->T = nsteps;
    a->every = checkpoint_every;
    a->nseg = L.nseg;
    a->ckpt_bytes = L.ckpt_bytes;
    a->ckpt = ws + L.ckpt;
    for (int q = 0; q < 2; ++q) {
        a->tapes[q] = ws + L.tape[q];
        a->tape_of[q] = -1;
    }
    a->tapeT = ws + L.tapeT;
    for (int q = 0; q < 2; ++q) a->lam[q] = ws + L.lam[q];
    a->dir = ws + L.dir;
    a->part = reinterpret_cast<double*>(ws + L.part);
    a->partE = reinterpret_cast<double*>(ws + L.partE);
    a->partA = reinterpret_cast<double*>(ws + L.partA);
    a->drho = reinterpret_cast<double*>(ws + L.drho);
    a->blocks = L.blocks;
    a->tile = L.tile;
    a->have_forward = false;
    a->graph_G1 = a->ap.G1;
    a->graph_G2 = a->ap.G2;
    a->use_graphs = hip_stream != nullptr;
    // The re-steps get a stream of their own (default priority) when the
    // context has one; on the null stream everything runs in turn.
    a->side = c->stream;
    a->own_side = false;
    a->ev_r[0] = a->ev_r[1] = a->ev_a[0] = a->ev_a[1] = nullptr;
    {
        DeviceGuard dg(c->device);
        hipError_t e = dg.err;
        a->host = nullptr;
        if (!e) e = hipHostMalloc(reinterpret_cast<void**>(&a->host), 16 * sizeof(double), hipHostMallocMapped);
        if (!e) e = hipHostGetDevicePointer(reinterpret_cast<void**>(&a->red), a->host, 0);
        for (hipEvent_t* ev : {&a->ev_r[0], &a->ev_r[1], &a->ev_a[0], &a->ev_a[1]})
            if (!e) e = hipEventCreateWithFlags(ev, hipEventDisableTiming);
        if (!e && hip_stream) {
            e = hipStreamCreateWithFlags(&a->side, hipStreamNonBlocking);
            a->own_side = e == hipSuccess;
        }
        if (e) {
            for (hipEvent_t ev : {a->ev_r[0], a->ev_r[1], a->ev_a[0], a->ev_a[1]})
                if (ev) (void)hipEventDestroy(ev);
            if (a->host) (void)hipHostFree(a->host);
            delete a;
            lb_destroy(c);
            return hip_fail(e, "adjoint stream and events");
        }
    }
    {
        std::lock_guard<std::mutex> lk(g_mu);
        g_adjs.insert(a);
    }
    *out = a;
    return LB_OK;
}

int lb_adj_forward(lb_adj* a, const double* rho_init, int on_device, double G1, double G2,
                   const lb_adj_loss* loss, double out[4])
{
    int rc = check_adj(a);
    if (rc) return rc;
    if (!rho_init || !loss || !out) return fail(LB_ERR_INVALID, "NULL argument");
    if (!std::isfinite(G1) || !std::isfinite(G2)) return fail(LB_ERR_INVALID, "G1, G2 must be finite");
    if (!std::isfinite(loss->E_target) || !std::isfinite(loss->beta) || !std::isfinite(loss->eps) ||
        !(loss->eps > 0.0))
        return fail(LB_ERR_INVALID, "loss: E_target and beta must be finite, eps finite and > 0");
    lb_ctx* c = a->fwd;
    DeviceGuard dg(c->device);
    if (dg.err) return hip_fail(dg.err, "select device");
    const int64_t N = (int64_t)c->p.nx * c->p.ny;
    hipStream_t st = c->stream;
    hipError_t e;
    // The density is validated before anything of the last run is overwritten.
    const double* r = rho_init;
    if (on_device) {
        int* const bad = reinterpret_cast<int*>(a->host + 12);
        *bad = 0;
        if ((e = lbk::launch_check(rho_init, N, true, reinterpret_cast<int*>(a->red + 12), st)) ||
            (e = hipStreamSynchronize(st)))
            return hip_fail(e, "check rho_init");
        if (*bad && (rc = field_check_device(rho_init, N, true, "rho_init", st))) return rc;
    } else {
        if ((rc = field_check_host(rho_init, N, true, "rho_init"))) return rc;
        if ((e = hipMemcpyAsync(c->staging, rho_init, N * sizeof(double), hipMemcpyHostToDevice, st)))
            return hip_fail(e, "copy rho_init");
        r = c->staging;
    }
    a->have_forward = false;
    a->tape_of[0] = a->tape_of[1] = -1;
    // Work left on the side stream by an earlier backward pass reads the
    // lattice buffers this run overwrites.
    if (a->own_side && (e = hipStreamSynchronize(a->side))) return hip_fail(e, "synchronise");
    c->p.G1 = G1;
    c->p.G2 = G2;
    c->coef = make_coef(c->p);
    a->ap.G1 = G1;
    a->ap.G2 = G2;
    c->cur = 0;
    c->t = 0;
    if ((e = lbk::launch_init(c->p.storage, r, nullptr, nullptr, c->buf[0], c->g, c->coef, st)))
        return hip_fail(e, "init kernel");
    for (int32_t s = 0; s < a->nseg; ++s) {
        if ((e = hipMemcpyAsync(a->ckpt + (size_t)s * align_up(a->ckpt_bytes), c->buf[c->cur],
                                a->ckpt_bytes, hipMemcpyDeviceToDevice, st)))
            return hip_fail(e, "checkpoint copy");
        const int64_t t0 = (int64_t)s * a->every;
        const int64_t n = a->T - t0 < a->every ? a->T - t0 : a->every;
        // The last segment is taped on the way, so the backward pass
        // starts without recomputing it.
        if (s + 1 < a->nseg) {
            if ((rc = lb_step(c, n))) return rc;
        } else {
            if ((e = adj_tape_steps(a, n, a->tapes[s & 1], st))) return hip_fail(e, "step kernel launch");
            a->tape_of[s & 1] = s;
        }
    }
    if ((e = lbk::adj_tape(c->p.storage, c->buf[c->cur], c->g, a->ap, a->tapeT, st)) ||
        (e = lbk::adj_area(a->ap, a->tapeT, loss->eps, a->dir, a->partA, st)) ||
        (e = lbk::adj_reduce(a->partA, a->blocks, 1, a->red + 6, st)))
        return hip_fail(e, "interface measure");
    if ((rc = energy_row(c, lbk::MODE_ENERGY, c->buf[c->cur], c->buf[c->cur ^ 1], a->red))) return rc;
    if ((e = hipStreamSynchronize(st))) return hip_fail(e, "loss terms");
    const double* const row = a->host;
    const double A = a->host[6];
    a->E = row[2] + row[3];
    a->A = A;
    a->E_target = loss->E_target;
    a->beta = loss->beta;
    a->eps = loss->eps;
    const double d = a->E - a->E_target;
    out[0] = d * d + a->beta * A;
    out[1] = a->E;
    out[2] = A;
    out[3] = row[1];
    if (!std::isfinite(out[0]) || !std::isfinite(out[3]))
        return fail(LB_ERR_NONFINITE, "non-finite loss or mass at T = %lld", (long long)a->T);
    a->have_forward = true;
    return LB_OK;
}

int lb_adj_backward(lb_adj* a, double dG[2], double* drho, int on_device)
{
    int rc = check_adj(a);
    if (rc) return rc;
    if (!dG || !drho) return fail(LB_ERR_INVALID, "NULL argument");
    if (!a->have_forward) return fail(LB_ERR_STATE, "lb_adj_backward needs a successful lb_adj_forward");
    lb_ctx* c = a->fwd;
    DeviceGuard dg(c->device);
    if (dg.err) return hip_fail(dg.err, "select device");
    const int64_t N = (int64_t)c->p.nx * c->p.ny;
    hipStream_t st = c->stream;
    const double two_dE = 2.0 * (a->E - a->E_target);
    hipError_t e;
    // The interface's directions are those of the forward pass.
    if ((e = lbk::adj_seed(a->ap, a->tapeT, a->dir, two_dE, a->beta, a->lam[0], a->partE, st)) ||
        (e = lbk::adj_zero(a->part, (int64_t)adj_waves(a->tile) * 2, st)))
        return hip_fail(e, "adjoint seed");
    if (a->use_graphs && (a->graph_G1 != a->ap.G1 || a->graph_G2 != a->ap.G2)) {
        adj_drop_graphs(a);
        a->graph_G1 = a->ap.G1;
        a->graph_G2 = a->ap.G2;
    }
    // Segments from the last to the first: the adjoint steps of segment s
    // (context stream) overlap the taped re-step of segment s - 1 (side
    // stream).  Both regions start out free, and the side stream starts
    // after the seed.
    if ((e = hipEventRecord(a->ev_a[0], st)) || (e = hipEventRecord(a->ev_a[1], st)))
        return hip_fail(e, "adjoint events");
    if (a->nseg > 0 && (e = adj_restep(a, a->nseg - 1))) return hip_fail(e, "adjoint re-step");
    int cur = 0;
    for (int32_t s = a->nseg - 1; s >= 0; --s) {
        if (s > 0 && (e = adj_restep(a, s - 1))) return hip_fail(e, "adjoint re-step");
        if ((e = adj_backseg(a, s, cur))) return hip_fail(e, "adjoint steps");
        const int64_t t0 = (int64_t)s * a->every;
        const int64_t n = a->T - t0 < a->every ? a->T - t0 : a->every;
        cur ^= adj_flips(a, n);
    }
    double* dst = on_device ? drho : a->drho;
    if ((e = lbk::adj_rho_grad(a->ap, a->lam[cur], dst, st)) ||
        (e = lbk::adj_reduce(a->part, adj_waves(a->tile), 2, a->red + 8, st)) ||
        (e = lbk::adj_reduce(a->partE, a->blocks, 2, a->red + 10, st)))
        return hip_fail(e, "adjoint reductions");
    if (!on_device && (e = hipMemcpyAsync(drho, a->drho, N * sizeof(double), hipMemcpyDeviceToHost, st)))
        return hip_fail(e, "copy gradients");
    if ((e = hipStreamSynchronize(st))) return hip_fail(e, "synchronise");
    const double* const r = a->host + 8;
    dG[0] = r[0] + two_dE * r[2];
    dG[1] = r[1] + two_dE * r[3];
    if (!std::isfinite(dG[0]) || !std::isfinite(dG[1]))
        return fail(LB_ERR_NONFINITE, "non-finite coupling gradient");
    return LB_OK;
}

int lb_adj_destroy(lb_adj* a)
{
    {
        std::lock_guard<std::mutex> lk(g_mu);
        if (!a || !g_adjs.count(a)) return fail(LB_ERR_STATE, "unknown or destroyed adjoint context");
        g_adjs.erase(a);
    }
    if (a->own_side) (void)hipStreamSynchronize(a->side);
    const int rc = lb_destroy(a->fwd);  // synchronises the stream first
    adj_drop_graphs(a);
    if (a->own_side) (void)hipStreamDestroy(a->side);
    for (hipEvent_t ev : {a->ev_r[0], a->ev_r[1], a->ev_a[0], a->ev_a[1]}) (void)hipEventDestroy(ev);
    (void)hipHostFree(a->host);
    delete a;
    return rc;
}


// ---------------------------------------------------------------------------
// Structure factor of a density field.
// ---------------------------------------------------------------------------
struct lb_sk {
    lbk::SkPlan plan;
    std::vector<int64_t> counts;  // modes per shell
    double* rho;                  // device staging of host input, L*L doubles
    double* host_shell;           // pinned: the last pass writes the shells here
    int device;
    hipStream_t stream;
};

namespace {

std::set<lb_sk*> g_sks;

int check_sk(lb_sk* s)
{
    std::lock_guard<std::mutex> lk(g_mu);
    if (!s || !g_sks.count(s)) return fail(LB_ERR_STATE, "unknown or destroyed structure-factor context");
    return LB_OK;
}

// Shell of a mode with l^2 + m^2 = q: the n with (2n-1)^2 <= 4q < (2n+1)^2
// (n - 1/2 <= sqrt(q) < n + 1/2), in integer arithmetic.
int64_t shell_of(int64_t q)
{
    int64_t n = (int64_t)std::floor(std::sqrt((double)q) + 0.5);
    while ((2 * n + 1) * (2 * n + 1) <= 4 * q) ++n;
    while (n > 0 && (2 * n - 1) * (2 * n - 1) > 4 * q) --n;
    return n;
}

int sk_check_L(int32_t L)
{
    if (L < 5 || L > lbk::kSkMaxL)
        return fail(LB_ERR_INVALID, "L must be in [5, %d] (got %d)", lbk::kSkMaxL, L);
    return LB_OK;
}

struct SkLayout {
    lbk::SkFft fft;
    size_t tw, chirp, filter, z, mean, spec, part, count, rho, total;
    int32_t nshell, hc, hp;
};

SkLayout sk_layout(int32_t L)
{
    SkLayout S;
    const int64_t N = (int64_t)L * L;
    const int64_t h = L / 2;  // largest |l| of an L-point transform
    S.nshell = (int32_t)shell_of(2 * h * h) + 1;
    S.hc = (L + 1) / 2;
    S.hp = (int32_t)h + 1;
    S.fft = lbk::sk_fft(L);
    size_t off = 0;
    S.tw = off; off += align_up((size_t)S.fft.m * 2 * sizeof(double));
    S.chirp = off; off += align_up((size_t)L * 2 * sizeof(double));
    S.filter = off; off += align_up((size_t)S.fft.m * 2 * sizeof(double));
    S.z = off; off += align_up((size_t)L * S.hc * 2 * sizeof(double));
    S.mean = off; off += align_up((size_t)L * sizeof(double));
    S.spec = off; off += align_up((size_t)S.hp * L * sizeof(double));
    S.part = off; off += align_up((size_t)S.nshell * S.hp * sizeof(double));
    S.count = off; off += align_up((size_t)S.nshell * sizeof(double));
    S.rho = off; off += align_up((size_t)N * sizeof(double));
    // At least 52 bytes per mode, what a full complex transform took (a host test
    // holds the size above 40); the regions take 23.
    S.total = std::max(off, align_up((size_t)N * 52));
    return S;
}

// Modes of every shell, from the quadrant l, m = 0 .. L/2 (l and -l, m and
// -m alike; 0 and, for even L, L/2 are their own opposites).
void shell_counts(int32_t L, std::vector<int64_t>& counts)
{
    auto twins = [&](int64_t v) { return v == 0 || 2 * v == L ? 1 : 2; };
    for (int64_t l = 0; l <= L / 2; ++l) {
        int64_t n = l;
        for (int64_t m = 0; m <= L / 2; ++m) {
            while ((2 * n + 1) * (2 * n + 1) <= 4 * (l * l + m * m)) ++n;
            counts[n] += twins(l) * twins(m);
        }
    }
}

}  // namespace

int lb_sk_shells(int32_t L, int32_t* nshell)
{
    int rc = sk_check_L(L);
    if (rc) return rc;
    if (!nshell) return fail(LB_ERR_INVALID, "nshell is NULL");
    *nshell = sk_layout(L).nshell;
    return LB_OK;
}

size_t lb_sk_workspace_bytes(int32_t L)
{
    return sk_check_L(L) ? 0 : sk_layout(L).total;
}

int lb_sk_init(lb_sk** out, int32_t L, void* workspace, size_t bytes, void* hip_stream)
{
    if (!out) return fail(LB_ERR_INVALID, "out is NULL");
    *out = nullptr;
    int rc = sk_check_L(L);
    if (rc) return rc;
    const SkLayout S = sk_layout(L);
    if (!workspace) return fail(LB_ERR_INVALID, "workspace is NULL");
    if (reinterpret_cast<uintptr_t>(workspace) % kAlign)
        return fail(LB_ERR_INVALID, "workspace must be %zu-byte aligned", kAlign);
    if (bytes < S.total) return fail(LB_ERR_INVALID, "workspace too small: %zu < %zu bytes", bytes, S.total);
    int ndev = 0;
    hipError_t e = hipGetDeviceCount(&ndev);
    if (e != hipSuccess || ndev <= 0) return fail(LB_ERR_HIP, "no HIP device available");
    int dev = 0;
    if ((e = hipGetDevice(&dev))) return hip_fail(e, "hipGetDevice");

    char* ws = static_cast<char*>(workspace);
    hipStream_t st = static_cast<hipStream_t>(hip_stream);
    lb_sk* s = new lb_sk();
    lbk::SkPlan& p = s->plan;
    p.fft = S.fft;
    p.nshell = S.nshell;
    p.hc = S.hc;
    p.hp = S.hp;
    // Columns per workgroup: four (64-byte pieces of a row of z) when that
    // still gives a workgroup to every CU, else two or one; and no more than
    // fit the LDS.  The line is not sharp: with two columns from 120 groups
    // on, 1000^2 takes 52.3 us against 51.3 and 600^2 44.1 against 42.9.
    p.log_cols = 2;
    while (p.log_cols > 0 &&
           ((p.hc + (1 << p.log_cols) - 1) >> p.log_cols < 256 ||
            p.fft.m << p.log_cols > 8192 ||
            lbk::sk_lds(p.fft, 1 << p.log_cols) > (size_t)lbk::kSkColumnLds))
        --p.log_cols;
    double2* tw = reinterpret_cast<double2*>(ws + S.tw);
    double2* chirp = reinterpret_cast<double2*>(ws + S.chirp);
    double2* filter = reinterpret_cast<double2*>(ws + S.filter);
    p.t = lbk::SkTables{tw, chirp, filter};
    p.z = reinterpret_cast<double2*>(ws + S.z);
    p.mean = reinterpret_cast<double*>(ws + S.mean);
    p.spec = reinterpret_cast<double*>(ws + S.spec);
    p.part = reinterpret_cast<double*>(ws + S.part);
    p.count = reinterpret_cast<const double*>(ws + S.count);
    s->rho = reinterpret_cast<double*>(ws + S.rho);
    s->device = dev;
    s->stream = st;
    s->counts.assign(S.nshell, 0);
    shell_counts(L, s->counts);
    const std::vector<double> counts(s->counts.begin(), s->counts.end());
    // The shells leave the device by the last pass's own stores: a copy to
    // pageable memory costs a copy launch and a staging pass more.
    if ((e = hipHostMalloc(reinterpret_cast<void**>(&s->host_shell), S.nshell * sizeof(double),
                           hipHostMallocMapped))) {
        delete s;
        return hip_fail(e, "pinned shell buffer");
    }
    if ((e = hipHostGetDevicePointer(reinterpret_cast<void**>(&p.shell), s->host_shell, 0)) ||
        (e = hipMemcpyAsync(ws + S.count, counts.data(), counts.size() * sizeof(double),
                            hipMemcpyHostToDevice, st)) ||
        (e = lbk::sk_prepare(p, tw, chirp, filter, st)) || (e = hipStreamSynchronize(st))) {
        (void)hipHostFree(s->host_shell);
        delete s;
        return hip_fail(e, "structure-factor tables");
    }
    {
        std::lock_guard<std::mutex> lk(g_mu);
        g_sks.insert(s);
    }
    *out = s;
    return LB_OK;
}

int lb_sk_compute(lb_sk* s, const double* rho, int on_device, double* shell, int64_t* counts,
                  int32_t cap, double* kbar, double* spectrum)
{
    int rc = check_sk(s);
    if (rc) return rc;
    if (!rho) return fail(LB_ERR_INVALID, "rho is NULL");
    if (cap < 0 || (cap > 0 && !shell && !counts)) return fail(LB_ERR_INVALID, "bad shell outputs");
    const lbk::SkPlan& p = s->plan;
    const int64_t N = (int64_t)p.fft.n * p.fft.n;
    DeviceGuard dg(s->device);
    if (dg.err) return hip_fail(dg.err, "select device");
    hipError_t e;
    const double* r = rho;
    if (!on_device) {
        if ((rc = field_check_host(rho, N, false, "rho"))) return rc;
        if ((e = hipMemcpyAsync(s->rho, rho, N * sizeof(double), hipMemcpyHostToDevice, s->stream)))
            return hip_fail(e, "copy rho");
        r = s->rho;
    }
    if ((e = lbk::sk_compute(p, r, spectrum, s->stream))) return hip_fail(e, "structure-factor kernels");
    if ((e = hipStreamSynchronize(s->stream))) return hip_fail(e, "structure factor");
    const int32_t n = cap < p.nshell ? cap : p.nshell;
    const double* sh = s->host_shell;
    double num = 0.0, den = 0.0;
    bool finite = true;
    for (int32_t i = 0; i < p.nshell; ++i) {
        num += (double)i * sh[i];
        den += sh[i];
        finite = finite && std::isfinite(sh[i]);
    }
    for (int32_t i = 0; i < n; ++i) {
        if (shell) shell[i] = sh[i];
        if (counts) counts[i] = s->counts[i];
    }
    if (kbar) *kbar = num / den;
    if (!finite) return fail(LB_ERR_NONFINITE, "non-finite structure factor");
    if (kbar && !std::isfinite(num / den))
        return fail(LB_ERR_NONFINITE, "kbar is not finite (uniform field: every S_n is 0)");
    return LB_OK;
}

int lb_sk_destroy(lb_sk* s)
{
    {
        std::lock_guard<std::mutex> lk(g_mu);
        if (!s || !g_sks.count(s)) return fail(LB_ERR_STATE, "unknown or destroyed structure-factor context");
        g_sks.erase(s);
    }
    DeviceGuard dg(s->device);
    hipError_t e = hipStreamSynchronize(s->stream);
    (void)hipHostFree(s->host_shell);
    delete s;
    if (e) return hip_fail(e, "synchronise");
    return LB_OK;
}

}  // extern "C"
