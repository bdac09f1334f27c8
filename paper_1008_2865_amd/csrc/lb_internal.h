// Internal interface between the C ABI (lb_api.hip) and the HIP kernels
// (lb_kernels.hip).  Not installed; the public interface is include/lb.h.
#pragma once

#include <hip/hip_runtime.h>

#include <cstdint>

namespace lbk {

// Population storage codes (same values as enum lb_storage).
enum Storage { ST_F64 = 0, ST_F32 = 1, ST_F16DEV = 2 };

// Work done by one launch of the step kernel.
enum Mode {
    MODE_STEP = 0,         // stream + collide + store
    MODE_STEP_ENERGY = 1,  // the same, plus the energy/mass block partials
    MODE_ENERGY = 2,       // energy/mass block partials only, no store
    MODE_STEP_TAPE = 3     // stream + collide + store, plus (rho, jx, jy, psi)
                           // of every site's pre-collision state into a dense
                           // [4][ny][nx] array of the arithmetic type, passed
                           // in place of the partials (F64 and F32 only)
};

// Lattice geometry and launch shape.  Populations live in two buffers of
// 9 planes each; plane i holds population i as ny rows of `pitch` elements
// (x fastest, pitch a multiple of 64 elements), planes `plane` elements apart.
struct Geom {
    int32_t nx, ny;
    int32_t pitch;    // elements per row; ny * pitch < 2^31
    int64_t plane;    // elements per population plane
    int32_t tile_x;   // columns per workgroup (= threads per workgroup)
    int32_t tile_y;   // rows per workgroup
    int32_t tiles_x;  // column strips
    int32_t blocks;   // workgroups of the step kernel
    int32_t rows_per_iter;  // rows each workgroup updates per pipeline stage (1 or 2)
};

// Physical coefficients, in double; the launchers convert them to the
// arithmetic precision of the storage.
// Half storage: the populations are kept as deviations f_i - w_i rho' from
// offsets built on one single-precision value a = rho'/9 (the axis offset):
// a is rho_ref/9 rounded to 20 significant bits, so that the rest offset
// 4a, the diagonal offset a/4 and the sum of all nine offsets, 9a, are
// exact.  The encoder subtracts that sum from the density; were it rounded,
// every site would gain the same rounding error at every step, a drift of
// the total mass linear in time.
__host__ __device__ inline float dev_axis_offset(float rho_ref)
{
    float v = rho_ref * (1.0f / 9.0f);
    uint32_t u;
    __builtin_memcpy(&u, &v, sizeof u);
    u = (u + 8u) & ~15u;  // nearest value with the low 4 significand bits clear
    __builtin_memcpy(&v, &u, sizeof v);
    return v;
}

struct Coef {
    double K1, K2, K4, K5, K8;  // link coupling of each |c|^2 class (Table 1)
    double KE0;                 // rest coupling of E_s: G1 w_0 + G2 p_s0
    double tau, omega;          // BGK relaxation time and 1/tau
    double sqrt_rho0, inv_rho0; // psi = sqrt(rho0) (1 - exp(-rho/rho0))
    double rho_ref;             // deviation reference of ST_F16DEV
    uint32_t step;              // time step of the launch
};

// Several plain steps in one launch (lb_tile.hip): tiles of tx x ty sites,
// whose region of the first step, tx + 6 steps - 2 by ty + 6 steps - 2
// sites, fits kTilePitch x kTileRows and wraps around the lattice at most
// once.  A population plane spans less than 2^32 bytes.  With a tape (F64 and
// F32 only), step j also writes the tape entry of the state it leaves to
// tape + 4 j nx ny.
constexpr int kTilePitch = 44, kTileRows = 46, kTileMaxSteps = 5;
struct TileGeom {
    int32_t nx, ny, pitch;
    int64_t plane;
    int32_t tx, ty, tiles_x, tiles, threads;
    int32_t steps;                  // of this launch
    uint32_t magic[kTileMaxSteps];  // division by the region's width, by steps left after it
};
// One lattice of a batch, as the batched kernels read it (device memory).
struct BatchLattice {
    Geom geom;
    Geom geom2;          // two-step geometry (used when the batch runs two steps per launch)
    Coef coef;
    void* buf[2];        // population buffers; the step reads buf[parity]
    double* trace;       // this lattice's trace rows
    double half_A1;      // (G1 + G2) / 2
    int32_t tile_begin;  // first logical tile of this lattice in the batch
    int32_t tile_begin2; // first logical tile of this lattice in the two-step tile list
    int32_t tile_begin3; // first tile of this lattice in the list of lb_tile.hip's tiles
    float coef_f[13];    // coef converted to single precision (coef_to_f32), so the
                         // single-precision kernels read it without converting
    TileGeom tile;       // tiles of several steps per launch (when the batch runs them)
};

// coef in single precision, exactly as the single-lattice launchers pass it:
// K1, K2, K4, K5, K8, KE0, tau, omega, sqrt_rho0, inv_rho0, rho_ref, 2 K4, 2 K8.
void coef_to_f32(const Coef& c, float out[13]);

// Bytes of one stored population value.
inline int storage_bytes(int storage)
{
    return storage == ST_F64 ? 8 : storage == ST_F32 ? 4 : 2;
}

hipError_t launch_step(int storage, int mode, const void* src, void* dst,
                       const Geom& g, const Coef& c, double* partials,
                       hipStream_t s);
// Two plain steps in one launch (ST_F32 and ST_F16DEV storage).  g is the two-step
// geometry: tile_x lanes produce tile_x - 6 output columns, tiles_x =
// ceil(nx / (tile_x - 6)), blocks = tiles_x * ceil(ny / tile_y).
hipError_t launch_step2(int storage, const void* src, void* dst, const Geom& g, const Coef& c,
                        hipStream_t s);
// Two plain steps of every lattice of a batch in one launch (tau1: tau is 1 in
// every lattice): tiles logical tiles of kBatchLanes2 lanes (the lattices of a
// batch are narrow), tile_lattice maps each to its lattice, whose geom2 gives the
// tile's place; the launch reads buf[parity] and writes buf[parity ^ 1] of every
// lattice.
constexpr int kBatchLanes2 = 128;
hipError_t launch_step2_batch(int storage, bool tau1, const BatchLattice* desc, const int32_t* tile_lattice, int tiles,
                              int parity, uint32_t step, hipStream_t s);
// Workgroups of tile_x lanes of the two-step kernel (ST_F32 or ST_F16DEV)
// resident on the current device at once: the runtime's occupancy for the
// kernel's registers and LDS, per compute unit, times the compute units.
// -1 when no device can be asked.
int step2_resident(int storage, int tile_x);
hipError_t launch_tile(int storage, const void* src, void* dst, const TileGeom& g, const Coef& c, void* tape,
                       hipStream_t s);
// The same for every lattice of a batch, whose tiles have at most tx x ty sites.
struct TileBatch {
    const BatchLattice* desc;
    const int32_t* tile_lattice;  // lattice of each tile
    int tiles, tx, ty, threads;
    int parity, steps;            // reads buf[parity], writes buf[parity ^ 1]
    uint32_t step;                // time level of the first step
    bool tau1;                    // tau is 1 in every lattice
};
hipError_t launch_tile_batch(int storage, const TileBatch& b, hipStream_t s);
hipError_t launch_final(const double* partials, int blocks, double t,
                        double half_A1, double* out_row, hipStream_t s);
hipError_t launch_step_batch(int storage, int mode, int tile_x, int rows_per_iter, int min_tile_y,
                             const BatchLattice* desc, const int32_t* tile_lattice, int tiles,
                             int parity, uint32_t step, double* partials, hipStream_t s);
hipError_t launch_final_batch(const BatchLattice* desc, int count, const double* partials,
                              double t, int64_t row, hipStream_t s);
// Sets *flag (device memory or mapped host memory) to 1 if a value of v is not
// finite or, with positive, not > 0; the flag is otherwise left alone.
hipError_t launch_check(const double* v, int64_t n, bool positive, int* flag, hipStream_t s);
hipError_t launch_clear(int* flag, hipStream_t s);
hipError_t launch_moments(int storage, const void* src, const Geom& g,
                          const Coef& c, double* rho, double* ux, double* uy,
                          hipStream_t s);
hipError_t launch_init(int storage, const double* rho, const double* ux,
                       const double* uy, void* dst, const Geom& g,
                       const Coef& c, hipStream_t s);
hipError_t launch_get_state(int storage, const void* src, void* dense,
                            const Geom& g, hipStream_t s);
hipError_t launch_set_state(int storage, const void* dense, void* dst,
                            const Geom& g, hipStream_t s);

// Section V observables {t, M, E_s, E_m, sum psi^2, E_bulk} of a dense
// [9][ny][nx] pre-collision population array of the given storage (device
// memory) into out (host, 6 doubles), with every intermediate in the
// library's static device scratch (lb_noalloc.hip): no allocation, and the
// stream is synchronised before returning.
hipError_t noalloc_energy(int storage, const void* state, int nx, int ny, const Coef& c, double t,
                          double half_A1, double* out, hipStream_t s);

// Adjoint kernels (lb_adjoint.hip).  Arithmetic is double when f64 != 0,
// float otherwise; arrays are dense [component][ny][nx] of that type.
struct AdjParams {
    int32_t nx, ny;
    int32_t f64;
    double G1, G2, tau, sqrt_rho0, inv_rho0;
};

// Workgroups of every per-site adjoint kernel (one thread per site).
int adj_blocks(int64_t sites);
// tape[4][ny][nx] = (rho, jx, jy, psi) of the state held in a pitched
// population buffer of the given storage (ST_F64 or ST_F32).
hipError_t adj_tape(int storage, const void* buf, const Geom& g, const AdjParams& p, void* tape,
                    hipStream_t s);
// Adjoint steps in one launch: tiles of tx x ty sites, at most kAdjTileMax
// squared, whose halo of 3 steps - 1 sites holds at most as many again.  The
// tile with 3 steps + 1 sites more on each side wraps around the lattice at
// most once.
constexpr int kAdjTileMax = 32, kAdjMaxSteps = 3;
struct AdjTile {
    int32_t tx, ty, tiles_x, tiles, threads;
    int32_t steps;  // of this launch
    uint32_t magic_tx;                                         // division by tx, and by step:
    uint32_t magic_w[kAdjMaxSteps], magic_2r[kAdjMaxSteps];    // by the halo region's width, twice the halo
    uint32_t magic_e[kAdjMaxSteps];                            // by that width + 4
};
// `steps` adjoint steps: lam_in[9][ny][nx] at t -> lam_out at t - steps, from
// the tape entry of t - 1 at `tape` and the earlier ones before it;
// part[tiles * threads / 64][2] accumulates dL/dG1, dL/dG2, the same bits for
// any split of a run into launches.
hipError_t adj_steps(const AdjParams& p, const AdjTile& g, const void* lam_in, const void* tape, void* lam_out,
                     double* part, hipStream_t s);
// Interface measure of a tape entry: dir[2][ny][nx], part[adj_blocks] sums.
hipError_t adj_area(const AdjParams& p, const void* tape, double eps, void* dir, double* part,
                    hipStream_t s);
// Adjoint at T of L = (E - E*)^2 + beta A; part[adj_blocks][2] receives the
// workgroup sums of dE/dG1, dE/dG2.
hipError_t adj_seed(const AdjParams& p, const void* tape, const void* dir, double two_dE, double beta,
                    void* lam, double* part, hipStream_t s);
// out[ny][nx] (double) = sum_i w_i lam_i.
hipError_t adj_rho_grad(const AdjParams& p, const void* lam, double* out, hipStream_t s);
// out[v] = sum_b part[b * nv + v] for v < nv, fixed order.
hipError_t adj_reduce(const double* part, int blocks, int nv, double* out, hipStream_t s);
hipError_t adj_zero(double* p, int64_t n, hipStream_t s);

// Structure factor (lb_structure.hip) of an L x L density field, L <= kSkMaxL.
constexpr int kSkMaxL = 2048;
// LDS a workgroup of the column pass may use (160 KB less its static part; the
// runtime launches that much without a function's limit being raised).
constexpr int kSkColumnLds = 159 * 1024;
// The transform of n points: its passes over m points, m = n or, where n has a
// prime factor above 7, a smooth m >= 2 n - 1 (by convolution: two transforms
// of m points); radix[p] after sub-transforms of length s (the product of the
// radices before it), with the multipliers that divide by s and by
// m / radix[p].  The line lies at 7: as radices, 11 and 13 took 98 us for
// 1001^2, the convolution 67 for 1003^2.
struct SkFft {
    int32_t n, m, passes;
    int32_t chirp;  // by convolution
    int32_t radix[12];
    uint32_t magic_s[12], magic_m[12];
};
struct SkTables {
    const double2* tw;      // m twiddles exp(-2 pi i k / m)
    const double2* chirp;   // n (with SkFft::chirp)
    const double2* filter;  // m
};
struct SkPlan {
    SkFft fft;
    int32_t nshell;      // shells 0 .. nshell-1
    int32_t hc;          // columns of the row spectra: L/2, (L+1)/2 for odd L
    int32_t log_cols;    // columns per workgroup of the column pass, log2
    int32_t hp;          // L/2 + 1, columns of the half spectrum
    SkTables t;
    double2* z;          // L*hc: row spectra, [y][l]
    double* mean;        // L: the numbers subtracted from the rows
    double* spec;        // hp*L: S at (l, m), l <= L/2, stored [l][m]
    double* part;        // nshell*hp: run sums, [n][l]
    const double* count; // nshell: modes per shell
    double* shell;       // nshell shell averages (pinned host memory)
};
SkFft sk_fft(int L);
// LDS of a workgroup with `cols` lines.
size_t sk_lds(const SkFft& f, int cols);
// Runs every pass on rho (device, L*L doubles); spectrum (device, [m][l])
// may be NULL.
hipError_t sk_compute(const SkPlan& p, const double* rho, double* spectrum, hipStream_t s);
// Fills the tables of p.t (once per plan).
hipError_t sk_prepare(const SkPlan& p, double2* tw, double2* chirp, double2* filter, hipStream_t s);

}  // namespace lbk
