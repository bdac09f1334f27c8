// Adjoint (reverse-mode) kernels of the two-belt Shan-Chen step, for the
// gradients of a functional of the state at time T with respect to G1, G2
// and the initial density.
//
// Forward step at a site x (section II moments, eq. (FORCE), velocity-shift
// BGK collision, streaming of eq. (1)):
//   rho = sum f, j = sum c f, psi = sqrt(rho0) (1 - exp(-rho/rho0)),
//   F = -psi(x) S(x), S(x) = sum_k K_k psi(x + c_k) c_k, u = (j + tau F)/rho,
//   f*_l = f_l + w (feq_l(rho, u) - f_l), f_l(x + c_l, t+1) = f*_l(x),
//   feq_l = w_l rho phi_l(u), phi_l = 1 + 3 c_l.u + 4.5 (c_l.u)^2 - 1.5 u^2.
// Write lambda_i(x, t) = dL/df_i(x, t) (pre-collision populations).  The
// transpose of the pull streaming hands each site the adjoint of its
// post-collision populations, mu_l(x) = lambda_l(x + c_l, t+1), taken here as
// a gather so that no two threads write one value.  With
//   M0 = sum_l mu_l w_l phi_l,  V = sum_l mu_l w_l grad_u phi_l,
//   grad_u phi_l = 3 c_l + 9 (c_l.u) c_l - 3 u,
// one adjoint step is
//   lambda_i(x, t) = (1 - w) mu_i + w (M0 - V.u) + w V.c_i + g_rho(x),
//   g_F(x) = w tau V                                (dL/dF(x)),
//   g_rho(y) = psi'(rho(y)) * (-sum_k K_k psi(y + c_k) (g_F(y) - g_F(y + c_k)).c_k),
//   dL/dG1 += sum_x g_F(x).(-psi(x) sum_{first belt} w_k psi(x + c_k) c_k),
//   dL/dG2 += sum_x g_F(x).(-psi(x) sum_k p_k psi(x + c_k) c_k),
// where the g_rho sum is the force's dependence on psi, transposed from the
// 24-link gather into a 24-link gather of g_F (K_{-k} = K_k).
//
// Storage: lambda as nine dense planes, the site term g_rho included.  Tape
// entries are (rho, jx, jy, psi) of the pre-collision state.  All arrays are
// dense [component][ny][nx].  Sums are FP64 partials combined in a fixed
// order (no atomics), so gradients are bit-reproducible.
#include "lb_site.h"

#include <type_traits>

namespace lbk {
namespace {

// The 24 links (first belt in D2Q9 order, then |c|^2 = 4, 5, 8), the D2Q9
// weight of the first-belt links (0 on the second belt) and the Table 1
// weight p(|c|^2) of every link: K_k = G1 w_k + G2 p_k.
constexpr int kLx[24] = {1, 0, -1, 0, 1, -1, -1, 1, 2, 0, -2, 0,
                         2, 1, -1, -2, -2, -1, 1, 2, 2, -2, -2, 2};
constexpr int kLy[24] = {0, 1, 0, -1, 1, 1, -1, -1, 0, 2, 0, -2,
                         1, 2, 2, 1, -1, -2, -2, -1, 2, 2, -2, -2};
constexpr double kLw[24] = {1.0 / 9, 1.0 / 9, 1.0 / 9, 1.0 / 9, 1.0 / 36, 1.0 / 36, 1.0 / 36, 1.0 / 36,
                            0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0};
constexpr double kLp[24] = {4.0 / 63, 4.0 / 63, 4.0 / 63, 4.0 / 63,
                            4.0 / 135, 4.0 / 135, 4.0 / 135, 4.0 / 135,
                            1.0 / 180, 1.0 / 180, 1.0 / 180, 1.0 / 180,
                            2.0 / 945, 2.0 / 945, 2.0 / 945, 2.0 / 945,
                            2.0 / 945, 2.0 / 945, 2.0 / 945, 2.0 / 945,
                            1.0 / 15120, 1.0 / 15120, 1.0 / 15120, 1.0 / 15120};
// The same by |c|^2, the D2Q9 weights by population, and the rest weight p_s0
// of E_s.
constexpr double kP1 = 4.0 / 63, kP2 = 4.0 / 135, kP4 = 1.0 / 180, kP5 = 2.0 / 945, kP8 = 1.0 / 15120;
constexpr double kW0 = 4.0 / 9, kW1 = 1.0 / 9, kW2 = 1.0 / 36, kPS0 = 247.0 / 420.0;
constexpr double kQw[9] = {kW0, kW1, kW1, kW1, kW1, kW2, kW2, kW2, kW2};

constexpr int kThreads = 256;

__device__ __forceinline__ int wrapn(int v, int n)
{
    v = v < 0 ? v + n : v;
    return v >= n ? v - n : v;
}

// base[e] with the byte offset formed in 32 bits (a uniform base plus a
// per-lane 32-bit offset, which needs no 64-bit address arithmetic).
template <typename T>
__device__ __forceinline__ T ld32(const T* base, int e)
{
    const uint32_t b = (uint32_t)e * (uint32_t)sizeof(T);
    return *reinterpret_cast<const T*>(reinterpret_cast<const char*>(base) + b);
}

__device__ __forceinline__ double ex(double v) { return exp(v); }
__device__ __forceinline__ float ex(float v) { return expf(v); }
__device__ __forceinline__ double sq(double v) { return sqrt(v); }
__device__ __forceinline__ float sq(float v) { return sqrtf(v); }

template <typename C>
struct AdjArgs {
    int nx, ny;
    int64_t N;
    C G1, G2, tau, omega, sqrt_rho0, inv_rho0;
    C K1, K2, K4x2, K5, K8x2;  // link couplings by |c|^2, twice those of |c_x| = 2 pairs
};

// Workgroup sums of NV values, written to part[block * NV + v].
template <int NV>
__device__ __forceinline__ void block_sum(double (&v)[NV], double* __restrict__ part)
{
    __shared__ double red[NV][kThreads / 64];
    const int lane = threadIdx.x & 63, wid = threadIdx.x >> 6;
#pragma unroll
    for (int q = 0; q < NV; ++q) {
        double s = v[q];
#pragma unroll
        for (int m = 32; m >= 1; m >>= 1) s += __shfl_xor(s, m, 64);
        if (lane == 0) red[q][wid] = s;
    }
    __syncthreads();
    if (threadIdx.x < NV) {
        const int q = threadIdx.x;
        part[(int64_t)blockIdx.x * NV + q] = (red[q][0] + red[q][1]) + (red[q][2] + red[q][3]);
    }
}

// Tape entry of the pre-collision state held (as post-collision values of
// the previous step) in a pitched population buffer: rho, jx, jy, psi.
template <typename S, typename C>
__global__ void __launch_bounds__(kThreads)
k_adj_tape(const S* __restrict__ st, Geom g, AdjArgs<C> a, C* __restrict__ tape)
{
    const int64_t s = (int64_t)blockIdx.x * kThreads + threadIdx.x;
    if (s >= a.N) return;
    const int x = (int)(s % a.nx), y = (int)(s / a.nx);
    C r = 0, jx = 0, jy = 0;
#pragma unroll
    for (int i = 0; i < 9; ++i) {
        const int xs = wrapn(x - kQCx[i], a.nx), ys = wrapn(y - kQCy[i], a.ny);
        const C f = (C)st[(int64_t)i * g.plane + (int64_t)ys * g.pitch + xs];
        r += f;
        if (kQCx[i]) jx += kQCx[i] > 0 ? f : -f;
        if (kQCy[i]) jy += kQCy[i] > 0 ? f : -f;
    }
    tape[s] = r;
    tape[a.N + s] = jx;
    tape[2 * a.N + s] = jy;
    tape[3 * a.N + s] = a.sqrt_rho0 * ((C)1 - ex(-r * a.inv_rho0));
}

// ---------------------------------------------------------------------------
// Adjoint steps on tiles.  A workgroup owns tx x ty sites and takes them
// `steps` levels back in time on chip.  One step, for the tile and a halo:
//   the psi of the level (tape) into LDS, mu gathered from memory (the
//   launch's first step) or from the lambda planes in LDS | barrier |
//   the force sums, the collision's adjoint lambda (registers) and
//   psi g_F into LDS | barrier |
//   g_rho from the 24-link sums of psi g_F, lambda + g_rho into LDS (the
//   last step: to memory) | barrier.
// g_rho of a site needs g_F two sites out and mu needs lambda one site out,
// so a step consumes three sites of halo, as a forward step does.  The
// force's transpose sum_k K_k psi_k (g_F - g_F,k).c_k is g_F.S less the link
// sums of psi g_F, with S the force's own link sums, and those sums pair
// opposite links, so that a site costs about 200 vector instructions where a
// link-by-link gather of three arrays in two kernels cost 650.
//
// A tile's own sites keep their thread whatever the halo (the halo's sites
// follow in a second round), so the dL/dG partials are the same bits for any
// number of steps per launch.  The next step's psi is loaded a step ahead
// (its rho and j too: 2% faster on one tile per CU, but the registers cost two
// workgroups of 512 threads per CU, 26% at 1024^2).
//
// What bounds it: at 512^2 FP32 one tile per CU, whose loads (104 bytes a
// site for two steps, the tape's from HBM) and arithmetic (7 us for two steps)
// overlap little: 16.4 us per two steps, against 28.6 for the two kernels a
// step that gathered from memory.  FP64 96x80: 4.7 us a step against 9.6.
// ---------------------------------------------------------------------------
constexpr int kEPitch = kAdjTileMax + 14, kARegion = kAdjTileMax + 10, kBRegion = kAdjTileMax + 6;

__device__ __forceinline__ int div32(int v, uint32_t magic) { return (int)__umulhi((uint32_t)v, magic); }

// Site q of the ring of width r around a w x h rectangle at (0, 0): the rows
// above and below, w + 2 r wide, then the sides.
__device__ __forceinline__ void ring_site(int q, int w, int h, int r, uint32_t magic_w, uint32_t magic_2r,
                                          int& x, int& y)
{
    const int W = w + 2 * r, top = 2 * r * W;
    if (q < top) {
        const int row = div32(q, magic_w);
        x = q - row * W - r;
        y = row < r ? row - r : row - r + h;
    } else {
        const int p = q - top, row = div32(p, magic_2r), c = p - row * 2 * r;
        y = row;
        x = c < r ? c - r : c - r + w;
    }
}

// The collision adjoint of one site: st the psi stencil, rho, jx, jy its tape
// values, M its mu, which become lambda without the site term.  Multiply-adds
// are written out and nothing else is contracted in the adjoint step, so
// that a site of the tile and the same site in a neighbour's halo get the
// same bits.
template <typename C>
struct SiteAdjoint {
    C hx, hy;                  // psi g_F
    C q, dpsi;                 // g_F.S, psi'
    C gx, gy, s1x, s1y, s2x, s2y;  // g_F and the two belts' sums
};

template <typename C>
__device__ __forceinline__ SiteAdjoint<C>
adjoint_collide(const Stencil<C>& st, C rho, C jx, C jy, const AdjArgs<C>& a, C (&M)[9])
{
#pragma clang fp contract(off)
    SiteAdjoint<C> r;
    const C p = st.p;
    const C d1x = st.e1 - st.w1, d1y = st.n1 - st.s1v;
    const C d2a = st.ne - st.sw, d2b = st.se - st.nw;
    const C d8a = st.ne2 - st.sw2, d8b = st.se2 - st.nw2;
    const C d5a = st.e2n - st.w2s, d5b = st.e2s - st.w2n;
    const C d5c = st.n2e - st.s2w, d5d = st.n2w - st.s2e;
    r.s1x = fma_c((C)kW1, d1x, (C)kW2 * (d2a + d2b));
    r.s1y = fma_c((C)kW1, d1y, (C)kW2 * (d2a - d2b));
    r.s2x = fma_c((C)kP1, d1x,
                  fma_c((C)kP2, d2a + d2b,
                        fma_c((C)(2 * kP4), st.e2 - st.w2,
                              fma_c((C)kP5, fma_c((C)2, d5a + d5b, d5c - d5d), (C)(2 * kP8) * (d8a + d8b)))));
    r.s2y = fma_c((C)kP1, d1y,
                  fma_c((C)kP2, d2a - d2b,
                        fma_c((C)(2 * kP4), st.n2 - st.s2v,
                              fma_c((C)kP5, fma_c((C)2, d5c + d5d, d5a - d5b), (C)(2 * kP8) * (d8a - d8b)))));
    // F = -psi S, S = G1 s1 + G2 s2: the two belts' sums, weighted.
    const C Sx = fma_c(a.G1, r.s1x, a.G2 * r.s2x), Sy = fma_c(a.G1, r.s1y, a.G2 * r.s2y);
    const C inv = (C)1 / rho, tp = a.tau * p;
    const C ux = fma_c(-tp, Sx, jx) * inv, uy = fma_c(-tp, Sy, jy) * inv;
    // Moments of w_l mu_l up to second order.
    const C ay = M[2] + M[4], da = M[5] + M[7], db = M[6] + M[8];
    const C ea = M[5] - M[7], eb = M[8] - M[6];
    const C dd = (C)kW2 * (da + db);
    const C mxx = fma_c((C)kW1, M[1] + M[3], dd), myy = fma_c((C)kW1, ay, dd), mxy = (C)kW2 * (da - db);
    const C m0 = fma_c((C)kW0, M[0], fma_c((C)kW1, ay, mxx));
    const C mx = fma_c((C)kW1, M[1] - M[3], (C)kW2 * (ea + eb));
    const C my = fma_c((C)kW1, M[2] - M[4], (C)kW2 * (ea - eb));
    const C uxx = fma_c(ux, mxx, uy * mxy), uyy = fma_c(ux, mxy, uy * myy);
    const C Vx = (C)3 * fma_c(-ux, m0, fma_c((C)3, uxx, mx)), Vy = (C)3 * fma_c(-uy, m0, fma_c((C)3, uyy, my));
    const C M0 = fma_c(m0, fma_c((C)-1.5, fma_c(ux, ux, uy * uy), (C)1),
                       fma_c((C)3, fma_c(ux, mx, uy * my), (C)4.5 * fma_c(ux, uxx, uy * uyy)));
    const C om = a.omega, keep = (C)1 - om;
    const C base = om * (M0 - fma_c(Vx, ux, Vy * uy)), ox = om * Vx, oy = om * Vy;
    const C add[9] = {base,             base + ox,        base + oy,        base - ox,       base - oy,
                      base + (ox + oy), base + (oy - ox), base - (ox + oy), base + (ox - oy)};
#pragma unroll
    for (int i = 0; i < 9; ++i) M[i] = fma_c(keep, M[i], add[i]);
    r.gx = a.tau * ox;
    r.gy = a.tau * oy;
    r.hx = p * r.gx;
    r.hy = p * r.gy;
    r.q = fma_c(r.gx, Sx, r.gy * Sy);
    // psi' = exp(-rho/rho0) sqrt(rho0)/rho0 = (sqrt(rho0) - psi)/rho0.
    r.dpsi = (a.sqrt_rho0 - p) * a.inv_rho0;
    return r;
}

// sum_k K_k (h_k . c_k) around a site whose psi g_F sit at X and Y.
template <typename C, int kPitch>
__device__ __forceinline__ C link_sums(const C* X, const C* Y, const AdjArgs<C>& a)
{
#pragma clang fp contract(off)
    // Opposite links, (dx, dy) less (-dx, -dy).
    auto dX = [&](int dx, int dy) { return X[dy * kPitch + dx] - X[-dy * kPitch - dx]; };
    auto dY = [&](int dx, int dy) { return Y[dy * kPitch + dx] - Y[-dy * kPitch - dx]; };
    const C sx = fma_c(a.K1, dX(1, 0),
                       fma_c(a.K2, dX(1, 1) + dX(1, -1),
                             fma_c(a.K4x2, dX(2, 0),
                                   fma_c(a.K5, fma_c((C)2, dX(2, 1) + dX(2, -1), dX(1, 2) + dX(1, -2)),
                                         a.K8x2 * (dX(2, 2) + dX(2, -2))))));
    const C sy = fma_c(a.K1, dY(0, 1),
                       fma_c(a.K2, dY(1, 1) + dY(-1, 1),
                             fma_c(a.K4x2, dY(0, 2),
                                   fma_c(a.K5, fma_c((C)2, dY(1, 2) + dY(-1, 2), dY(2, 1) + dY(-2, 1)),
                                         a.K8x2 * (dY(2, 2) + dY(-2, 2))))));
    return sx + sy;
}

// The sums of a and b over a wave's 64 lanes: a's in lanes 0 .. 31, b's in
// lanes 32 .. 63.  Lane swaps and row permutations of the vector unit, no LDS.
__device__ __forceinline__ double wave_sums(double a, double b)
{
    auto bits = [](double v) { return __builtin_bit_cast(uint2, v); };
    auto from = [](uint32_t lo, uint32_t hi) { return __builtin_bit_cast(double, make_uint2(lo, hi)); };
    const uint2 ua = bits(a), ub = bits(b);
    // The upper half of a against the lower half of b.
    const auto l = __builtin_amdgcn_permlane32_swap(ua.x, ub.x, false, false);
    const auto h = __builtin_amdgcn_permlane32_swap(ua.y, ub.y, false, false);
    double v = from(l[0], h[0]) + from(l[1], h[1]);
    // Odd rows of 16 lanes against even ones.
    const uint2 uv = bits(v);
    const auto rl = __builtin_amdgcn_permlane16_swap(uv.x, uv.x, false, false);
    const auto rh = __builtin_amdgcn_permlane16_swap(uv.y, uv.y, false, false);
    v = from(rl[0], rh[0]) + from(rl[1], rh[1]);
    // Within a row: mirrored, mirrored by halves, and two exchanges in fours.
    auto moved = [&](auto ctrl) {
        const uint2 u = bits(v);
        return from(__builtin_amdgcn_update_dpp(0, (int)u.x, decltype(ctrl)::value, 0xf, 0xf, false),
                    __builtin_amdgcn_update_dpp(0, (int)u.y, decltype(ctrl)::value, 0xf, 0xf, false));
    };
    v += moved(std::integral_constant<int, 0x140>{});  // row_mirror
    v += moved(std::integral_constant<int, 0x141>{});  // row_half_mirror
    v += moved(std::integral_constant<int, 0x4e>{});   // quad_perm [2, 3, 0, 1]
    v += moved(std::integral_constant<int, 0xb1>{});   // quad_perm [1, 0, 3, 2]
    return v;
}

template <typename C, int NT>
__global__ void __launch_bounds__(NT)
k_adj_tile(const C* __restrict__ lam_in, const C* __restrict__ tape, AdjArgs<C> a, AdjTile g,
           C* __restrict__ lam_out, double* __restrict__ part)
{
#pragma clang fp contract(off)
    constexpr int NC = kAdjTileMax * kAdjTileMax / NT, NS = 2 * NC;  // slots: own sites, then the halo's
    constexpr int kPlane = kBRegion * kBRegion;
    extern __shared__ double lds[];
    C* const psi = reinterpret_cast<C*>(lds);
    C* const hx = psi + kEPitch * kEPitch;
    C* const hy = hx + kARegion * kARegion;
    C* const lam = hy + kARegion * kARegion;

    const int tid = threadIdx.x, lane = tid & 63;
    const int lb = xcd_remap(blockIdx.x, gridDim.x);
    const int sy = lb / g.tiles_x;
    const int x0 = (lb - sy * g.tiles_x) * g.tx, y0 = sy * g.ty;
    const int nx = a.nx, ny = a.ny, own = g.tx * g.ty;
    const int h0 = 3 * (g.steps - 1);  // halo of the lambda planes; psi g_F has 2 more, psi 4 more

    // The slot's site at step j with halo r, as y 2^16 + x, each off by kOff; -1
    // where it has none (waves without any skip the slot).
    constexpr int kOff = 64;
    auto place = [&](int m, int j, int r) {
        const int i = tid + (m < NC ? m : m - NC) * NT;
        int x, y, n = own;
        if (m < NC) {
            y = div32(i, g.magic_tx);
            x = i - y * g.tx;
        } else {
            n = 2 * r * (g.tx + 2 * r + g.ty);
            ring_site(i, g.tx, g.ty, r, g.magic_w[j], g.magic_2r[j], x, y);
        }
        return i < n ? (y + kOff) << 16 | (x + kOff) : -1;
    };
    auto site = [&](int place, int& x, int& y) {
        x = (place & 0xffff) - kOff;
        y = (place >> 16) - kOff;
        return place >= 0;
    };
    auto at = [&](int x, int y) { return wrapn(y0 + y, ny) * nx + wrapn(x0 + x, nx); };

    int pos[NS];                // the step's sites
    C P[NS] = {}, edge = (C)0;  // their psi, and that of the ring outside the halo
    auto load_psi = [&](int j) {
        const C* t = tape - (int64_t)j * 4 * a.N;
        const int r = 3 * (g.steps - 1 - j) + 2, w = g.tx + 2 * r, h = g.ty + 2 * r;
#pragma unroll
        for (int m = 0; m < NS; ++m) {
            pos[m] = place(m, j, r);
            int x, y;
            if (site(pos[m], x, y)) P[m] = ld32(t + 3 * a.N, at(x, y));
        }
        int x, y;
        ring_site(tid, w, h, 2, g.magic_e[j], 1u << 30, x, y);
        if (tid < 4 * (w + 4 + h)) edge = ld32(t + 3 * a.N, at(x - r, y - r));
    };
    load_psi(0);

    double* const slot = part + ((int64_t)lb * (NT / 64) + (tid >> 6)) * 2 + (lane >> 5);
    double sum = *slot;

#pragma unroll 1
    for (int j = 0; j < g.steps; ++j) {
        const int r = 3 * (g.steps - 1 - j) + 2;
        const bool last = j + 1 == g.steps;
        // Offsets and addresses anew in each part of the step: kept across the
        // steps, those of the tile's own sites would take half the registers.
        int64_t N = a.N;
        auto renew = [&](int (&v)[NS]) {
#pragma unroll
            for (int m = 0; m < NS; ++m) asm volatile("" : "+v"(v[m]));
            asm volatile("" : "+s"(N));
        };
        renew(pos);
        C M[NS][9], T[NS][3];
        const C* t = tape - (int64_t)j * 4 * a.N;
        // psi into LDS, mu into registers.
        {
            const int w = g.tx + 2 * r, h = g.ty + 2 * r;
            int x, y;
            ring_site(tid, w, h, 2, g.magic_e[j], 1u << 30, x, y);
            if (tid < 4 * (w + 4 + h)) psi[(y - r + h0 + 4) * kEPitch + x - r + h0 + 4] = edge;
        }
#pragma unroll
        for (int m = 0; m < NS; ++m) {
            int x, y;
            if (!site(pos[m], x, y)) continue;
            psi[(y + h0 + 4) * kEPitch + x + h0 + 4] = P[m];
            const int here = at(x, y);
#pragma unroll
            for (int v = 0; v < 3; ++v) T[m][v] = ld32(t + v * N, here);
            if (j == 0) {
                const int gx = wrapn(x0 + x, nx), gy = wrapn(y0 + y, ny) * nx;
                const int xs[3] = {gx == 0 ? nx - 1 : gx - 1, gx, gx == nx - 1 ? 0 : gx + 1};
                const int ys[3] = {gy == 0 ? (ny - 1) * nx : gy - nx, gy, gy == (ny - 1) * nx ? 0 : gy + nx};
#pragma unroll
                for (int i = 0; i < 9; ++i)
                    M[m][i] = ld32(lam_in + i * N, ys[1 + kQCy[i]] + xs[1 + kQCx[i]]);
            } else {
                const int e = (y + h0) * kBRegion + x + h0;
#pragma unroll
                for (int i = 0; i < 9; ++i) M[m][i] = lam[i * kPlane + e + kQCy[i] * kBRegion + kQCx[i]];
            }
        }
        __syncthreads();

        // Collision adjoint; M becomes lambda without the site term.
        renew(pos);
        C q[NS], dpsi[NS];
        double v0 = 0.0, v1 = 0.0;
#pragma unroll
        for (int m = 0; m < NS; ++m) {
            __builtin_amdgcn_sched_barrier(0);  // one site at a time: registers
            int x, y;
            if (!site(pos[m], x, y)) continue;
            const C* c = psi + (y + h0 + 4) * kEPitch + x + h0 + 4;
            const Stencil<C> st(c - 2 * kEPitch, c - kEPitch, c, c + kEPitch, c + 2 * kEPitch, 0);
            const SiteAdjoint<C> sa = adjoint_collide(st, T[m][0], T[m][1], T[m][2], a, M[m]);
            const int e = (y + h0 + 2) * kARegion + x + h0 + 2;
            hx[e] = sa.hx;
            hy[e] = sa.hy;
            q[m] = sa.q;
            dpsi[m] = sa.dpsi;
            if (m < NC && x0 + x < nx && y0 + y < ny) {
                v0 -= (double)st.p * ((double)sa.gx * (double)sa.s1x + (double)sa.gy * (double)sa.s1y);
                v1 -= (double)st.p * ((double)sa.gx * (double)sa.s2x + (double)sa.gy * (double)sa.s2y);
            }
        }
        sum += wave_sums(v0, v1);
        int now[NS];
#pragma unroll
        for (int m = 0; m < NS; ++m) now[m] = pos[m];
        if (!last) load_psi(j + 1);
        __syncthreads();

        // The site term, and lambda into LDS or, from the last step, memory.
        renew(now);
#pragma unroll
        for (int m = 0; m < NS; ++m) {
            if (m >= NC && last) break;
            __builtin_amdgcn_sched_barrier(0);
            int x, y;
            if (!site(now[m], x, y) || x < 2 - r || x >= g.tx + r - 2 || y < 2 - r || y >= g.ty + r - 2) continue;
            const int c = (y + h0 + 2) * kARegion + x + h0 + 2;
            const C gs = (link_sums<C, kARegion>(hx + c, hy + c, a) - q[m]) * dpsi[m];
            if (!last) {
                const int e = (y + h0) * kBRegion + x + h0;
#pragma unroll
                for (int i = 0; i < 9; ++i) lam[i * kPlane + e] = M[m][i] + gs;
            } else if (x0 + x < nx && y0 + y < ny) {
                const int64_t e = (int64_t)(y0 + y) * nx + x0 + x;
#pragma unroll
                for (int i = 0; i < 9; ++i) lam_out[i * N + e] = M[m][i] + gs;
            }
        }
        if (!last) __syncthreads();
    }
    if ((lane & 31) == 0) *slot = sum;
}

// Interface measure: a(x) = sqrt(Dx^2 + Dy^2 + eps^2) from central
// differences of rho; stores (Dx/a, Dy/a) and the workgroup sums of a.
template <typename C>
__global__ void __launch_bounds__(kThreads)
k_adj_area(const C* __restrict__ tape, AdjArgs<C> a, C eps, C* __restrict__ dir,
           double* __restrict__ part)
{
    const int64_t s = (int64_t)blockIdx.x * kThreads + threadIdx.x;
    double v[1] = {0.0};
    if (s < a.N) {
        const int x = (int)(s % a.nx), y = (int)(s / a.nx);
        const int64_t row = (int64_t)y * a.nx;
        const C dx = (C)0.5 * (tape[row + wrapn(x + 1, a.nx)] - tape[row + wrapn(x - 1, a.nx)]);
        const C dy = (C)0.5 * (tape[(int64_t)wrapn(y + 1, a.ny) * a.nx + x] -
                               tape[(int64_t)wrapn(y - 1, a.ny) * a.nx + x]);
        const C len = sq(dx * dx + dy * dy + eps * eps);
        dir[s] = dx / len;
        dir[a.N + s] = dy / len;
        v[0] = (double)len;
    }
    block_sum<1>(v, part);
}

// Seed at T: lambda_i(x, T) = dL/drho(x) for every i, with
// dL/drho = 2 (E - E*) dE/dpsi psi' + beta dA/drho,
// dE/dpsi(x) = KE_0 psi(x) + sum_k K_k psi(x + c_k); also the workgroup sums
// of dE/dG1 = 1/2 sum psi (w_0 psi + sum w_k psi_k) and dE/dG2 likewise with
// p_s0, p_k.
template <typename C>
__global__ void __launch_bounds__(kThreads)
k_adj_seed(const C* __restrict__ tape, const C* __restrict__ dir, AdjArgs<C> a, C two_dE, C beta,
           C* __restrict__ lam, double* __restrict__ part)
{
    const int64_t s = (int64_t)blockIdx.x * kThreads + threadIdx.x;
    double v[2] = {0.0, 0.0};
    if (s < a.N) {
        const int x = (int)(s % a.nx), y = (int)(s / a.nx);
        const C* psi = tape + 3 * a.N;
        const C p = psi[s];
        C e1 = (C)kW0 * p, e2 = (C)kPS0 * p;
#pragma unroll
        for (int k = 0; k < 24; ++k) {
            const C pn = psi[(int64_t)wrapn(y + kLy[k], a.ny) * a.nx + wrapn(x + kLx[k], a.nx)];
            if (k < 8) e1 += (C)kLw[k] * pn;
            e2 += (C)kLp[k] * pn;
        }
        const int64_t row = (int64_t)y * a.nx;
        const C dA = (C)0.5 * ((dir[row + wrapn(x - 1, a.nx)] - dir[row + wrapn(x + 1, a.nx)]) +
                               (dir[a.N + (int64_t)wrapn(y - 1, a.ny) * a.nx + x] -
                                dir[a.N + (int64_t)wrapn(y + 1, a.ny) * a.nx + x]));
        const C dpsi = (a.sqrt_rho0 - p) * a.inv_rho0;
        const C g = two_dE * (a.G1 * e1 + a.G2 * e2) * dpsi + beta * dA;
#pragma unroll
        for (int i = 0; i < 9; ++i) lam[i * a.N + s] = g;
        v[0] = 0.5 * (double)p * (double)e1;
        v[1] = 0.5 * (double)p * (double)e2;
    }
    block_sum<2>(v, part);
}

// dL/drho_init(x) = sum_i w_i lambda_i(x, 0) (populations start at w_i rho).
template <typename C>
__global__ void __launch_bounds__(kThreads)
k_adj_rho_grad(const C* __restrict__ lam, int64_t N, double* __restrict__ out)
{
    const int64_t s = (int64_t)blockIdx.x * kThreads + threadIdx.x;
    if (s >= N) return;
    double acc = 0.0;
#pragma unroll
    for (int i = 0; i < 9; ++i) acc += kQw[i] * (double)lam[i * N + s];
    out[s] = acc;
}

// out[v] = sum_b part[b * nv + v], in a fixed order (one workgroup).
__global__ void __launch_bounds__(kThreads)
k_adj_reduce(const double* __restrict__ part, int blocks, int nv, double* __restrict__ out)
{
    __shared__ double sm[kThreads];
    for (int v = 0; v < nv; ++v) {
        double s = 0.0;
        for (int b = threadIdx.x; b < blocks; b += kThreads) s += part[(int64_t)b * nv + v];
        sm[threadIdx.x] = s;
        __syncthreads();
        for (int w = kThreads / 2; w > 0; w >>= 1) {
            if ((int)threadIdx.x < w) sm[threadIdx.x] += sm[threadIdx.x + w];
            __syncthreads();
        }
        if (threadIdx.x == 0) out[v] = sm[0];
        __syncthreads();
    }
}

__global__ void __launch_bounds__(kThreads) k_adj_zero(double* __restrict__ p, int64_t n)
{
    const int64_t s = (int64_t)blockIdx.x * kThreads + threadIdx.x;
    if (s < n) p[s] = 0.0;
}

template <typename C>
AdjArgs<C> adj_args(const AdjParams& p)
{
    return AdjArgs<C>{p.nx, p.ny, (int64_t)p.nx * p.ny, (C)p.G1, (C)p.G2, (C)p.tau,
                      (C)(1.0 / p.tau), (C)p.sqrt_rho0, (C)p.inv_rho0,
                      (C)(p.G1 * kW1 + p.G2 * kP1), (C)(p.G1 * kW2 + p.G2 * kP2), (C)(2.0 * p.G2 * kP4),
                      (C)(p.G2 * kP5), (C)(2.0 * p.G2 * kP8)};
}

dim3 grid_of(int64_t n) { return dim3((unsigned)((n + kThreads - 1) / kThreads)); }

template <typename C, int NT>
hipError_t steps_nt(const AdjParams& p, const AdjTile& g, const void* lam_in, const void* tape, void* lam_out,
                    double* part, hipStream_t s)
{
    constexpr size_t lds = sizeof(C) * (kEPitch * kEPitch + 2 * kARegion * kARegion + 9 * kBRegion * kBRegion);
    hipLaunchKernelGGL((k_adj_tile<C, NT>), dim3(g.tiles), dim3(NT), lds, s, static_cast<const C*>(lam_in),
                       static_cast<const C*>(tape), adj_args<C>(p), g, static_cast<C*>(lam_out), part);
    return hipGetLastError();
}

template <typename C>
hipError_t steps_t(const AdjParams& p, const AdjTile& g, const void* lam_in, const void* tape, void* lam_out,
                   double* part, hipStream_t s)
{
    if constexpr (sizeof(C) == 4)
        if (g.threads == 1024) return steps_nt<C, 1024>(p, g, lam_in, tape, lam_out, part, s);
    return g.threads == 512 ? steps_nt<C, 512>(p, g, lam_in, tape, lam_out, part, s) : hipErrorInvalidValue;
}

template <typename C>
hipError_t seed_t(const AdjParams& p, const void* tape, const void* dir, double two_dE, double beta,
                  void* lam, double* part, hipStream_t s)
{
    const AdjArgs<C> a = adj_args<C>(p);
    hipLaunchKernelGGL(k_adj_seed<C>, grid_of(a.N), dim3(kThreads), 0, s,
                       static_cast<const C*>(tape), static_cast<const C*>(dir), a, (C)two_dE,
                       (C)beta, static_cast<C*>(lam), part);
    return hipGetLastError();
}

}  // namespace

int adj_blocks(int64_t n) { return (int)((n + kThreads - 1) / kThreads); }

hipError_t adj_tape(int storage, const void* st, const Geom& geom, const AdjParams& p, void* tape,
                    hipStream_t s)
{
    const int64_t N = (int64_t)p.nx * p.ny;
    if (storage == ST_F64)
        hipLaunchKernelGGL((k_adj_tape<double, double>), grid_of(N), dim3(kThreads), 0, s,
                           static_cast<const double*>(st), geom, adj_args<double>(p),
                           static_cast<double*>(tape));
    else if (storage == ST_F32)
        hipLaunchKernelGGL((k_adj_tape<float, float>), grid_of(N), dim3(kThreads), 0, s,
                           static_cast<const float*>(st), geom, adj_args<float>(p),
                           static_cast<float*>(tape));
    else
        return hipErrorInvalidValue;
    return hipGetLastError();
}

hipError_t adj_steps(const AdjParams& p, const AdjTile& g, const void* lam_in, const void* tape, void* lam_out,
                     double* part, hipStream_t s)
{
    const int r = 3 * g.steps - 1;  // halo of the first step
    if (g.steps < 1 || g.steps > kAdjMaxSteps || g.tx < 2 || g.tx + 6 * g.steps - 6 > kAdjTileMax + 6 ||
        g.ty + 6 * g.steps - 6 > kAdjTileMax + 6 || g.tx * g.ty > kAdjTileMax * kAdjTileMax ||
        2 * r * (g.tx + 2 * r + g.ty) > kAdjTileMax * kAdjTileMax || 4 * (g.tx + g.ty + 4 * r + 4) > g.threads)
        return hipErrorInvalidValue;
    return p.f64 ? steps_t<double>(p, g, lam_in, tape, lam_out, part, s)
                 : steps_t<float>(p, g, lam_in, tape, lam_out, part, s);
}

hipError_t adj_area(const AdjParams& p, const void* tape, double eps, void* dir, double* part,
                    hipStream_t s)
{
    const int64_t N = (int64_t)p.nx * p.ny;
    if (p.f64)
        hipLaunchKernelGGL(k_adj_area<double>, grid_of(N), dim3(kThreads), 0, s,
                           static_cast<const double*>(tape), adj_args<double>(p), eps,
                           static_cast<double*>(dir), part);
    else
        hipLaunchKernelGGL(k_adj_area<float>, grid_of(N), dim3(kThreads), 0, s,
                           static_cast<const float*>(tape), adj_args<float>(p), (float)eps,
                           static_cast<float*>(dir), part);
    return hipGetLastError();
}

hipError_t adj_seed(const AdjParams& p, const void* tape, const void* dir, double two_dE, double beta,
                    void* lam, double* part, hipStream_t s)
{
    return p.f64 ? seed_t<double>(p, tape, dir, two_dE, beta, lam, part, s)
                 : seed_t<float>(p, tape, dir, two_dE, beta, lam, part, s);
}

hipError_t adj_rho_grad(const AdjParams& p, const void* lam, double* out, hipStream_t s)
{
    const int64_t N = (int64_t)p.nx * p.ny;
    if (p.f64)
        hipLaunchKernelGGL(k_adj_rho_grad<double>, grid_of(N), dim3(kThreads), 0, s,
                           static_cast<const double*>(lam), N, out);
    else
        hipLaunchKernelGGL(k_adj_rho_grad<float>, grid_of(N), dim3(kThreads), 0, s,
                           static_cast<const float*>(lam), N, out);
    return hipGetLastError();
}

hipError_t adj_reduce(const double* part, int blocks, int nv, double* out, hipStream_t s)
{
    hipLaunchKernelGGL(k_adj_reduce, dim3(1), dim3(kThreads), 0, s, part, blocks, nv, out);
    return hipGetLastError();
}

hipError_t adj_zero(double* p, int64_t n, hipStream_t s)
{
    hipLaunchKernelGGL(k_adj_zero, grid_of(n), dim3(kThreads), 0, s, p, n);
    return hipGetLastError();
}

}  // namespace lbk
