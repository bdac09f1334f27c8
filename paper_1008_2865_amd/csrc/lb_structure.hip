// Structure factor of the density field (the Fourier analysis of section
// IV): S(k) = (1/N) |sum_x (rho(x) - mean rho) e^{i k.x}|^2 on the modes
// k = (2 pi / L)(l, m) of an L x L lattice, its average over the circular
// shells (n - 1/2) <= |k| L / 2 pi < n + 1/2 and the first moment
// kbar = sum_n n S_n / sum_n S_n (eq. (rad), k in units of 2 pi / L).
//
// Three passes, all in double precision:
//   k_sk_rows    two real rows per workgroup as one complex line, transformed
//                in LDS and separated; only l = 0 .. L/2 is stored, since
//                S(k) = S(-k);
//   k_sk_columns 4, 2 or 1 columns per workgroup, transformed in LDS; S of
//                the columns, and the sum of S over each run of a column's
//                modes that lies in one shell;
//   k_sk_shells  one wave per shell adds those runs over the columns.
// The sign of the exponent does not matter for |.|^2 of a real field; the
// passes use e^{-i k.x}.  Twiddles come from a table computed once
// (sincospi).  Every sum has a fixed order, so results are bit-reproducible.
//
// What bounds it: the passes' chains of LDS round trips (a barrier twice per
// radix), one round of workgroups each; at 2048^2 22 us for the rows, 30 for
// the columns, 4 for the shells, against 20 us for the bytes at a copy's
// rate.  The passes move 33.5 MB of density, 33.6 MB of row spectra out and
// in again, and 2 x 6 MB of run sums, where a full complex transform with a
// transpose and a gather of every mode into its shell moved 386 MB.  A whole
// evaluation on MI355X: 2048^2 235 -> 71.5 us, 1000^2 (radices 8, 5, 5, 5 in
// place of the direct sum) 1407 -> 51, 521^2 (by convolution) 347 -> 59, 2039^2
// 9339 -> 160, 512^2 82 -> 40, 40^2 71 -> 29.
#include "lb_internal.h"

#include <hip/hip_runtime.h>

#include <initializer_list>

namespace lbk {
namespace {

constexpr int kThreads = 256;
constexpr int kTile = 32;

// tw[k] = exp(-2 pi i k / L), k < L (once per context).
__global__ void __launch_bounds__(kThreads) k_sk_twiddles(int L, double2* __restrict__ tw)
{
    const int k = blockIdx.x * kThreads + threadIdx.x;
    if (k >= L) return;
    double s, c;
    sincospi(-2.0 * (double)k / (double)L, &s, &c);
    tw[k] = make_double2(c, s);
}

// ---------------------------------------------------------------------------
// One-line transforms in LDS: a Stockham autosort FFT of mixed radix.  A pass
// of radix r over sub-transforms of length s takes, for j < L/r, jd = j / s
// and k = j % s, the inputs x[j + q L/r] times w_{rs}^{q k}, q < r, and
// writes their r-point transform to x[jd s r + k + p s], p < r.  A thread
// holds its butterflies in registers between reading and writing, so the
// line stays in one LDS buffer; at most kPerThread values per thread.
// ---------------------------------------------------------------------------
constexpr int kPerThread = 8;

// LDS position of element i: one element of padding after every eight, so
// that the first pass's stores (8 elements apart) spread over the banks.
__host__ __device__ __forceinline__ int pad(int i) { return i + (i >> 3); }

// v / d for 0 <= v < 2^16 with magic = ceil(2^32 / d), d >= 2; d = 1 has
// magic 0.
__device__ __forceinline__ int divm(int v, uint32_t magic)
{
    return magic ? (int)__umulhi((uint32_t)v, magic) : v;
}

__device__ __forceinline__ double2 add(double2 a, double2 b) { return make_double2(a.x + b.x, a.y + b.y); }
__device__ __forceinline__ double2 sub(double2 a, double2 b) { return make_double2(a.x - b.x, a.y - b.y); }
__device__ __forceinline__ double2 mul(double2 a, double2 w)
{
    return make_double2(a.x * w.x - a.y * w.y, a.x * w.y + a.y * w.x);
}
__device__ __forceinline__ double2 mul_mi(double2 a) { return make_double2(a.y, -a.x); }  // -i a

__device__ __forceinline__ void dft(double2 (&v)[2])
{
    const double2 a = v[0];
    v[0] = add(a, v[1]);
    v[1] = sub(a, v[1]);
}
__device__ __forceinline__ void dft(double2 (&v)[3])
{
    constexpr double kS = 0.86602540378443864676;  // sin(2 pi / 3)
    const double2 t = add(v[1], v[2]), d = sub(v[1], v[2]);
    const double2 a = make_double2(v[0].x - 0.5 * t.x, v[0].y - 0.5 * t.y);
    const double2 b = make_double2(kS * d.y, -kS * d.x);
    v[0] = add(v[0], t);
    v[1] = add(a, b);
    v[2] = sub(a, b);
}
__device__ __forceinline__ void dft(double2 (&v)[4])
{
    const double2 a = add(v[0], v[2]), b = sub(v[0], v[2]);
    const double2 c = add(v[1], v[3]), d = mul_mi(sub(v[1], v[3]));
    v[0] = add(a, c);
    v[1] = add(b, d);
    v[2] = sub(a, c);
    v[3] = sub(b, d);
}
__device__ __forceinline__ void dft(double2 (&v)[5])
{
    constexpr double kC1 = 0.30901699437494742410, kC2 = -0.80901699437494742410;  // cos 72, cos 144
    constexpr double kS1 = 0.95105651629515357212, kS2 = 0.58778525229247312917;   // sin 72, sin 144
    const double2 t1 = add(v[1], v[4]), t2 = add(v[2], v[3]);
    const double2 d1 = sub(v[1], v[4]), d2 = sub(v[2], v[3]);
    const double2 a1 = make_double2(v[0].x + kC1 * t1.x + kC2 * t2.x, v[0].y + kC1 * t1.y + kC2 * t2.y);
    const double2 a2 = make_double2(v[0].x + kC2 * t1.x + kC1 * t2.x, v[0].y + kC2 * t1.y + kC1 * t2.y);
    const double2 b1 = mul_mi(make_double2(kS1 * d1.x + kS2 * d2.x, kS1 * d1.y + kS2 * d2.y));
    const double2 b2 = mul_mi(make_double2(kS2 * d1.x - kS1 * d2.x, kS2 * d1.y - kS1 * d2.y));
    v[0] = add(v[0], add(t1, t2));
    v[1] = add(a1, b1);
    v[4] = sub(a1, b1);
    v[2] = add(a2, b2);
    v[3] = sub(a2, b2);
}
__device__ __forceinline__ void dft(double2 (&v)[7])
{
    // cos and sin of 2 pi k / 7, k = 1 .. 3.
    constexpr double kC[3] = {0.62348980185873353053, -0.22252093395631440429, -0.90096886790241912624};
    constexpr double kS[3] = {0.78183148246802980871, 0.97492791218182360702, 0.43388373911755812048};
    double2 t[3], d[3], out[7];
    out[0] = v[0];
#pragma unroll
    for (int q = 0; q < 3; ++q) {
        t[q] = add(v[q + 1], v[6 - q]);
        d[q] = sub(v[q + 1], v[6 - q]);
        out[0] = add(out[0], t[q]);
    }
#pragma unroll
    for (int p = 1; p < 4; ++p) {
        double2 a = v[0], b = make_double2(0.0, 0.0);
#pragma unroll
        for (int q = 0; q < 3; ++q) {
            const int k = p * (q + 1) % 7, m = k > 3 ? 7 - k : k;  // cos k = cos m, sin k = -sin m beyond 3
            const double sn = k > 3 ? -kS[m - 1] : kS[m - 1];
            a = make_double2(a.x + kC[m - 1] * t[q].x, a.y + kC[m - 1] * t[q].y);
            b = make_double2(b.x + sn * d[q].x, b.y + sn * d[q].y);
        }
        b = mul_mi(b);
        out[p] = add(a, b);
        out[7 - p] = sub(a, b);
    }
#pragma unroll
    for (int p = 0; p < 7; ++p) v[p] = out[p];
}
__device__ __forceinline__ void dft(double2 (&v)[8])
{
    constexpr double kH = 0.70710678118654752440;
    double2 e[4] = {v[0], v[2], v[4], v[6]}, o[4] = {v[1], v[3], v[5], v[7]};
    dft(e);
    dft(o);
    o[1] = make_double2(kH * (o[1].x + o[1].y), kH * (o[1].y - o[1].x));   // e^{-i pi/4}
    o[2] = mul_mi(o[2]);
    o[3] = make_double2(kH * (o[3].y - o[3].x), -kH * (o[3].x + o[3].y));  // e^{-3 i pi/4}
#pragma unroll
    for (int q = 0; q < 4; ++q) {
        v[q] = add(e[q], o[q]);
        v[q + 4] = sub(e[q], o[q]);
    }
}

template <int R>
__device__ __forceinline__ void
fft_pass(double2* x, int lines, int lp, int n, int s, uint32_t magic_s, uint32_t magic_m,
         const double2* __restrict__ tw)
{
    constexpr int NB = (kPerThread + R - 1) / R;  // butterflies per thread
    const int T = blockDim.x, tid = threadIdx.x;
    const int m = n / R, total = lines * m, tstep = m / s;
    double2 v[NB][R];
    int at[NB];
#pragma unroll
    for (int b = 0; b < NB; ++b) {
        // Past the end: the last butterfly again, not stored, so that the
        // loads of all of a thread's butterflies overlap.
        const int idx = min(tid + b * T, total - 1);
        const int c = divm(idx, magic_m), j = idx - c * m;
        const int jd = divm(j, magic_s), k = j - jd * s;
        const double2* in = x + c * lp;
#pragma unroll
        for (int q = 0; q < R; ++q) v[b][q] = in[pad(j + q * m)];
        if (s > 1) {
            const int t = k * tstep;
            double2 w[R];
            if constexpr (R == 8) {
                // Three table reads; the other four are single products.
                w[1] = tw[t];
                w[2] = tw[2 * t];
                w[4] = tw[4 * t];
                w[3] = mul(w[1], w[2]);
                w[5] = mul(w[1], w[4]);
                w[6] = mul(w[2], w[4]);
                w[7] = mul(w[3], w[4]);
            } else {
#pragma unroll
                for (int q = 1; q < R; ++q) w[q] = tw[q * t];
            }
#pragma unroll
            for (int q = 1; q < R; ++q) v[b][q] = mul(v[b][q], w[q]);
        }
        dft(v[b]);
        at[b] = jd * s * R + k;
    }
    __syncthreads();
#pragma unroll
    for (int b = 0; b < NB; ++b) {
        const int idx = tid + b * T;
        if (idx >= total) continue;
        double2* out = x + divm(idx, magic_m) * lp;
#pragma unroll
        for (int p = 0; p < R; ++p) out[pad(at[b] + p * s)] = v[b][p];
    }
    __syncthreads();
}

// All passes of `lines` lines of length f.m, line c at x[c lp + pad(i)].
// Needs lines * f.m <= kPerThread * blockDim.x, and a barrier before it.
__device__ __forceinline__ void
fft_passes(double2* x, int lines, int lp, const SkFft& f, const double2* __restrict__ tw)
{
    int s = 1;
    for (int p = 0; p < f.passes; ++p) {
        const int r = f.radix[p];
        const uint32_t ms = f.magic_s[p], mm = f.magic_m[p];
        switch (r) {
        case 8: fft_pass<8>(x, lines, lp, f.m, s, ms, mm, tw); break;
        case 4: fft_pass<4>(x, lines, lp, f.m, s, ms, mm, tw); break;
        case 2: fft_pass<2>(x, lines, lp, f.m, s, ms, mm, tw); break;
        case 3: fft_pass<3>(x, lines, lp, f.m, s, ms, mm, tw); break;
        case 5: fft_pass<5>(x, lines, lp, f.m, s, ms, mm, tw); break;
        default: fft_pass<7>(x, lines, lp, f.m, s, ms, mm, tw); break;
        }
        s *= r;
    }
}

// The transform of `lines` lines of length f.n.  A length with a prime factor
// above 7 goes by Bluestein's convolution: with b_i = e^{i pi i^2 / n},
//   X_k = b*_k sum_i (x_i b*_i) b_{k-i},
// a cyclic convolution of a smooth length f.m >= 2 n - 1: transform x b*, times
// the transform of b (over m), inverse transform (by conjugation).  The line
// then holds f.m elements.
template <bool kChirp>
__device__ __forceinline__ void
fft_lines(double2* x, int lines, int lp, const SkFft& f, const SkTables& t)
{
    if constexpr (!kChirp) {
        fft_passes(x, lines, lp, f, t.tw);
    } else {
        const int T = blockDim.x, tid = threadIdx.x, m = f.m;
        // This thread's elements of the lines, each time the same.
        auto each = [&](auto&& fn) {
#pragma unroll
            for (int b = 0; b < kPerThread; ++b) {
                const int idx = tid + b * T;
                if (idx >= lines * m) break;
                const int c = idx / m, i = idx - c * m;
                fn(x[c * lp + pad(i)], i);
            }
            __syncthreads();
        };
        auto conj = [](double2 v) { return make_double2(v.x, -v.y); };
        each([&](double2& v, int i) { v = i < f.n ? mul(v, conj(t.chirp[i])) : make_double2(0.0, 0.0); });
        fft_passes(x, lines, lp, f, t.tw);
        each([&](double2& v, int i) { v = conj(mul(v, t.filter[i])); });
        fft_passes(x, lines, lp, f, t.tw);
        each([&](double2& v, int i) {
            if (i < f.n) v = conj(mul(v, t.chirp[i]));
        });
    }
}

// chirp[i] = e^{i pi i^2 / n}, i < n, and the filter: its transform as a
// cyclic sequence of length m (b_i at i and m - i), over m.  One workgroup.
__global__ void __launch_bounds__(512)
k_sk_chirp(SkFft f, const double2* __restrict__ tw, double2* __restrict__ chirp, double2* __restrict__ filter)
{
    extern __shared__ double2 lds[];
    const int n = f.n, m = f.m;
    for (int i = threadIdx.x; i < m; i += blockDim.x) {
        const int d = min(i, m - i);  // distance on the cycle
        double2 v = make_double2(0.0, 0.0);
        if (d < n) {
            double sn, cs;
            sincospi((double)((int64_t)d * d % (2 * n)) / (double)n, &sn, &cs);
            v = make_double2(cs, sn);
            if (i < n) chirp[i] = v;
        }
        lds[pad(i)] = v;
    }
    __syncthreads();
    fft_passes(lds, 1, 0, f, tw);
    for (int i = threadIdx.x; i < m; i += blockDim.x) {
        const double2 v = lds[pad(i)];
        filter[i] = make_double2(v.x / (double)m, v.y / (double)m);
    }
}

// Fixed-order workgroup sum of NV values per thread; every thread receives
// the results.  red holds NV x waves doubles (at most 16 waves) and serves one
// sum: nothing waits for its readers.
template <int NV>
__device__ __forceinline__ void block_sum(double (&v)[NV], double* red)
{
    const int lane = threadIdx.x & 63, wid = threadIdx.x >> 6, waves = blockDim.x >> 6;
#pragma unroll
    for (int q = 0; q < NV; ++q) {
#pragma unroll
        for (int m = 32; m >= 1; m >>= 1) v[q] += __shfl_xor(v[q], m, 64);
        if (lane == 0) red[q * 16 + wid] = v[q];
    }
    __syncthreads();
#pragma unroll
    for (int q = 0; q < NV; ++q) {
        double t[16];
#pragma unroll
        for (int w = 0; w < 16; ++w) t[w] = w < waves ? red[q * 16 + w] : 0.0;
#pragma unroll
        for (int h = 8; h >= 1; h >>= 1)
#pragma unroll
            for (int w = 0; w < h; ++w) t[w] += t[w + h];
        v[q] = t[0];
    }
}

// Sum of kPerThread values, pairwise.
__device__ __forceinline__ double pairwise(const double (&v)[kPerThread])
{
    return ((v[0] + v[1]) + (v[2] + v[3])) + ((v[4] + v[5]) + (v[6] + v[7]));
}

// Rows 2b and 2b + 1 of rho as the real and imaginary part of one line, each
// less a number close to its mean, which mean[y] keeps: l = 0 of the transform is
// then the sum of what is left, and neither it nor mean[y] - mean[0] carries the
// rounding of the mean (S(0, m) of noise 1e-6 about 0.7 would be wrong by 5e-9 of
// itself if the rows' plain sums were stored).  That number is taken from the
// differences to the row's first value, so a uniform row leaves exact zeros.
// z[y][l], l < hc: the row spectra for l = 0 .. hc - 1; for even L the real
// values at l = 0 and l = L/2 share entry 0, as its real and imaginary part.
// LDS: pad(f.m) + 2 elements.
template <bool kChirp>
__global__ void __launch_bounds__(kChirp ? 512 : 256)
k_sk_rows(const double* __restrict__ rho, SkFft f, SkTables t, int hc, double2* __restrict__ z,
          double* __restrict__ mean)
{
    extern __shared__ double2 lds[];
    __shared__ double red[2 * 16];
    const int n = f.n, tid = threadIdx.x, T = blockDim.x;
    double2* x = lds;
    const int64_t ya = 2 * (int64_t)blockIdx.x;
    const bool two = ya + 1 < n;
    const double* ra = rho + ya * n;
    const double* rb = two ? ra + n : ra;
    const double a0 = ra[0], b0 = rb[0];
    double va[kPerThread], vb[kPerThread], da[kPerThread], db[kPerThread];
#pragma unroll
    for (int b = 0; b < kPerThread; ++b) {
        const int i = tid + b * T;
        va[b] = i < n ? ra[i] : a0;
        vb[b] = i < n ? rb[i] : b0;
        da[b] = va[b] - a0;
        db[b] = vb[b] - b0;
    }
    double sum[2] = {pairwise(da), pairwise(db)};
    block_sum<2>(sum, red);
    const double ma = a0 + sum[0] / (double)n, mb = b0 + sum[1] / (double)n;
#pragma unroll
    for (int b = 0; b < kPerThread; ++b) {
        const int i = tid + b * T;
        if (i < n) x[pad(i)] = make_double2(va[b] - ma, vb[b] - mb);
    }
    if (tid == 0) {
        mean[ya] = ma;
        if (two) mean[ya + 1] = mb;
    }
    __syncthreads();
    fft_lines<kChirp>(x, 1, 0, f, t);
    double2* za = z + ya * hc;
    double2* zb = za + hc;
    for (int k = tid; k < hc; k += T) {
        const double2 p = x[pad(k)], q = x[pad(k ? n - k : 0)];
        double2 a = make_double2(0.5 * (p.x + q.x), 0.5 * (p.y - q.y));
        double2 b = make_double2(0.5 * (p.y + q.y), 0.5 * (q.x - p.x));
        if (k == 0) {
            const double2 h = (n & 1) ? make_double2(0.0, 0.0) : x[pad(n / 2)];
            a = make_double2(p.x, h.x);
            b = make_double2(p.y, h.y);
        }
        za[k] = a;
        if (two) zb[k] = b;
    }
}

// Smallest m >= 0 with 4 (l^2 + m^2) >= (2n - 1)^2: the first mode of
// column l in shell n or beyond.
__device__ __forceinline__ int shell_begin(int n, int l)
{
    if (n == 0) return 0;
    const int v = (2 * n - 1) * (2 * n - 1) - 4 * l * l;
    if (v <= 0) return 0;
    int m = (int)(0.5f * sqrtf((float)v));
    while (4 * m * m < v) ++m;
    while (m > 0 && 4 * (m - 1) * (m - 1) >= v) --m;
    return m;
}

// Shell of l^2 + h^2.
__device__ __forceinline__ int shell_at(int l, int h)
{
    const int q4 = 4 * (l * l + h * h);
    int n = (int)(0.5f * sqrtf((float)q4) + 0.5f);
    while ((2 * n + 1) * (2 * n + 1) <= q4) ++n;
    while (n > 0 && (2 * n - 1) * (2 * n - 1) > q4) --n;
    return n;
}

// `cols` columns per workgroup (a power of two, log2 = lc).  mean: the numbers
// subtracted from the rows.  spec (may be
// NULL): S at [l][m], l = 0 .. L/2.  part[n][l], pitch hp: the sum of S over
// the modes (+-l, m) of shell n, each m in ascending order with its -m.  LDS:
// cols (pad(f.m) + 2) elements.  A segment of four columns is 64 bytes of a row
// of z.
template <bool kChirp>
__global__ void __launch_bounds__(1024)
k_sk_columns(const double2* __restrict__ z, const double* __restrict__ mean, SkFft f, SkTables t, int hc, int lc,
             double invN,
             double* __restrict__ spec, double* __restrict__ part, int hp)
{
    extern __shared__ double2 lds[];
    __shared__ double red[16];
    const int n = f.n, tid = threadIdx.x, T = blockDim.x;
    const int cols = 1 << lc, lp = pad(f.m) + 2, h = n / 2;
    const bool even = (n & 1) == 0;
    double2* x = lds;
    // Consecutive column groups share the lines of z: keep them on one XCD.
    const int per_xcd = gridDim.x / 8, rem = gridDim.x % 8, xcd = blockIdx.x % 8;
    const int group = xcd * per_xcd + min(xcd, rem) + blockIdx.x / 8;
    const int l0 = group << lc;
    const int nc = min(cols, hc - l0);
    {
        // Column l = 0 also needs the rows' means: loaded with the rest.
        double2 v[kPerThread];
        double m[kPerThread] = {}, m0 = 0.0;
        if (l0 == 0) {
            m0 = mean[0];
#pragma unroll
            for (int b = 0; b < kPerThread; ++b) {
                const int i = tid + b * T, y = i >> lc;
                m[b] = mean[(i & (cols - 1)) == 0 && y < n ? y : 0];
            }
        }
#pragma unroll
        for (int b = 0; b < kPerThread; ++b) {
            const int i = tid + b * T, y = i >> lc, c = i & (cols - 1);
            v[b] = y < n && c < nc ? z[(int64_t)y * hc + l0 + c] : make_double2(0.0, 0.0);
        }
#pragma unroll
        for (int b = 0; b < kPerThread; ++b) {
            const int i = tid + b * T, y = i >> lc, c = i & (cols - 1);
            if (y < n) x[c * lp + pad(y)] = v[b];
        }
        if (l0 == 0) {
            // Column l = 0 (real parts): the rows' sums, each the transform's l = 0
            // and n times what the row's mean differs from theirs.
            double s[kPerThread];
#pragma unroll
            for (int b = 0; b < kPerThread; ++b) s[b] = m[b] - m0;
            double sum[1] = {pairwise(s)};
            block_sum<1>(sum, red);
            const double centre = m0 + sum[0] / (double)n;
#pragma unroll
            for (int b = 0; b < kPerThread; ++b) {
                const int i = tid + b * T, y = i >> lc;
                if ((i & (cols - 1)) == 0 && y < n) x[pad(y)].x = v[b].x + (double)n * (m[b] - centre);
            }
        }
    }
    __syncthreads();
    fft_lines<kChirp>(x, cols, lp, f, t);

    // S in place: .x of every column; for column 0 the columns l = 0 (.x)
    // and, for even L, l = L/2 (.y), separated as in k_sk_rows.
    for (int i = tid; i < nc * n; i += T) {
        const int c = i / n, y = i - c * n;
        if (l0 + c == 0) {
            if (2 * y > n) continue;
            const int y2 = y ? n - y : 0;
            const double2 p = x[pad(y)], q = x[pad(y2)];
            const double ar = 0.5 * (p.x + q.x), ai = 0.5 * (p.y - q.y);
            const double br = 0.5 * (p.y + q.y), bi = 0.5 * (q.x - p.x);
            const double2 s = make_double2((ar * ar + ai * ai) * invN, (br * br + bi * bi) * invN);
            x[pad(y)] = s;
            x[pad(y2)] = s;
        } else {
            const double2 p = x[c * lp + pad(y)];
            x[c * lp + pad(y)].x = (p.x * p.x + p.y * p.y) * invN;
        }
    }
    __syncthreads();

    // Each column has T / cols threads (and column l = L/2 all of them, after
    // the others): a column's longest runs are those of its first shells, so
    // one thread group per column overlaps them.
    auto column = [&](int l, int first, int stride, auto S) {
        if (spec)
            for (int m = first; m < n; m += stride) spec[(int64_t)l * n + m] = S(m);
        const double w = l == 0 || (even && l == h) ? 1.0 : 2.0;
        const int last = shell_at(l, h);
        for (int sh = l + first; sh <= last; sh += stride) {
            int m = shell_begin(sh, l);
            const int b = min(shell_begin(sh + 1, l) - 1, h);
            auto both = [&](int v) { return v == 0 || (even && v == h) ? S(v) : S(v) + S(n - v); };
            double s = 0.0;
            for (; m + 3 <= b; m += 4) {
                const double v0 = both(m), v1 = both(m + 1), v2 = both(m + 2), v3 = both(m + 3);
                s += (v0 + v1) + (v2 + v3);
            }
            for (; m <= b; ++m) s += both(m);
            part[(int64_t)sh * hp + l] = w * s;
        }
    };
    const int per = T >> lc, c = tid / per;  // T is a multiple of 64, cols of at most 4
    if (c < nc) column(l0 + c, tid - c * per, per, [&](int m) { return x[c * lp + pad(m)].x; });
    if (l0 == 0 && even) column(h, tid, T, [&](int m) { return x[pad(m)].y; });
}

// Shell n (one wave each): the run sums of its columns over its modes.
__global__ void __launch_bounds__(kThreads)
k_sk_shells(const double* __restrict__ part, int hp, int L, int nshell,
            const double* __restrict__ count, double* __restrict__ shell)
{
    const int n = blockIdx.x * (kThreads / 64) + (threadIdx.x >> 6), lane = threadIdx.x & 63;
    if (n >= nshell) return;
    const int h = L / 2;
    // Columns with modes in shell n: from the first whose last mode (l, h)
    // reaches it up to l = n.
    const int a = shell_begin(n, h), b = min(n, h);
    double s = 0.0;
#pragma unroll 4
    for (int l = a + lane; l <= b; l += 64) s += part[(int64_t)n * hp + l];
#pragma unroll
    for (int m = 32; m >= 1; m >>= 1) s += __shfl_xor(s, m, 64);
    if (lane == 0) shell[n] = s / count[n];
}

// The caller's full spectrum out[m][l] from the half spectrum in[l][m],
// l <= L/2, through 32 x 32 LDS tiles: each value at (l, m) and (-l, -m).
__global__ void __launch_bounds__(kThreads)
k_sk_spread(const double* __restrict__ in, int L, double* __restrict__ out)
{
    __shared__ double tile[kTile][kTile + 1];
    const int tx = threadIdx.x & (kTile - 1), ty = threadIdx.x / kTile;  // 32 x 8
    const int m0 = blockIdx.x * kTile, l0 = blockIdx.y * kTile, h = L / 2;
    for (int r = ty; r < kTile; r += kThreads / kTile)
        if (l0 + r <= h && m0 + tx < L) tile[r][tx] = in[(int64_t)(l0 + r) * L + m0 + tx];
    __syncthreads();
    for (int r = ty; r < kTile; r += kThreads / kTile) {
        const int m = m0 + r, l = l0 + tx;
        if (m >= L || l > h) continue;
        const double v = tile[tx][r];
        out[(int64_t)m * L + l] = v;
        if (l > 0 && 2 * l != L) out[(int64_t)(m ? L - m : 0) * L + L - l] = v;
    }
}

// Whole waves of kPerThread values a thread.
dim3 lanes(int values) { return dim3((values + 64 * kPerThread - 1) / (64 * kPerThread) * 64); }

template <bool kChirp>
hipError_t passes(const SkPlan& p, const double* rho, double* spec, hipStream_t s)
{
    const SkFft& f = p.fft;
    const int n = f.n, cols = 1 << p.log_cols;
    hipLaunchKernelGGL(k_sk_rows<kChirp>, dim3((n + 1) / 2), lanes(f.m), sk_lds(f, 1), s, rho, f, p.t, p.hc, p.z, p.mean);
    hipLaunchKernelGGL(k_sk_columns<kChirp>, dim3((p.hc + cols - 1) / cols), lanes(f.m * cols), sk_lds(f, cols), s,
                       p.z, p.mean, f, p.t, p.hc, p.log_cols, 1.0 / ((double)n * (double)n), spec, p.part, p.hp);
    return hipGetLastError();
}

}  // namespace

size_t sk_lds(const SkFft& f, int cols)
{
    return (size_t)(pad(f.m) + 2) * cols * sizeof(double2);
}

SkFft sk_fft(int L)
{
    SkFft f{};
    f.n = f.m = L;
    auto smooth = [](int v, std::initializer_list<int> primes) {
        for (int r : primes)
            while (v % r == 0) v /= r;
        return v == 1;
    };
    if (!smooth(L, {2, 3, 5, 7})) {
        // The smallest length of factors 2, 3, 5 that is a multiple of 8.
        f.chirp = 1;
        for (f.m = (2 * L - 1 + 7) / 8 * 8; !smooth(f.m, {2, 3, 5});) f.m += 8;
    }
    auto magic = [](int d) { return d > 1 ? (uint32_t)(((uint64_t(1) << 32) + d - 1) / d) : 0u; };
    int s = 1;
    for (int r : {8, 4, 2, 5, 3, 7})
        for (; f.m / s % r == 0; s *= r) {
            f.radix[f.passes] = r;
            f.magic_s[f.passes] = magic(s);
            f.magic_m[f.passes] = magic(f.m / r);
            ++f.passes;
        }
    return f;
}

hipError_t sk_prepare(const SkPlan& p, double2* tw, double2* chirp, double2* filter, hipStream_t s)
{
    const SkFft& f = p.fft;
    hipLaunchKernelGGL(k_sk_twiddles, dim3((f.m + kThreads - 1) / kThreads), dim3(kThreads), 0, s, f.m, tw);
    if (f.chirp)
        hipLaunchKernelGGL(k_sk_chirp, dim3(1), lanes(f.m), sk_lds(f, 1), s, f, tw, chirp, filter);
    return hipGetLastError();
}

hipError_t sk_compute(const SkPlan& p, const double* rho, double* spectrum, hipStream_t s)
{
    double* spec = spectrum ? p.spec : nullptr;
    const hipError_t e = p.fft.chirp ? passes<true>(p, rho, spec, s) : passes<false>(p, rho, spec, s);
    if (e) return e;
    const int L = p.fft.n, per = kThreads / 64;
    hipLaunchKernelGGL(k_sk_shells, dim3((p.nshell + per - 1) / per), dim3(kThreads), 0, s, p.part, p.hp, L,
                       p.nshell, p.count, p.shell);
    if (spectrum)
        hipLaunchKernelGGL(k_sk_spread, dim3((L + kTile - 1) / kTile, (L / 2 + kTile) / kTile),
                           dim3(kThreads), 0, s, spec, L, spectrum);
    return hipGetLastError();
}

}  // namespace lbk
