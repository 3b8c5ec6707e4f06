// Device bodies of the solve's kernels (gfx950): each takes its work item and
// its LDS explicitly, so that the single-solve kernels (one item per block)
// and the batched kernels (a work table over many plans) share one code path.
// The block size every body expects is given next to it.
#pragma once

#include <hip/hip_runtime.h>

#include "device_common.hpp"
#include "fft_reg.hpp"
#include "solver_kernels.hpp"

namespace phi {

__device__ __forceinline__ int posmod_dev(int a, int b) {
    int r = a % b;
    return r < 0 ? r + b : r;
}


// ---------------------------------------------------------------------------
// rows_forward
// ---------------------------------------------------------------------------

// Distance between the LDS buffers of the sequences of one block: the padded
// length plus 8 entries, so that lanes working on the same position of
// different sequences fall into different banks.
__host__ __device__ constexpr int lds_group_stride(int f) { return lds_padded_size(f) + 8; }

// Grid rows per block of the row kernels: as many as fit 1024 threads and about
// 70 KB of LDS (one FFT buffer per row, two blocks per CU), so the column-major
// spectrum is written and read in segments of G consecutive rows (two rows in
// FP32, one in FP64 at the long transforms: measured best among 1, 2 and 4).
template <typename R, int LOG>
constexpr int rows_per_block() {
    constexpr int nt = FftShape<LOG>::NT;
    constexpr int by_threads = 1024 / nt;
    constexpr int by_lds = static_cast<int>((70 * 1024) / (lds_group_stride(1 << LOG) * sizeof(cpx<R>)));
    constexpr int n = (1 << LOG) / 2;
    int lim = by_threads < by_lds ? by_threads : by_lds;
    lim = lim < n ? lim : n;
    int g = 1;                      // largest power of two <= lim (the last block of a
    while (2 * g <= lim) g *= 2;    // grid whose side it does not divide is partly idle)
    return g;
}

// A grid line of n points (n even, F >= 2n) sits at the centred positions
// n' mod F of an F-point transform, n' = index - n/2: n' >= 0 at positions
// [0, n/2), n' < 0 at [F - n/2, F).  In the register layout (position
// p = tid + NT i) those are slots 0..3 and 12..15 (n/2 <= F/4), so slots 4..11
// are zero padding at compile time; the grid index of position p is
// p + n/2 (slots 0..3, p < n/2) or p - F + n/2 (slots 12..15, p >= F - n/2).
// The kernels address a line through one base pointer at index n/2 with the
// offsets p or p - F, so every load and store of a thread shares one address
// register.

// Rows of the grid, G per block, at centred positions n' mod F:
// z = rho + i rho d(n1) d(n2) (the type-2 deconvolution rides in the imaginary
// part), one F-point FFT; the transform of the real part on m = 0..F/2 (I1
// half spectrum) goes to the column-major XT, that of the imaginary part on
// the Q window frequencies (the type-2 row window) to TT.  Rows at or beyond
// N (the last block of a grid whose side G does not divide) transform zeros
// and store nothing.
// EXACT: the grid side is F/2 (a power of two at kappa = 2), so every bound
// below is a compile-time constant (the general form tests each slot and row).
template <typename R, int LOG, int DIR, int G, bool EXACT>
__device__ __forceinline__ void rows_forward_body(const DevPlan& P, const R* __restrict__ rho, int row0,
                                                  cpx<R>* lds_all) {
    using Sh = FftShape<LOG>;
    constexpr int F = Sh::F;
    constexpr int HALF = F / 2;
    constexpr int NT = Sh::NT;
    constexpr int LP = lds_group_stride(F);
    const int n = EXACT ? F / 2 : P.n;
    const int g = threadIdx.x / NT;
    const int tid = threadIdx.x - g * NT;
    cpx<R>* lds = lds_all + g * LP;
    const cpx<R>* tw = static_cast<const cpx<R>*>(P.twr);
    const bool row_ok = EXACT || row0 + g < n;
    const int row = row_ok ? row0 + g : n - 1;
    const double dy = P.deconv[row];
    // grid column n1 = position + N/2 (n' >= 0) or position - F + N/2 (n' < 0):
    // one base address per array serves every slot
    const int half = EXACT ? F / 4 : (n >> 1);
    const R* src = rho + static_cast<size_t>(row) * n + half;
    const double* dx = P.deconv + half;
    cpx<R> v[16];
#pragma unroll
    for (int i = 0; i < 16; ++i) {
        const int p = tid + NT * i;
        v[i] = {R(0), R(0)};
        if (i < 4 || i >= 12) {
            const int o = (i < 4) ? p : p - F;
            const bool inside = (i < 4) ? (p < half) : (p >= F - half);
            if (row_ok && inside) {
                const R r = src[o];
                v[i] = {r, static_cast<R>(static_cast<double>(r) * dx[o] * dy)};
            }
        }
    }
    fft_reg<R, LOG, DIR>(v, lds, tw, tid);
    __syncthreads();
#pragma unroll
    for (int i = 0; i < 16; ++i) lds[lds_pad(tid + NT * i)] = v[i];
    __syncthreads();
    // outputs of the G rows, row index fastest: G-element runs of each column;
    // a compile-time number of passes with clamped indices
    cpx<R>* xt = static_cast<cpx<R>*>(P.xt);
    constexpr int ITEMS = (HALF + 1) * G;
    constexpr int PASSES = (ITEMS + NT * G - 1) / (NT * G);
#pragma unroll
    for (int k = 0; k < PASSES; ++k) {
        const int idx = threadIdx.x + k * NT * G;
        const int idc = idx < ITEMS ? idx : ITEMS - 1;
        const int gg = idc % G;
        const int m = idc / G;
        const cpx<R>* l = lds_all + gg * LP;
        const cpx<R> a = l[lds_pad(m)];
        const cpx<R> b = l[lds_pad((F - m) & (F - 1))];
        // transform of the real part: X[m] = (Z[m] + conj Z[-m]) / 2
        if (idx < ITEMS && (EXACT || row0 + gg < n))
            xt[static_cast<size_t>(m) * P.col_stride + row0 + gg] = {R(0.5) * (a.x + b.x), R(0.5) * (a.y - b.y)};
    }
    // the window columns that the nodes' taps touch
    cpx<R>* tt = static_cast<cpx<R>*>(P.tt);
    for (int idx = threadIdx.x; idx < (P.nd.col_hi - P.nd.col_lo) * G; idx += NT * G) {
        const int gg = idx % G;
        const int i = P.nd.col_lo + idx / G;
        const int lf = P.patch_lo + i;
        const cpx<R>* l = lds_all + gg * LP;
        const cpx<R> a = l[lds_pad(lf & (F - 1))];
        const cpx<R> b = l[lds_pad((-lf) & (F - 1))];
        // transform of the imaginary part: (Z[l] - conj Z[-l]) / (2i)
        if (EXACT || row0 + gg < n)
            tt[static_cast<size_t>(i) * P.col_stride + row0 + gg] = {R(0.5) * (a.y + b.y), R(-0.5) * (a.x - b.x)};
    }
}

// Two spectrum values of one column, the rows of a pair, stored and loaded as one.
template <typename R>
struct alignas(16) cpx_pair {
    cpx<R> a, b;
};

// Rows of the grid two at a time, G pairs per block: z = rho_a + i rho_b, one
// F-point FFT for both rows.  With the row spectra X_a = (Z[m] + conj Z[-m]) / 2
// and X_b = (Z[m] - conj Z[-m]) / (2i):
//   XT      X_a, X_b on m = 0..F/2 (I1 half spectrum), the pair side by side;
//   TT      the type-2 row window, the transform of rho d: the factor d(n1) is a
//           cosine series (DevPlan::delta), so along x it is the convolution
//           sum_j delta_|j| X[l - j] on the window columns in use, summed in FP64
//           by 4 lanes per value; then times d(n2) of the row.
// Against the one-row form above: half the transforms, LDS traffic and twiddles,
// and runs of 2 G rows in each spectrum column.  The long rows are bound by the
// scattered spectrum stores and loads (2048^2, timed apart: FP32 17.3 us with
// 32-byte runs, 16.1 with 64-byte ones, 10 to 12 without the stores; FP64 38.2,
// 32.5, 16 to 18), so G is chosen for 64-byte runs (launch_pairs).  The rows'
// values do not depend on G.
template <typename R, int LOG, int DIR, int G, bool EXACT>
__device__ __forceinline__ void rows_forward_pair_body(const DevPlan& P, const R* __restrict__ rho, int pair0,
                                                       cpx<R>* lds_all) {
    using Sh = FftShape<LOG>;
    constexpr int F = Sh::F;
    constexpr int HALF = F / 2;
    constexpr int NT = Sh::NT;
    constexpr int LP = lds_group_stride(F);
    constexpr int BT = NT * G;
    const int n = EXACT ? F / 2 : P.n;
    const int pairs = n >> 1;
    const int g = threadIdx.x / NT;
    const int tid = threadIdx.x - g * NT;
    cpx<R>* lds = lds_all + g * LP;
    const cpx<R>* tw = static_cast<const cpx<R>*>(P.twr);
    // pairs at or beyond N/2 (the last block) transform the last pair and store nothing
    const int pair = min(pair0 + g, pairs - 1);
    const int half = EXACT ? F / 4 : (n >> 1);
    const R* src = rho + static_cast<size_t>(2 * pair) * n + half;
    cpx<R> v[16];
#pragma unroll
    for (int i = 0; i < 16; ++i) {
        const int p = tid + NT * i;
        v[i] = {R(0), R(0)};
        if (i < 4 || i >= 12) {
            const int o = (i < 4) ? p : p - F;
            const bool inside = (i < 4) ? (p < half) : (p >= F - half);
            if (inside) v[i] = {src[o], src[n + o]};
        }
    }
    fft_reg<R, LOG, DIR>(v, lds, tw, tid);
    __syncthreads();
#pragma unroll
    for (int i = 0; i < 16; ++i) lds[lds_pad(tid + NT * i)] = v[i];
    __syncthreads();
    cpx<R>* xt = static_cast<cpx<R>*>(P.xt) + 2 * static_cast<size_t>(pair0);
    constexpr int ITEMS = (HALF + 1) * G;
    constexpr int PASSES = (ITEMS + BT - 1) / BT;
#pragma unroll
    for (int k = 0; k < PASSES; ++k) {
        const int idx = threadIdx.x + k * BT;
        const int idc = idx < ITEMS ? idx : ITEMS - 1;
        const int gg = idc % G;
        const int m = idc / G;
        const cpx<R>* l = lds_all + gg * LP;
        const cpx<R> z = l[lds_pad(m)];
        const cpx<R> zc = l[lds_pad((F - m) & (F - 1))];
        if (idx < ITEMS && (EXACT || pair0 + gg < pairs))
            *reinterpret_cast<cpx_pair<R>*>(xt + static_cast<size_t>(m) * P.col_stride + 2 * gg) = {
                {R(0.5) * (z.x + zc.x), R(0.5) * (z.y - zc.y)}, {R(0.5) * (z.y + zc.y), R(-0.5) * (z.x - zc.x)}};
    }
    cpx<R>* tt = static_cast<cpx<R>*>(P.tt) + 2 * static_cast<size_t>(pair0);
    constexpr int L = 4;
    const int part = threadIdx.x % L;
    const int B = P.pair_taps;
    const int items = (P.nd.col_hi - P.nd.col_lo) * G;
    for (int e = threadIdx.x / L; e < items; e += BT / L) {
        const int gg = e % G;
        const int i = P.nd.col_lo + e / G;
        const int lf = P.patch_lo + i;
        const cpx<R>* l = lds_all + gg * LP;
        double ax = 0, ay = 0, bx = 0, by = 0;
#pragma unroll 4
        for (int j = part - B; j <= B; j += L) {
            const double d = P.delta[j < 0 ? -j : j];
            const cpx<R> z = l[lds_pad((lf - j) & (F - 1))];
            const cpx<R> zc = l[lds_pad((j - lf) & (F - 1))];
            const double zx = z.x, zy = z.y, cx = zc.x, cy = zc.y;
            ax += d * (zx + cx);
            ay += d * (zy - cy);
            bx += d * (zy + cy);
            by += d * (cx - zx);
        }
#pragma unroll
        for (int off = 1; off < L; off <<= 1) {
            ax += __shfl_xor(ax, off, L);
            ay += __shfl_xor(ay, off, L);
            bx += __shfl_xor(bx, off, L);
            by += __shfl_xor(by, off, L);
        }
        if (part == 0 && (EXACT || pair0 + gg < pairs)) {
            const double da = 0.5 * P.deconv[2 * (pair0 + gg)], db = 0.5 * P.deconv[2 * (pair0 + gg) + 1];
            *reinterpret_cast<cpx_pair<R>*>(tt + static_cast<size_t>(i) * P.col_stride + 2 * gg) = {
                {static_cast<R>(ax * da), static_cast<R>(ay * da)}, {static_cast<R>(bx * db), static_cast<R>(by * db)}};
        }
    }
}

// ---------------------------------------------------------------------------
// cols_highfreq: FFT along y, multiplier, inverse FFT along y (in place in XT)
// ---------------------------------------------------------------------------

// Sequences per block of a register-FFT kernel: blocks of at least 256 threads.
template <int LOG>
constexpr int lines_per_block() {
    constexpr int nt = FftShape<LOG>::NT;
    return nt >= 256 ? 1 : 256 / nt;
}

template <typename R>
__device__ __forceinline__ R recip(R x) {
    if constexpr (sizeof(R) == 4) {
        const float r = __builtin_amdgcn_rcpf(x);
        return r * (2.0f - x * r);      // one Newton step: correctly rounded to within an ulp
    } else {
        // hardware estimate and two Newton steps (each doubles the correct bits):
        // within an ulp, at a third of the cost of an IEEE division
        double r = __builtin_amdgcn_rcp(x);
        r = fma(r, fma(-x, r, 1.0), r);
        return fma(r, fma(-x, r, 1.0), r);
    }
}

// The smallest positive normal number: added to a denominator that is either
// zero (where the numerator is zero too) or far above it, so the quotient is
// 0 at the origin without a comparison and unchanged elsewhere.
template <typename R>
__device__ __forceinline__ constexpr R tiny_normal() {
    if constexpr (sizeof(R) == 4) return 1.17549435e-38f;
    else return 2.2250738585072014e-308;
}

// FP32: the rotations by e^{i pi/4} inside the butterflies scale by sqrt(2) times
// the float nearest 1/sqrt(2), 1 - 1.7e-8 (no float does better), and a quarter of
// a radix-16 or radix-8 stage's terms pass one: the four transforms of a solve
// lose 1.7e-8 of the amplitude per such stage, which the multiplier gives back.
// Measured as the mean scale of a solve against float64 sums, x, y and xy, 100^2 to
// 4096^2: -1.6e-7 to +2.6e-8 with one row per transform and the tabulated quotient;
// now +0.3e-8 to +1.7e-8 below padded side 4096, +1.7e-8 to +3.6e-8 from there on.
// The whole relative L2 error is 1.0e-7 to 2.3e-7 either way.  The Coulomb kinds
// go without: their mean scale is -4e-8 to +1.4e-8 as it is, and giving them the
// same would add 3.4e-8 or 5.1e-8.  (FP64 constants lose nothing that matters.)
template <typename R, int LOG>
__device__ __forceinline__ constexpr R norm_loss() {
    constexpr int stages = FftShape<LOG>::S16 + (FftShape<LOG>::REM == 3 ? 1 : 0);
    return sizeof(R) == 4 ? R(1.7e-8) * R(stages) : R(0);
}

// Column m1 of the half spectrum (contiguous in XT, N values at centred y
// positions) is transformed along y with the zero padding implicit: in the
// register layout only slots 0..3 and 12..15 can hold grid rows (see above),
// so the other inputs are compile-time zeros and the inverse transform's
// outputs there are never formed.
// KIND selects the multiplier at compile time (separate instantiations, so that
// the DS multiplier's code is unchanged by the others):
//   0  -kx^2/|k|^2 or -ky^2/|k|^2 (P.component 0 / 1)
//   1  -kx ky/|k|^2
//   2  1/|k| with the Gaussian partition:  g1 = (1 - e^{-|k|^2/sigma^2}) / |k|
//   3  1/|k| with the erfc partition:      g1 = erf(|k|/sigma) / |k|
//   4, 5  as 0, 1 with the quotient from the tables in FP32 (plain arithmetic)
constexpr int kKindQuadratic = 0, kKindMixed = 1, kKindCoulombGauss = 2, kKindCoulombErfc = 3;
constexpr int kKindQuadraticPlain = 4, kKindMixedPlain = 5;

// erf(x)/x for x >= 0, an even entire function: the series 2/sqrt(pi) (1 - x^2/3)
// below a threshold where the next term (x^4/10) is below the precision's
// rounding, the library erf above it.
template <typename R>
__device__ __forceinline__ R erf_over_x(R x, R x2) {
    constexpr R two_over_sqrt_pi = R(1.1283791670955126);
    if constexpr (sizeof(R) == 4) {
        return x < 1e-2f ? two_over_sqrt_pi * (1.0f - x2 * (1.0f / 3.0f)) : erff(x) / x;
    } else {
        return x < 1e-5 ? two_over_sqrt_pi * (1.0 - x2 * (1.0 / 3.0)) : erf(x) / x;
    }
}

// The multiplier g1 along spectrum column m1.
// g1 = -(k_a k_b/|k|^2) (1 - e^{-|k|^2/sigma^2}) / F^2 with a = kx^2/sigma^2,
// b = ky^2/sigma^2 and 1 - e^{-(a+b)} = A + B - A B, A = 1 - e^{-a},
// B = 1 - e^{-b} (all terms >= 0); branch-free per point, g1(0) = 0.  The
// numerator is a or b, or for the mixed component (kx/sigma)(ky/sigma) with
// the signed frequency index of the point.
// The mixed numerator is odd in each frequency, and a bin on a Nyquist line
// (|index| = F/2) stands for +k and -k: it takes the mean of the multiplier
// over them, 0 (also at the corner).
template <typename R, int LOG, int KIND>
struct ColumnFactor {
    static constexpr int HALF = (1 << LOG) / 2;
    R a, A, scale, fs, fx, inv_sigma;
    bool ycomp;
    // FP32: frequency index of the column (mx2 is positive at the origin too,
    // where the numerator is 0; the mixed one is 0 on the Nyquist column), and A,
    // 1 - A = e^{-a} with the sign and the power of two 1 / F^2
    R mxn, mx2, part_a, part_e;

    __device__ __forceinline__ ColumnFactor(const DevPlan& P, int m1) {
        a = static_cast<R>(P.gx[2 * m1]);
        A = static_cast<R>(P.gx[2 * m1 + 1]);
        scale = static_cast<R>(P.inv_f2);
        ycomp = P.component == 1;
        fs = static_cast<R>(P.freq_scale);
        fx = (m1 == HALF) ? R(0) : static_cast<R>(m1) * fs;
        inv_sigma = static_cast<R>(P.inv_sigma);
        mxn = m1 == HALF ? R(0) : static_cast<R>(m1);
        mx2 = static_cast<R>(m1) * static_cast<R>(m1) + tiny_normal<R>();
        part_a = static_cast<R>(-P.gx[2 * m1 + 1] * P.inv_f2);
        part_e = static_cast<R>((P.gx[2 * m1 + 1] - 1.0) * P.inv_f2);
    }

    // at signed frequency index my along y (nyquist: my = -F/2), (b, B) its table entry
    __device__ __forceinline__ R at(R my, bool nyquist, R b, R B) const {
        if constexpr (KIND == kKindCoulombGauss) {
            // (1 - e^{-(a+b)}) / (sigma sqrt(a+b)): 0 * finite at k = 0
            const R s2 = a + b + tiny_normal<R>();
            return (A + B - A * B) * (inv_sigma * scale) / sqrt(s2);
        } else if constexpr (KIND == kKindCoulombErfc) {
            const R s2 = a + b;
            return erf_over_x<R>(sqrt(s2), s2) * (inv_sigma * scale);
        } else if constexpr (sizeof(R) == 4 && (KIND == kKindQuadratic || KIND == kKindMixed)) {
            // the quotient of the integer frequency indices (exact products up to
            // 2^24), corrected by its remainder: within an ulp; A + B - A B as
            // A + B e^{-a}, rounded once
            const R den = fma(my, my, mx2);
            R num;
            if constexpr (KIND == kKindMixed) num = nyquist ? R(0) : mxn * my;
            else num = ycomp ? my * my : mx2;
            const R r = __builtin_amdgcn_rcpf(den);
            const R q0 = num * r;
            const R q = fma(fma(-q0, den, num), r, q0);
            const R w = fma(B, part_e, part_a);
            // 0.3 (one stage) to 1.7 (three) half ulps: added before the product is rounded
            return fma(q, w, (q * norm_loss<R, LOG>()) * w);
        } else {
            R num;
            if constexpr (KIND == kKindMixed || KIND == kKindMixedPlain) num = nyquist ? R(0) : fx * (my * fs);
            else num = ycomp ? b : a;
            // den = 0 only at k = 0, where num = 0: the quotient is 0 there
            const R den = a + b + tiny_normal<R>();
            return -(num * recip(den)) * (A + B - A * B) * scale;
        }
    }
};

template <typename R, int LOG, int DIR, int G, int KIND, bool EXACT>
__device__ __forceinline__ void cols_highfreq_body(const DevPlan& P, int m1_base, cpx<R>* lds_all) {
    using Sh = FftShape<LOG>;
    constexpr int F = Sh::F;
    constexpr int HALF = F / 2;
    constexpr int NT = Sh::NT;
    const int n = EXACT ? F / 2 : P.n;
    const int g = threadIdx.x / NT;
    const int tid = threadIdx.x - g * NT;
    cpx<R>* lds = lds_all + g * lds_group_stride(F);
    const cpx<R>* tw = static_cast<const cpx<R>*>(P.twr);
    const int m1 = m1_base + g;   // 0..F/2 (+ idle lanes of the last block)
    const bool active = m1 <= HALF;
    // idle lanes load column F/2 and never store: no branch around the loads
    cpx<R>* col = static_cast<cpx<R>*>(P.xt) + static_cast<size_t>(active ? m1 : HALF) * P.col_stride;
    // rows n' >= 0 at positions [0, N/2), n' < 0 at [F - N/2, F): one base
    // address (row N/2 - position 0) serves every slot
    const int half = EXACT ? F / 4 : (n >> 1);
    const cpx<R>* base = col + half;
    cpx<R> v[16];
#pragma unroll
    for (int i = 0; i < 16; ++i) {
        const int p = tid + NT * i;
        v[i] = {R(0), R(0)};
        if (i < 4) {
            if (p < half) v[i] = base[p];
        } else if (i >= 12) {
            if (p >= F - half) v[i] = base[p - F];
        }
    }
    fft_reg<R, LOG, DIR>(v, lds, tw, tid);
    // (b, 1 - e^{-b}) of the 16 rows this thread multiplies, fetched only now:
    // held through the transform they would take 32 more registers and, in
    // FP32, cut the resident blocks per CU from four to three
    const cpx<R>* gyr = static_cast<const cpx<R>*>(P.gyr);
    cpx<R> gb[16];
#pragma unroll
    for (int i = 0; i < 16; ++i) gb[i] = gyr[tid + NT * i];
    const ColumnFactor<R, LOG, KIND> factor(P, active ? m1 : HALF);
    const R fy = static_cast<R>(tid);
#pragma unroll
    for (int i = 0; i < 16; ++i) {
        const R my = fy + static_cast<R>(NT * i - (i < 8 ? 0 : F));
        v[i] = cscale(v[i], factor.at(my, i == 8 && tid == 0, gb[i].x, gb[i].y));
    }
    fft_reg<R, LOG, -DIR>(v, lds, tw, tid);
    if (active) {
        cpx<R>* out = col + half;
#pragma unroll
        for (int i = 0; i < 16; ++i) {
            const int p = tid + NT * i;
            if (i < 4) {
                if (p < half) out[p] = v[i];
            } else if (i >= 12) {
                if (p >= F - half) out[p - F] = v[i];
            }
        }
    }
}

// The same column in two transforms of F/2 points, for F = 8192.  The data has at
// most F/2 points, so its even frequencies are the F/2-point transform of x and the
// odd ones that of x e^{DIR 2 pi i n / F}, without sums between the two; each half
// goes through its own multiplier and inverse transform, and the column is the even
// result plus e^{-DIR 2 pi i n / F} times the odd one.  8192 = 16^3 2 takes three
// exchanges and a radix-2 stage per transform, 4096 = 16^3 two: a third less through
// LDS, and a quarter of the LDS per wave.  The halves run one after the other (x is
// read again), so one half's 16 points and the even result are held at a time.
// The e^{-2 pi i k / F} are the last stage's twiddles of the F-point table, whose
// earlier stages are the F/2-point table.  The column launch of a solve, before and
// after: 3000^2 FP32 183 and 129 us, 4096^2 FP32 195 and 134, FP64 261 and 228, FP64
// Coulomb at 3000^2 369 and 318.  (Both halves held at once, or their table reads
// hoisted together, take 170 to 250 registers and cost more than they save.)
template <typename R, int LOG, int DIR, int KIND, bool EXACT>
__device__ __forceinline__ void cols_highfreq_halves_body(const DevPlan& P, int m1, cpx<R>* lds) {
    using Sh = FftShape<LOG>;
    using Hs = FftShape<LOG - 1>;
    static_assert(Sh::REM == 1 && Sh::tw_offset(Sh::NSTAGE - 1) == Hs::tw_size(), "shared tables");
    constexpr int F = Sh::F;
    constexpr int H = F / 2;
    constexpr int NT = Hs::NT;
    int tid = threadIdx.x;
    const cpx<R>* tw = static_cast<const cpx<R>*>(P.twr);
    const cpx<R>* turn = tw + Hs::tw_size();   // e^{-2 pi i k / F}, k = 0 .. H - 1
    const cpx<R>* gyr = static_cast<const cpx<R>*>(P.gyr);
    const int half = EXACT ? F / 4 : (P.n >> 1);
    cpx<R>* base = static_cast<cpx<R>*>(P.xt) + static_cast<size_t>(m1) * P.col_stride + half;
    const ColumnFactor<R, LOG, KIND> factor(P, m1);
    // slot i holds row n = p below F/4, n = p - H above: e^{.. n / F} = -e^{.. p / F} there
    auto holds = [&](int i) { return EXACT || (i < 8 ? tid + NT * i < half : tid + NT * i >= H - half); };
    cpx<R> even[16];
#pragma unroll 1
    for (int odd = 0; odd < 2; ++odd) {
        // the thread's number is made opaque where a part begins: the tables are read
        // there again, not held in registers through the parts before
        asm volatile("" : "+v"(tid));
        cpx<R> v[16];
#pragma unroll
        for (int i = 0; i < 16; ++i) {
            v[i] = {R(0), R(0)};
            if (holds(i)) v[i] = base[tid + NT * i - (i < 8 ? 0 : H)];
        }
        if (odd) {
#pragma unroll
            for (int i = 0; i < 16; ++i) {
                const cpx<R> t = turn[tid + NT * i];
                v[i] = tw_mul<R, DIR>(v[i], i < 8 ? t : cpx<R>{-t.x, -t.y});
            }
        }
        fft_reg<R, LOG - 1, DIR>(v, lds, tw, tid);
        cpx<R> gb[16];
#pragma unroll
        for (int i = 0; i < 16; ++i) gb[i] = gyr[2 * (tid + NT * i) + odd];
#pragma unroll
        for (int i = 0; i < 16; ++i) {
            const R my = static_cast<R>(2 * tid) + static_cast<R>(2 * NT * i + odd - (i < 8 ? 0 : F));
            v[i] = cscale(v[i], factor.at(my, !odd && i == 8 && tid == 0, gb[i].x, gb[i].y));
        }
        asm volatile("" : "+v"(tid));
        fft_reg<R, LOG - 1, -DIR>(v, lds, tw, tid);
        asm volatile("" : "+v"(tid));
        if (!odd) {
#pragma unroll
            for (int i = 0; i < 16; ++i) even[i] = v[i];
        } else {
#pragma unroll
            for (int i = 0; i < 16; ++i) {
                const cpx<R> t = turn[tid + NT * i];
                const cpx<R> o = cadd(even[i], tw_mul<R, -DIR>(v[i], i < 8 ? t : cpx<R>{-t.x, -t.y}));
                if (holds(i)) base[tid + NT * i - (i < 8 ? 0 : H)] = o;
            }
        }
    }
}

// ---------------------------------------------------------------------------
// cols_type2: FFT along y of the type-2 row window, keep the Q window rows
// ---------------------------------------------------------------------------
template <typename R, int LOG, int DIR, int G, bool EXACT>
__device__ __forceinline__ void cols_type2_body(const DevPlan& P, int i1_base, cpx<R>* lds_all) {
    using Sh = FftShape<LOG>;
    constexpr int F = Sh::F;
    constexpr int NT = Sh::NT;
    const int g = threadIdx.x / NT;
    const int tid = threadIdx.x - g * NT;
    cpx<R>* lds = lds_all + g * lds_group_stride(F);
    const cpx<R>* tw = static_cast<const cpx<R>*>(P.twr);
    const int q = P.patch;
    const int i1 = i1_base + g;
    const bool active = i1 < P.nd.col_hi;
    const cpx<R>* col =
        static_cast<const cpx<R>*>(P.tt) + static_cast<size_t>(active ? i1 : P.nd.col_lo) * P.col_stride;
    const cpx<R> zero = {R(0), R(0)};
    const int half = EXACT ? F / 4 : (P.n >> 1);
    const cpx<R>* base = col + half;
    cpx<R> v[16];
#pragma unroll
    for (int i = 0; i < 16; ++i) {
        const int p = tid + NT * i;
        v[i] = zero;
        if (i < 4) {
            if (active && p < half) v[i] = base[p];
        } else if (i >= 12) {
            if (active && p >= F - half) v[i] = base[p - F];
        }
    }
    fft_reg<R, LOG, DIR>(v, lds, tw, tid);
    cpx<R>* win = static_cast<cpx<R>*>(P.win);
    if (active) {
#pragma unroll
        for (int i = 0; i < 16; ++i) {
            const int i2 = posmod_dev(tid + NT * i - P.patch_lo, F);   // window row of this position
            if (i2 < q) win[static_cast<size_t>(i2) * q + i1] = v[i];
        }
    }
}

// ---------------------------------------------------------------------------
// nodes: interpolation, polar multiplier and spreading of one subproblem
// ---------------------------------------------------------------------------
// A subproblem is a run of at most 64 nodes whose first kernel taps lie in one
// bin of bin x bin window cells, so all their taps fall in the E x E tile
// (E = bin + w - 1) at the bin's corner.  The block stages that tile of the
// type-2 window, the nodes' tap values and first-tap offsets in LDS, then
//   interp:  c_j = sum_{t2} psi_y[t2] sum_{t1} tile[oy+t2][ox+t1] psi_x[t1]
//            (16 lanes per node, lane t2 sums its tap row, then a fixed
//            rotate-and-add tree across the 16 lanes)          [eq. (16), (12)]
//   a_j = q_j h^2 c_j                                          [eq. (12)]
//   spread:  T[cb][ca] = sum_j a_j psi_x[ca-ox_j] psi_y[cb-oy_j] (one thread per
//            tile cell, nodes in order, compensated in FP32)   [eq. (15)]
// and writes its whole tile T to its own slot: no atomics.  The tiles are
// summed onto the window by cols_type1 through a precomputed index list.
// MODE 0: all three steps; MODE 1: interp only, out[j] = h^2 c_j (type-2 stage);
// MODE 2: spread only, of coef (type-1 stage).  NTH threads per block: the
// order of every sum is fixed by kLanesPerNode and kSpreadParts alone, so
// blocks of any size give the same bits.
constexpr int kNodeThreads = 256;         // batched blocks
// one plan's subproblems in their own launch: 512 threads, so a block's tile
// loads, taps and spreading run in fewer rounds (graph replay on MI355X: the
// FP64 node stage 10.7 -> 9.3 us at 1024^2, the 1024^2 FP64 solve 64.2 -> 61.9 us)
constexpr int kNodeThreadsSingle = 512;
constexpr int kLanesPerNode = 16;
constexpr int kSpreadParts = 2;
constexpr int kTileMax = kMaxTile;

// WMAX: the widest kernel the block serves (kMaxEsWidth, or kMaxKernelWidth for
// the Gaussian), which sizes the tap store
template <typename R, int WMAX>
struct NodeLds {
    cpx<R> tile[kTileMax * kTileMax];
    R taps[kMaxNodesPerSub * 2 * WMAX];   // per node: w x-taps, then w y-taps
    int2 off[kMaxNodesPerSub];            // first-tap offset (x, y) in the tile
    double qh[kMaxNodesPerSub];   // q_j h^2
    cpx<R> val[kMaxNodesPerSub];
};

// Sum over the 16 lanes of each row of the wave (lanes 16r .. 16r + 15), in a
// fixed order: four rotate-and-add steps (rotations by 8, 4, 2, 1 lanes within
// the row, DPP row_ror on the vector ALU, no LDS round trip).  Every lane ends
// with the row's sum; lane 16r's association order is the same in every call.
template <int CTRL>
__device__ __forceinline__ float row_rotate(float v) {
    return __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, v), CTRL, 0xf, 0xf, false));
}
template <int CTRL>
__device__ __forceinline__ double row_rotate(double v) {
    const long long b = __builtin_bit_cast(long long, v);
    const int lo = __builtin_amdgcn_update_dpp(0, static_cast<int>(b & 0xffffffffll), CTRL, 0xf, 0xf, false);
    const int hi = __builtin_amdgcn_update_dpp(0, static_cast<int>(b >> 32), CTRL, 0xf, 0xf, false);
    return __builtin_bit_cast(double, (static_cast<long long>(hi) << 32) | static_cast<unsigned>(lo));
}
template <typename R>
__device__ __forceinline__ R row16_sum(R v) {
    constexpr int kRowRor = 0x120;   // DPP row_ror:n is kRowRor + n
    v += row_rotate<kRowRor + 8>(v);
    v += row_rotate<kRowRor + 4>(v);
    v += row_rotate<kRowRor + 2>(v);
    v += row_rotate<kRowRor + 1>(v);
    return v;
}

template <typename R>
__device__ __forceinline__ void kahan_add(R& s, R& c, R v) {
    if constexpr (sizeof(R) == 4) {
        const R y = v - c;
        const R t = s + y;
        c = (t - s) - y;
        s = t;
    } else {
        s += v;
    }
}

// x / d for 0 <= x < 1024 and 1 <= d <= 31 as (x * ceil(2^16 / d)) >> 16: the
// rounded-up reciprocal adds less than x / 2^16 < 1/64 to x / d, less than
// the gap 1/d between x / d and the next integer
__device__ __forceinline__ unsigned small_div_magic(int d) {
    return (65536u + static_cast<unsigned>(d) - 1u) / static_cast<unsigned>(d);
}
__device__ __forceinline__ int small_div(int x, unsigned magic) {
    return static_cast<int>((static_cast<unsigned>(x) * magic) >> 16);
}

// W: the kernel width when it is fixed at compile time (0: read from the plan).
// A fixed width lets the interpolation's tap loop unroll, so the LDS reads of a
// node's whole tap row issue together; the sums keep their order, so the bits
// are the same.
template <typename R, int MODE, int NTH, int WMAX, int W = 0>
__device__ __forceinline__ void nodes_body(const DevPlan& P, int sidx, const cpx<R>* __restrict__ coef,
                                           cpx<R>* __restrict__ out, NodeLds<R, WMAX>& s) {
    static_assert(W >= 0 && W <= WMAX, "a fixed width within the tap store");
    static_assert(NTH % kLanesPerNode == 0 && NTH % kSpreadParts == 0, "whole node and cell groups");
    static_assert(NTH >= kMaxNodesPerSub, "one thread per node for the node scalars");
    static_assert(kTileMax * kTileMax < 1024 && kTileMax <= 31 && WMAX * WMAX <= 1024 && WMAX <= kMaxKernelWidth,
                  "small_div covers the tile and tap indices");
    constexpr int TPT = (kMaxNodesPerSub * 2 * WMAX + NTH - 1) / NTH;   // taps per thread
    constexpr int CPT = (kTileMax * kTileMax + NTH - 1) / NTH;                     // tile cells per thread
    const int* sub = P.nd.sub + 4 * sidx;
    const int bx = sub[0], by = sub[1], first = sub[2], count = sub[3];
    const int w = W > 0 ? W : P.width;
    const int E = P.tile, q = P.patch, bin = P.bin;
    const int w2 = 2 * w;
    const int x0 = bx * bin, y0 = by * bin;   // tile corner in window cells
    const unsigned magic_e = small_div_magic(E);
    // every global load of the block is issued before the first LDS store, so
    // their latencies overlap: the subproblem's taps (contiguous, w2 per node),
    // the per-node scalars, the type-2 window tile
    const R* taps = static_cast<const R*>(P.nd.taps) + static_cast<size_t>(first) * w2;
    const int n_taps = count * w2;
    R tv[TPT];
#pragma unroll
    for (int k = 0; k < TPT; ++k) {
        const int e = threadIdx.x + k * NTH;
        tv[k] = e < n_taps ? taps[e] : R(0);
    }
    const int jn = threadIdx.x;
    const bool has_node = jn < count;
    int cx = 0, cy = 0;
    double qv = 0.0;
    cpx<R> cv = {R(0), R(0)};
    if (has_node) {
        cx = P.nd.cell[2 * (first + jn)];
        cy = P.nd.cell[2 * (first + jn) + 1];
        if constexpr (MODE == 0) qv = P.nd.q[first + jn];
        if constexpr (MODE == 2) cv = coef[first + jn];
    }
    cpx<R> tl[CPT];
    if constexpr (MODE != 2) {
        // the window side is a power of two and tiles only wrap when the window
        // is the whole periodic fine grid
        const bool whole = (q == P.n_fine);
        const cpx<R>* win = static_cast<const cpx<R>*>(P.win);
#pragma unroll
        for (int k = 0; k < CPT; ++k) {
            const int c = threadIdx.x + k * NTH;
            const int cb = small_div(c, magic_e), ca = c - cb * E;
            int wx = x0 + ca, wy = y0 + cb;
            bool inside = c < E * E;
            if (whole) {
                wx &= q - 1;
                wy &= q - 1;
            } else {
                inside = inside && wx < q && wy < q;
            }
            tl[k] = inside ? win[static_cast<size_t>(wy) * q + wx] : cpx<R>{R(0), R(0)};
        }
    }
#pragma unroll
    for (int k = 0; k < TPT; ++k) {
        const int e = threadIdx.x + k * NTH;
        if (e < n_taps) s.taps[e] = tv[k];
    }
    if (has_node) {
        s.off[jn] = make_int2(cx - x0, cy - y0);
        if constexpr (MODE == 0) s.qh[jn] = qv * P.h2;
        if constexpr (MODE == 2) s.val[jn] = cv;
    }
    // the staged tile's rows are ES = E | 1 entries apart: an odd stride puts
    // the 16 lanes of a node, one tap row each, in distinct LDS banks
    const int ES = E | 1;
    if constexpr (MODE != 2) {
#pragma unroll
        for (int k = 0; k < CPT; ++k) {
            const int c = threadIdx.x + k * NTH;
            const int cb = small_div(c, magic_e), ca = c - cb * E;
            if (c < E * E) s.tile[cb * ES + ca] = tl[k];
        }
    }
    __syncthreads();
    if constexpr (MODE != 2) {
        static_assert(kLanesPerNode == 16, "one DPP row per node");
        const int lane = threadIdx.x % kLanesPerNode;
        for (int jj0 = 0; jj0 < count; jj0 += NTH / kLanesPerNode) {
            const int jj = jj0 + threadIdx.x / kLanesPerNode;
            cpx<R> acc = {R(0), R(0)};
            if (jj < count) {
                const int2 o = s.off[jj];
                const R* tj = s.taps + jj * w2;
                // lane t2 (and t2 + 16 for the widest Gaussian kernels) sums one
                // tap row: psi_y[t2] sum_t1 tile[oy+t2][ox+t1] psi_x[t1], four
                // taps at a time with clamped indices and zero weights past w,
                // so the loads of a chunk issue together without branches
                for (int t2 = lane; t2 < w; t2 += kLanesPerNode) {
                    const cpx<R>* trow = s.tile + (o.y + t2) * ES + o.x;
                    cpx<R> row = {R(0), R(0)};
                    auto chunk = [&](int t0) {
                        R k[4];
                        cpx<R> b[4];
#pragma unroll
                        for (int u = 0; u < 4; ++u) {
                            const int t1 = min(t0 + u, w - 1);
                            const R kv = tj[t1];
                            k[u] = (t0 + u < w) ? kv : R(0);
                            b[u] = trow[t1];
                        }
#pragma unroll
                        for (int u = 0; u < 4; ++u) {
                            row.x += b[u].x * k[u];
                            row.y += b[u].y * k[u];
                        }
                    };
                    if constexpr (W > 0) {
#pragma unroll
                        for (int t0 = 0; t0 < W; t0 += 4) chunk(t0);
                    } else {
                        for (int t0 = 0; t0 < w; t0 += 4) chunk(t0);
                    }
                    const R ky = tj[w + t2];
                    acc.x += row.x * ky;
                    acc.y += row.y * ky;
                }
            }
            acc.x = row16_sum(acc.x);
            acc.y = row16_sum(acc.y);
            if (jj < count && lane == 0) {
                const int j = first + jj;
                if constexpr (MODE == 1) {
                    out[j] = {static_cast<R>(acc.x * P.h2), static_cast<R>(acc.y * P.h2)};
                } else {
                    const double scale = s.qh[jj];
                    s.val[jj] = {static_cast<R>(acc.x * scale), static_cast<R>(acc.y * scale)};
                }
            }
        }
    }
    if constexpr (MODE == 1) return;
    if constexpr (MODE == 0) __syncthreads();
    // kSpreadParts threads per tile cell, each summing one run of the nodes (in
    // order), then a fixed shuffle tree; the node loop is unrolled and
    // branch-free so the LDS reads of several nodes are in flight together
    cpx<R>* tile_out = static_cast<cpx<R>*>(P.tiles) + static_cast<size_t>(sidx) * E * E;
    constexpr int U = 8;
    const int part = threadIdx.x % kSpreadParts;
    const int run = (count + kSpreadParts - 1) / kSpreadParts;
    const int j_lo = min(count, part * run);
    const int j_hi = min(count, j_lo + run);
    for (int c = threadIdx.x / kSpreadParts; c < E * E; c += NTH / kSpreadParts) {
        const int cb = small_div(c, magic_e), ca = c - cb * E;
        R sx = 0, sy = 0, kx = 0, ky = 0;
        for (int j0 = j_lo; j0 < j_hi; j0 += U) {
            R kk[U];
            cpx<R> vv[U];
#pragma unroll
            for (int u = 0; u < U; ++u) {
                const int jj = j0 + u;
                const bool valid = jj < j_hi;
                const int jc = valid ? jj : j_lo;
                const int2 o = s.off[jc];
                const int t1 = ca - o.x;
                const int t2 = cb - o.y;
                const bool in = valid && static_cast<unsigned>(t1) < static_cast<unsigned>(w) &&
                                static_cast<unsigned>(t2) < static_cast<unsigned>(w);
                const R* tj = s.taps + jc * w2;
                const R k = tj[in ? t1 : 0] * tj[w + (in ? t2 : 0)];
                kk[u] = in ? k : R(0);
                vv[u] = s.val[jc];
            }
#pragma unroll
            for (int u = 0; u < U; ++u) {
                kahan_add(sx, kx, vv[u].x * kk[u]);
                kahan_add(sy, ky, vv[u].y * kk[u]);
            }
        }
        R vx = sx - kx, vy = sy - ky;
#pragma unroll
        for (int off = kSpreadParts / 2; off > 0; off >>= 1) {
            vx += __shfl_xor(vx, off, kSpreadParts);
            vy += __shfl_xor(vy, off, kSpreadParts);
        }
        if (part == 0) tile_out[c] = {vx, vy};
    }
}

// The node stage of a solve on matrix instructions (grouped node sets: tiles of
// at most 16 x 16 window cells).  With a group's 16 nodes as one dimension, both
// steps are products of 16 x 16 matrices, K = 16, in v_mfma_f64_16x16x4:
//   interp:  D[cb][j] = sum_ca tile[cb][ca] X[ca][j],  c_j = sum_cb Y[j][cb] D[cb][j]
//   spread:  T[cb][ca] += sum_j (Y[j][cb] a_j) X[j][ca],  a_j = q_j h^2 c_j
// where X and Y are the nodes' taps, zero outside the kernel.  A wave takes one
// group at a time: operands come straight from global memory in the lane layout of
// the instruction (lane l: row or column l % 16, k = l / 16 + 4 kk; the result's
// register i is row l / 16 + 4 i), so the only barrier is before the four waves'
// tiles are summed.  Both precisions accumulate in FP64 (same rate as FP32 on this
// path, and no compensation is needed); the tile is rounded to the data precision
// when it is stored.
// The general kernel above is bound by its LDS reads (four per node and tile
// cell); this one by the latency of two dependent global loads, 16 matrix
// instructions and the store: 8.9 -> 4.8 us in FP64 and 6.7 -> 4.7 us in FP32 on
// 64 x 128 nodes (91 blocks).  A wave's second group would start its loads after
// the first one's result (about 2 us each: 128 nodes per subproblem 7 us, 256
// 10.6 us, against 1 us less in the tile sums), so 64 nodes fill a block.
constexpr int kNodeWaves = 4;

struct NodeGroupLds {
    double part[kNodeWaves][2][kNodeGroup * kNodeGroup];   // each wave's tile, re and im
};

template <typename R>
__device__ __forceinline__ void nodes_group_body(const DevPlan& P, int sidx, NodeGroupLds& s) {
    typedef double d4 __attribute__((ext_vector_type(4)));
    constexpr int T = kNodeGroup;
    static_assert(T == 16, "one 16 x 16 x 4 matrix instruction per step");
    const int wave = threadIdx.x >> 6;
    const int lane = threadIdx.x & 63;
    const int lo = lane & 15, hi = lane >> 4;
    const int* sub = P.nd.sub + 4 * sidx;
    const int bx = sub[0], by = sub[1], first = sub[2], count = sub[3];
    const int groups = (count + T - 1) / T;
    const int q = P.patch;
    const bool whole = (q == P.n_fine);
    const int x0 = bx * P.bin, y0 = by * P.bin;
    d4 t_re = {0, 0, 0, 0}, t_im = {0, 0, 0, 0};
    for (int g = wave; g < groups; g += kNodeWaves) {
        const size_t base = static_cast<size_t>(first) + g * T;
        const R* tp = static_cast<const R*>(P.nd.taps) + base * 2 * T;
        R xi[4], yi[4], xs[4], ys[4];
        cpx<R> tl[4];
        const cpx<R>* win = static_cast<const cpx<R>*>(P.win);
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            const int kk = hi + 4 * k;
            xi[k] = tp[lo * 2 * T + kk];          // X[ca = kk][j = lo]
            yi[k] = tp[lo * 2 * T + T + kk];      // Y[j = lo][cb = kk]
            xs[k] = tp[kk * 2 * T + lo];          // X[j = kk][ca = lo]
            ys[k] = tp[kk * 2 * T + T + lo];      // Y[j = kk][cb = lo]
            // tile[cb = lo][ca = kk]: zero beyond the window columns in use (the
            // others are not written) and its last row
            int wx = x0 + kk, wy = y0 + lo;
            bool inside = true;
            if (whole) {
                wx &= q - 1;
                wy &= q - 1;
            } else {
                inside = wx < P.nd.col_hi && wy < q;
            }
            tl[k] = inside ? win[static_cast<size_t>(wy) * q + wx] : cpx<R>{R(0), R(0)};
        }
        const double qh = P.nd.q[base + lo] * P.h2;
        d4 d_re = {0, 0, 0, 0}, d_im = {0, 0, 0, 0};
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            d_re = __builtin_amdgcn_mfma_f64_16x16x4f64(tl[k].x, xi[k], d_re, 0, 0, 0);
            d_im = __builtin_amdgcn_mfma_f64_16x16x4f64(tl[k].y, xi[k], d_im, 0, 0, 0);
        }
        double c_re = 0.0, c_im = 0.0;
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            c_re += static_cast<double>(yi[i]) * d_re[i];
            c_im += static_cast<double>(yi[i]) * d_im[i];
        }
        c_re += __shfl_xor(c_re, 16);
        c_im += __shfl_xor(c_im, 16);
        c_re += __shfl_xor(c_re, 32);
        c_im += __shfl_xor(c_im, 32);
        const double a_re = c_re * qh, a_im = c_im * qh;   // node lo, in every quarter of the wave
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            const double ar = __shfl(a_re, hi + 4 * k), ai = __shfl(a_im, hi + 4 * k);
            const double y = ys[k];
            t_re = __builtin_amdgcn_mfma_f64_16x16x4f64(y * ar, xs[k], t_re, 0, 0, 0);
            t_im = __builtin_amdgcn_mfma_f64_16x16x4f64(y * ai, xs[k], t_im, 0, 0, 0);
        }
    }
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        s.part[wave][0][lane + 64 * i] = t_re[i];     // cell (cb = hi + 4 i) * 16 + (ca = lo)
        s.part[wave][1][lane + 64 * i] = t_im[i];
    }
    __syncthreads();
    static_assert(kNodeWaves * 64 == T * T, "one thread per tile cell");
    const int c = threadIdx.x;
    double v_re = s.part[0][0][c], v_im = s.part[0][1][c];
#pragma unroll
    for (int wv = 1; wv < kNodeWaves; ++wv) {
        v_re += s.part[wv][0][c];
        v_im += s.part[wv][1][c];
    }
    // the E x E cells the taps reach, as the general kernel stores them: 16 x 16 ones
    // would outgrow the workspace the general kernel needs
    const int E = P.tile, cb = c / T, ca = c % T;
    if (cb < E && ca < E)
        static_cast<cpx<R>*>(P.tiles)[static_cast<size_t>(sidx) * E * E + cb * E + ca] = {static_cast<R>(v_re),
                                                                                         static_cast<R>(v_im)};
}

// ---------------------------------------------------------------------------
// cols_type1: sum the spread tiles onto one window column, FFT along y (only
// the Q window inputs are non-zero), keep the N centred rows, times d(n2)
// ---------------------------------------------------------------------------
// A block transforms COLS window columns (COLS divides G).  Window cell
// (i1, i2) is the sum of the tile entries listed for it, in list order: 4
// lanes split the list, then a fixed shuffle tree; all threads of the block
// share the cells of its columns, so with COLS = 1 the length of the lists
// (set by the node count, not by N) is spread over a whole block at every
// grid size.  Column c is staged in group c's buffer; group g transforms
// column g % COLS (with COLS < G the other groups repeat a transform, which the
// block's barriers need anyway) and groups g < COLS store.
template <typename R, int LOG, int DIR, int G, int COLS, bool EXACT>
__device__ __forceinline__ void cols_type1_body(const DevPlan& P, int i1_base, cpx<R>* lds_all) {
    using Sh = FftShape<LOG>;
    constexpr int F = Sh::F;
    constexpr int NT = Sh::NT;
    constexpr int BT = NT * G;
    constexpr int L = 4;
    constexpr int LP = lds_group_stride(F);
    static_assert(COLS >= 1 && G % COLS == 0, "whole rounds of the groups");
    static_assert(BT % L == 0, "the block splits into whole lane groups");
    const int g = threadIdx.x / NT;
    const int tid = threadIdx.x - g * NT;
    cpx<R>* lds = lds_all + g * LP;
    const cpx<R>* tw = static_cast<const cpx<R>*>(P.twr);
    const int q = P.patch;
    // reduced window columns, staged at the start of their groups' FFT buffers
    // (q <= F entries); the FFT's first barrier orders the groups' reads of
    // them before its writes
    const cpx<R>* tiles = static_cast<const cpx<R>*>(P.tiles);
    const int lane = threadIdx.x % L;
    for (int e = threadIdx.x / L; e < COLS * q; e += BT / L) {
        const int c = e / q;
        const int i2 = e - c * q;
        const int i1 = i1_base + c;
        const int cell = (i1 < P.nd.col_hi ? i1 : P.nd.col_lo) * q + i2;
        const int k0 = P.nd.contrib_start[cell], k1 = P.nd.contrib_start[cell + 1];
        R sx = 0, sy = 0, kx = 0, ky = 0;
        // batches of U entries per lane: all index loads, then all value loads,
        // then the sums in list order
        constexpr int U = 8;
        for (int base = k0 + lane; base < k1; base += L * U) {
            int idx[U];
#pragma unroll
            for (int u = 0; u < U; ++u) idx[u] = (base + u * L < k1) ? P.nd.contrib[base + u * L] : -1;
            cpx<R> t[U];
#pragma unroll
            for (int u = 0; u < U; ++u) t[u] = (idx[u] >= 0) ? tiles[idx[u]] : cpx<R>{R(0), R(0)};
#pragma unroll
            for (int u = 0; u < U; ++u) {
                kahan_add(sx, kx, t[u].x);
                kahan_add(sy, ky, t[u].y);
            }
        }
        R vx = sx - kx, vy = sy - ky;
#pragma unroll
        for (int off = L / 2; off > 0; off >>= 1) {
            vx += __shfl_xor(vx, off, L);
            vy += __shfl_xor(vy, off, L);
        }
        if (lane == 0) lds_all[c * LP + i2] = {vx, vy};
    }
    // the deconvolution factors of the stored rows, fetched before the
    // transform (slots outside the crop read the factor of row N/2)
    const int half = EXACT ? F / 4 : (P.n >> 1);
    const double* dy = P.deconv + half;
    double dpre[8];
#pragma unroll
    for (int i = 0; i < 16; ++i) {
        if (i < 4 || i >= 12) {
            const int p = tid + NT * i;
            const int o = (i < 4) ? p : p - F;
            const bool inside = (i < 4) ? (p < half) : (p >= F - half);
            dpre[i < 4 ? i : i - 8] = dy[inside ? o : 0];
        }
    }
    __syncthreads();
    const int c = g % COLS;
    const int i1 = i1_base + c;
    const bool active = i1 < P.nd.col_hi;
    const cpx<R>* staged = lds_all + c * LP;
    cpx<R> v[16];
#pragma unroll
    for (int i = 0; i < 16; ++i) {
        const int i2 = posmod_dev(tid + NT * i - P.patch_lo, F);
        v[i] = (active && i2 < q) ? staged[i2] : cpx<R>{R(0), R(0)};
    }
    fft_reg<R, LOG, DIR>(v, lds, tw, tid);
    if (active && g < COLS) {
        cpx<R>* u = static_cast<cpx<R>*>(P.u) + static_cast<size_t>(half) * q + i1;
#pragma unroll
        for (int i = 0; i < 16; ++i) {
            const int p = tid + NT * i;
            if (i < 4 || i >= 12) {
                const int o = (i < 4) ? p : p - F;     // grid row n2 = o + N/2
                const bool inside = (i < 4) ? (p < half) : (p >= F - half);
                if (inside) {
                    const double d = dpre[i < 4 ? i : i - 8];
                    u[static_cast<ptrdiff_t>(o) * q] = {static_cast<R>(v[i].x * d), static_cast<R>(v[i].y * d)};
                }
            }
        }
    }
}

// ---------------------------------------------------------------------------
// rows_inverse: Phi row = Re IFFT(S1 + i H) + Im IFFT(S1 + i H) d(n1)
// ---------------------------------------------------------------------------

// For each of the block's G rows the full F-point row spectrum is assembled in
// LDS: the Hermitian extension of the I1 half spectrum (column m of XT, conj at
// F - m) plus i times the Hermitian part H[l] = (U[l] + conj U[-l]) / 2 of the
// type-1 row on the window frequencies.  One inverse FFT then gives I1 in the
// real part and Re(type-1 field) / d(n1) in the imaginary part.  Rows at or
// beyond N (the last block of a grid whose side G does not divide) transform
// zeros and store nothing.
template <typename R, int LOG, int DIR, bool USE_I1, bool USE_I2, int G, bool EXACT>
__device__ __forceinline__ void rows_inverse_body(const DevPlan& P, R* __restrict__ out, int row0,
                                                  cpx<R>* lds_all) {
    using Sh = FftShape<LOG>;
    constexpr int F = Sh::F;
    constexpr int HALF = F / 2;
    constexpr int NT = Sh::NT;
    constexpr int LP = lds_group_stride(F);
    const int n = EXACT ? F / 2 : P.n;
    const int g = threadIdx.x / NT;
    const int tid = threadIdx.x - g * NT;
    cpx<R>* lds = lds_all + g * LP;
    const cpx<R>* tw = static_cast<const cpx<R>*>(P.twr);
    const cpx<R>* xt = static_cast<const cpx<R>*>(P.xt);
    const cpx<R>* u = static_cast<const cpx<R>*>(P.u);
    const int q = P.patch, lo = P.patch_lo, c0 = P.nd.col_lo, c1 = P.nd.col_hi;
    // (F/2+1) G entries (column m, row gg), row index fastest; every load is
    // issued unconditionally (clamped index) so that all of them are in flight
    // at once
    constexpr int ITEMS = (HALF + 1) * G;
    constexpr int PASSES = (ITEMS + NT * G - 1) / (NT * G);
#pragma unroll
    for (int k = 0; k < PASSES; ++k) {
        const int idx = threadIdx.x + k * NT * G;
        const int idc = idx < ITEMS ? idx : ITEMS - 1;
        const int gg = idc % G;
        const int m = idc / G;
        const int r = (EXACT || row0 + gg < n) ? row0 + gg : n - 1;   // rows past N read row N - 1, never stored
        cpx<R> x = {R(0), R(0)};
        if constexpr (USE_I1) x = xt[static_cast<size_t>(m) * P.col_stride + r];
        cpx<R> hh = {R(0), R(0)};
        // only frequencies |m| <= Q/2 meet the window (m - lo or -m - lo in
        // [0, Q) mod F); pass k covers m in [k NT, (k+1) NT), so the later
        // passes skip the window loads altogether (a uniform branch)
        if (USE_I2 && k * NT <= (q >> 1)) {
            const int ia = posmod_dev(m - lo, F);
            const int ib = posmod_dev(-m - lo, F);
            const cpx<R>* urow = u + static_cast<size_t>(r) * q;
            // columns outside [c0, c1) hold no taps and are not written
            const bool in_a = ia >= c0 && ia < c1, in_b = ib >= c0 && ib < c1;
            const cpx<R> ua0 = urow[in_a ? ia : c0];
            const cpx<R> ub0 = urow[in_b ? ib : c0];
            const cpx<R> ua = in_a ? ua0 : cpx<R>{R(0), R(0)};
            const cpx<R> ub = in_b ? ub0 : cpx<R>{R(0), R(0)};
            hh = {R(0.5) * (ua.x + ub.x), R(0.5) * (ua.y - ub.y)};
        }
        // position m: X + i H;  position F - m: conj X + i conj H (the clamped
        // duplicate of the last entry rewrites the same values)
        cpx<R>* l = lds_all + gg * LP;
        l[lds_pad(m)] = {x.x - hh.y, x.y + hh.x};
        if (m > 0 && m < HALF) l[lds_pad(F - m)] = {x.x + hh.y, -x.y + hh.x};
    }
    // the deconvolution factors of the stored slots, fetched before the
    // transform so that their latency overlaps it (slots outside the crop read
    // the factor of row N/2)
    const int half = EXACT ? F / 4 : (n >> 1);
    const double* dx = P.deconv + half;
    double dpre[8];
#pragma unroll
    for (int i = 0; i < 16; ++i) {
        if (i < 4 || i >= 12) {
            const int p = tid + NT * i;
            const int o = (i < 4) ? p : p - F;
            const bool inside = (i < 4) ? (p < half) : (p >= F - half);
            dpre[i < 4 ? i : i - 8] = dx[inside ? o : 0];
        }
    }
    __syncthreads();
    cpx<R> v[16];
#pragma unroll
    for (int i = 0; i < 16; ++i) v[i] = lds[lds_pad(tid + NT * i)];
    fft_reg<R, LOG, DIR>(v, lds, tw, tid);
    if (EXACT || row0 + g < n) {
        R* dst = out + static_cast<size_t>(row0 + g) * n + half;
#pragma unroll
        for (int i = 0; i < 16; ++i) {
            const int p = tid + NT * i;
            if (i < 4 || i >= 12) {
                const int o = (i < 4) ? p : p - F;
                const bool inside = (i < 4) ? (p < half) : (p >= F - half);
                if (inside)
                    dst[o] = static_cast<R>(static_cast<double>(v[i].x) +
                                            static_cast<double>(v[i].y) * dpre[i < 4 ? i : i - 8]);
            }
        }
    }
}

// Two rows at a time (see rows_forward_pair_body): V = (S_a + E_a) + i (S_b + E_b)
// with S the Hermitian extension of a row's I1 half spectrum and E = sum_j
// delta_|j| H[m - j] the type-1 row's Hermitian part H with its deconvolution,
// in FP64; one inverse FFT, Phi_a = Re, Phi_b = Im.  E is zero beyond the window
// by more than B.  The windows' H sits in the start of the transform buffers
// while E is summed (into registers, the spectrum loads in flight), then the
// spectrum takes their place and E is added.
template <typename R, int LOG, int DIR, bool USE_I1, bool USE_I2, int G, bool EXACT>
__device__ __forceinline__ void rows_inverse_pair_body(const DevPlan& P, R* __restrict__ out, int pair0,
                                                       cpx<R>* lds_all) {
    using Sh = FftShape<LOG>;
    constexpr int F = Sh::F;
    constexpr int HALF = F / 2;
    constexpr int NT = Sh::NT;
    constexpr int LP = lds_group_stride(F);
    constexpr int BT = NT * G;
    const int n = EXACT ? F / 2 : P.n;
    const int pairs = n >> 1;
    const int g = threadIdx.x / NT;
    const int tid = threadIdx.x - g * NT;
    cpx<R>* lds = lds_all + g * LP;
    const cpx<R>* tw = static_cast<const cpx<R>*>(P.twr);
    const cpx<R>* xt = static_cast<const cpx<R>*>(P.xt);
    constexpr int ITEMS = (HALF + 1) * G;
    constexpr int PASSES = (ITEMS + BT - 1) / BT;
    cpx_pair<R> xr[PASSES];
#pragma unroll
    for (int k = 0; k < PASSES; ++k) {
        const int idx = threadIdx.x + k * BT;
        const int idc = idx < ITEMS ? idx : ITEMS - 1;
        const int pair = min(pair0 + idc % G, pairs - 1);   // pairs past N/2 read the last one, never stored
        xr[k] = cpx_pair<R>{{R(0), R(0)}, {R(0), R(0)}};
        if constexpr (USE_I1)
            xr[k] = *reinterpret_cast<const cpx_pair<R>*>(xt + static_cast<size_t>(idc / G) * P.col_stride + 2 * pair);
    }
    // E on m = 0 .. M-1: the NT threads of a transform do their pair's, PT lanes per value
    constexpr int PT = NT >= 256 ? 4 : NT >= 128 ? 2 : 1;
    constexpr int STEP = NT / PT;
    constexpr int KMAX = (kMaxPairWindow / 2 + kMaxPairTaps + 1 + STEP - 1) / STEP;
    const int B = P.pair_taps;
    const int q = P.patch, lo = P.patch_lo, c0 = P.nd.col_lo, c1 = P.nd.col_hi;
    const int lm = max(-(lo + c0), lo + c1 - 1);                      // |l| <= lm in the window columns
    const int M = lm + B + 1;
    const int part = tid % PT;
    double ea[KMAX][2], eb[KMAX][2];
    if constexpr (USE_I2) {
        // H[l], l = 0 .. lm, of both rows (H[-l] = conj H[l])
        const cpx<R>* u = static_cast<const cpx<R>*>(P.u);
        const int items = (lm + 1) * 2 * G;
        for (int e = threadIdx.x; e < items; e += BT) {
            const int l = e % (lm + 1);
            const int row = e / (lm + 1);                             // 2 gg + (0: a, 1: b)
            const int gg = row >> 1;
            const int r = 2 * min(pair0 + gg, pairs - 1) + (row & 1);
            const int ia = l - lo, ib = -l - lo;
            const bool in_a = ia >= c0 && ia < c1, in_b = ib >= c0 && ib < c1;
            const cpx<R>* urow = u + static_cast<size_t>(r) * q;
            const cpx<R> ua0 = urow[in_a ? ia : c0];
            const cpx<R> ub0 = urow[in_b ? ib : c0];
            const cpx<R> ua = in_a ? ua0 : cpx<R>{R(0), R(0)};
            const cpx<R> ub = in_b ? ub0 : cpx<R>{R(0), R(0)};
            lds_all[gg * LP + (row & 1) * (lm + 1) + l] = {R(0.5) * (ua.x + ub.x), R(0.5) * (ua.y - ub.y)};
        }
        __syncthreads();
        const cpx<R>* ha = lds;
        const cpx<R>* hb = ha + lm + 1;
#pragma unroll
        for (int k = 0; k < KMAX; ++k) {
            const int m = tid / PT + k * STEP;
            ea[k][0] = ea[k][1] = eb[k][0] = eb[k][1] = 0.0;
            if (m < M) {
                const int l1 = min(lm, m + B);
#pragma unroll 4
                for (int l = max(-lm, m - B) + part; l <= l1; l += PT) {
                    const int al = l < 0 ? -l : l;
                    const int j = m > l ? m - l : l - m;
                    const double d = P.delta[j];
                    const double ds = l < 0 ? -d : d;
                    const cpx<R> a = ha[al], b = hb[al];
                    ea[k][0] += d * a.x;
                    ea[k][1] += ds * a.y;
                    eb[k][0] += d * b.x;
                    eb[k][1] += ds * b.y;
                }
            }
#pragma unroll
            for (int off = 1; off < PT; off <<= 1) {
                ea[k][0] += __shfl_xor(ea[k][0], off, PT);
                ea[k][1] += __shfl_xor(ea[k][1], off, PT);
                eb[k][0] += __shfl_xor(eb[k][0], off, PT);
                eb[k][1] += __shfl_xor(eb[k][1], off, PT);
            }
        }
        __syncthreads();
    }
#pragma unroll
    for (int k = 0; k < PASSES; ++k) {
        const int idx = threadIdx.x + k * BT;
        const int gg = idx % G;
        const int m = idx / G;
        cpx<R>* l = lds_all + gg * LP;
        const cpx<R> a = xr[k].a, b = xr[k].b;
        // position m: S_a + i S_b;  position F - m: conj S_a + i conj S_b
        if (idx < ITEMS) {
            l[lds_pad(m)] = {a.x - b.y, a.y + b.x};
            if (m > 0 && m < HALF) l[lds_pad(F - m)] = {a.x + b.y, b.x - a.y};
        }
    }
    __syncthreads();
    if constexpr (USE_I2) {
#pragma unroll
        for (int k = 0; k < KMAX; ++k) {
            const int m = tid / PT + k * STEP;
            if (part == 0 && m < M) {
                cpx<R>* p = lds + lds_pad(m);
                *p = {static_cast<R>(p->x + (ea[k][0] - eb[k][1])), static_cast<R>(p->y + (ea[k][1] + eb[k][0]))};
                if (m > 0) {
                    cpx<R>* c = lds + lds_pad(F - m);
                    *c = {static_cast<R>(c->x + (ea[k][0] + eb[k][1])), static_cast<R>(c->y + (eb[k][0] - ea[k][1]))};
                }
            }
        }
        __syncthreads();
    }
    cpx<R> v[16];
#pragma unroll
    for (int i = 0; i < 16; ++i) v[i] = lds[lds_pad(tid + NT * i)];
    fft_reg<R, LOG, DIR>(v, lds, tw, tid);
    const int half = EXACT ? F / 4 : (n >> 1);
    if ((EXACT || pair0 + g < pairs)) {
        R* dst = out + static_cast<size_t>(2 * (pair0 + g)) * n + half;
#pragma unroll
        for (int i = 0; i < 16; ++i) {
            const int p = tid + NT * i;
            if (i < 4 || i >= 12) {
                const int o = (i < 4) ? p : p - F;
                const bool inside = (i < 4) ? (p < half) : (p >= F - half);
                if (inside) {
                    dst[o] = v[i].x;
                    dst[n + o] = v[i].y;
                }
            }
        }
    }
}

}  // namespace phi
