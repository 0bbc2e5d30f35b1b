// P2M of one leaf by one wavefront (device code only): the coefficients of
// sum_a w_a Upsilon_n^m(x_a - z) for weights w_a; used for the multipoles and, with
// weights that hold the velocities, for their rates.
#pragma once

#include "internal.h"
#include "harmonics.h"
#include "near.h"

namespace fmm {

namespace {

// The columns of Upsilon as monic polynomials: Upsilon_n^m = scale V_n with
// V_m = Upsilon_m^m, V_n = z V_{n-1} - step r^2 V_{n-2},
// step = ((n-1)^2 - m^2) / ((2n-1)(2n-3)), scale = prod_{i=m+1..n} (2i-1)/(i^2-m^2).
struct ColumnTable {
    double step[FMM_PMAX + 1][FMM_PMAX + 1], scale[FMM_PMAX + 1][FMM_PMAX + 1];
};
constexpr ColumnTable make_column_table() {
    ColumnTable tb{};
    for (int m = 0; m <= FMM_PMAX; ++m) {
        tb.scale[m][m] = 1.0;
        for (int n = m + 1; n <= FMM_PMAX; ++n) {
            tb.step[n][m] = n < 2 ? 0.0
                                  : (double)((n - 1) * (n - 1) - m * m) /
                                        (double)((2 * n - 1) * (2 * n - 3));
            tb.scale[n][m] = tb.scale[n - 1][m] * (double)(2 * n - 1) / (double)(n * n - m * m);
        }
    }
    return tb;
}
__constant__ ColumnTable kColumn = make_column_table();

struct FactTable {
    double v[2 * FMM_PMAX + 1];
};
constexpr FactTable make_fact_table() {
    FactTable f{};
    f.v[0] = 1.0;
    for (int i = 1; i <= 2 * FMM_PMAX; ++i) f.v[i] = f.v[i - 1] * i;
    return f;
}
__constant__ FactTable kFact = make_fact_table();

// Lanes are (particle slot, j):
// CP lanes per particle, lane j generates columns m = j and m = P - j of its
// particle's Upsilon (P + 2 coefficients in all, the same number on every
// lane, where a lane per column would leave the upper triangle n < m idle):
// the diagonals Upsilon_m^m = ((x + iy)/2)^m / m! by repeated squaring, then down
// the column, step q of the lane's sequence being (n, m) = (j + q, j) for
// q <= P - j and (q - 1, P - j) after that.  Each lane keeps the running sums of
// its sequence (unscaled); the particle slots are added at the end by lane
// swaps, which halve the values each lane holds, and moves within a row of 16.
// For even P the middle column (j = P / 2) is generated twice and stored once.
// Bound by FP64 instructions: 10^6 bodies in 3.6 x 10^4 leaves, p = 15: 179 us;
// with the diagonal as a chain, a table read and six operations per step and
// sums through LDS, 312 us.
template <int P>
struct P2MLeaf {
    static constexpr int NJ = P / 2 + 1;                       // column pairs (j <= P / 2)
    static constexpr int CP = NJ <= 2 ? 2 : NJ <= 4 ? 4 : NJ <= 8 ? 8 : 16;
    static constexpr int SL = FMM_WAVE / CP;                   // particles per step
    static constexpr int T = P + 2;                            // steps per lane
    typedef double Steps[T][CP];

    // the columns' step factors of every lane, from LDS in the loop: in registers
    // they leave room for two wavefronts per SIMD (234 us); a block of 256 fills them
    static __device__ __forceinline__ void fill(Steps &step) {
        for (int e = threadIdx.x; e < T * CP; e += 256) {
            const int q = e / CP, a = e % CP < NJ ? e % CP : 0;
            const bool one = q < P + 1 - a;
            step[q][e % CP] = kColumn.step[one ? a + q : q - 1][one ? a : P - a];
        }
        __syncthreads();
    }

    // weight(i): particle i's; out(n, m, half, v): the real (half 0) or imaginary
    // part of coefficient (n, m), once each
    template <class W, class O>
    static __device__ __forceinline__ void run(const Steps &step, int beg, int end,
                                               const double4 &cen, const double *x,
                                               const double *y, const double *z, W &&weight,
                                               O &&out) {
        const int lane = lane_id(), j = lane % CP, slot = lane / CP;
        const bool on = j < NJ;
        const int c1 = on ? j : 0, c2 = P - c1;
        const int L1 = P + 1 - c1;             // steps of the first column
        const bool two = c2 > c1;              // a second column (not the middle one)
        const double f1 = 1.0 / kFact.v[c1], f2 = 1.0 / kFact.v[c2];
        cplx acc[T];
#pragma unroll
        for (int q = 0; q < T; ++q) acc[q] = {0.0, 0.0};
        for (int i0 = beg; i0 < end; i0 += SL) {
            asm volatile("" ::: "memory");     // the factors stay in LDS
            const int i = i0 + slot;
            const bool valid = i < end && on;
            const double mu = valid ? weight(i) : 0.0;
            const double dx = valid ? x[i] - cen.x : 0.0, dy = valid ? y[i] - cen.y : 0.0,
                         dz = valid ? z[i] - cen.z : 0.0;
            const double r2 = fma(dx, dx, fma(dy, dy, dz * dz));
            cplx d1 = {mu * f1, 0.0}, d2 = {mu * f2, 0.0}, w = {0.5 * dx, 0.5 * dy};
#pragma unroll
            for (int b = 1; b <= P; b <<= 1) {
                if (c1 & b) d1 = cmul(d1, w);
                if (c2 & b) d2 = cmul(d2, w);
                w = {fma(w.re, w.re, -w.im * w.im), 2.0 * w.re * w.im};
            }
            cplx u1 = d1, u2 = {0.0, 0.0};
            acc[0].re += u1.re;
            acc[0].im += u1.im;
#pragma unroll
            for (int q = 1; q < T; ++q) {
                const double k = step[q][j] * r2;
                cplx u = {fma(dz, u1.re, -k * u2.re), fma(dz, u1.im, -k * u2.im)};
                u2 = u1;
                if (q >= P + 2 - NJ && q == L1) {      // the second column starts
                    u = d2;
                    u2 = {0.0, 0.0};
                }
                acc[q].re += u.re;
                acc[q].im += u.im;
                u1 = u;
            }
        }
        // lower lanes the real parts, upper lanes the imaginary ones; then even rows
        // of 16 the first half of the sequence, odd rows the second
        constexpr int H = (T + 1) / 2;
        double s[2 * H];
#pragma unroll
        for (int q = 0; q < T; ++q) {
            swap32(acc[q].re, acc[q].im);
            s[q] = acc[q].re + acc[q].im;
        }
        if (T < 2 * H) s[T] = 0.0;
        const int half = lane / 32, row = (lane / 16) & 1;
#pragma unroll
        for (int i = 0; i < H; ++i) {
            swap16(s[i], s[i + H]);
            double v = s[i] + s[i + H];
            if (CP <= 8) v += dpp_double<DPP_ROW_ROR + 8>(v);
            if (CP <= 4) v += dpp_double<DPP_ROW_ROR + 4>(v);
            if (CP <= 2) v += dpp_double<DPP_ROW_ROR + 2>(v);
            const int q = i + H * row;
            // the lanes of a row that hold the same sums store in turn
            if (!on || q >= T || (q >= L1 && !two) || (lane % 16) / CP != i % (16 / CP)) continue;
            const int n = q < L1 ? c1 + q : q - 1, col = q < L1 ? c1 : c2;
            out(n, col, half, half && col == 0 ? 0.0 : kColumn.scale[n][col] * v);
        }
    }
};

}  // namespace

}  // namespace fmm
