// Register-resident M2L kernel template (see m2l.hip for the algorithm).
// Included by the translation units that instantiate it for a range of
// expansion orders, so that the orders compile in parallel.
#pragma once

#include "internal.h"
#include "harmonics.h"

namespace fmm {
namespace m2l_detail {

// The interaction in the frame turned about z by the azimuth phi of r = s_B - z_A
// (Theta_n^m(r) = e^{im phi} T_n^m with T real): with M'_k^l = e^{-il phi} M_k^l,
//   F_n^m = e^{im phi} F'_n^m,   F'_n^m = sum_{k, l} conj(M'_k^l) T_{n+k}^{m+l},
// and conj(M'_k^{-l}) = (-1)^l M'_k^l, T_J^{-q} = (-1)^q T_J^q.  A real T halves
// both the registers of its rows and the multiply-adds.  The accumulators stay
// in the frame of the current source and are turned by the change of azimuth
// from one source to the next.
//
// The outputs are split by degree into passes of N0..N1, each generating T
// again: a pass keeps its accumulators and the rows N0 + k .. N1 + k that the
// multipoles of degree k meet (a ring of rows, one new row per k), together at
// most M2L_REGS registers, so that two wavefronts share a SIMD; each multipole
// is loaded once per pass, in storage order, M2L_AHEAD ahead of its use.  The lanes
// read different cells, so a load visits the L1 cache once per lane: the number
// of loads and of multiply-adds bound the kernel about equally.
//
// At 10^6 bodies, p = 15 (1.9 x 10^6 pairs) / 10^5, p = 13 / a list of 5.7 x 10^4
// pairs, p = 15: 2.05 / 0.24 / 0.20 ms.  With 150 registers (more passes) 2.42 /
// 0.24 / 0.18, with 235 (spills) 2.01 / 0.32 / 0.25; with 2 multipoles ahead 1.99 /
// 0.28 / 0.21, with 8 (more spills) 2.01 / 0.24 / 0.19.
constexpr int M2L_REGS = 195;    // 32-bit registers of accumulators and rows
constexpr int M2L_AHEAD = 4;     // multipoles in flight

// last degree of the pass that begins with degree n0
__host__ __device__ constexpr int pass_end(int p, int n0) {
    int n = n0;
    for (;; ++n) {
        if (n == p) return n;
        int acc = 0;
        for (int i = n0; i <= n + 1; ++i) acc += 2 * i + 1;
        int rows = n + 1 - n0 + 1;
        if (rows > p - n0 + 1) rows = p - n0 + 1;
        if (rows < 2) rows = 2;
        if (2 * (acc + rows * (p + 1)) > M2L_REGS) return n;
    }
}
__host__ __device__ constexpr int pass_count(int p) {
    int c = 0;
    for (int n0 = 0; n0 <= p; n0 = pass_end(p, n0) + 1) ++c;
    return c;
}

// Rows of T, the irregular harmonics at (rho, 0, z): the recurrences of
// App. A.5 with x + iy = rho, one degree at a time.  Row J sits in slot J % W.
template <int P, int W>
struct RealTheta {
    double rows[W][P + 1];
    double rho, z, ir2;
    __device__ __forceinline__ void start(double rho_, double z_) {
        rho = rho_;
        z = z_;
        const double ri = rsqrt_nr(fma(rho, rho, z * z));
        ir2 = ri * ri;
        rows[0][0] = ri;
    }
    template <int J>
    __device__ __forceinline__ void next() {
        static_assert(J > 0, "row 0 is set by start");
        double *cur = rows[J % W];
        const double *p1 = rows[(J - 1) % W], *p2 = rows[(J + W - 2) % W];
        const double a = 2.0 * J - 1.0, s = a * z;
#pragma unroll
        for (int m = 0; m <= J - 2; ++m)
            cur[m] = (s * p1[m] - (double)((J - 1) * (J - 1) - m * m) * p2[m]) * ir2;
        const double d = p1[J - 1] * ir2;
        cur[J - 1] = s * d;
        cur[J] = a * rho * d;
    }
    template <int J>
    __device__ __forceinline__ const double *row() const { return rows[J % W]; }
};

// (cos, sin) of an angle; advance turns it by d
struct Phase {
    double c, s;
    __device__ __forceinline__ void advance(const Phase &d) {
        const double c0 = c;
        c = c0 * d.c - s * d.s;
        s = s * d.c + c0 * d.s;
    }
};

// accumulators N0..N1 times e^{-im delta}
template <int N0, int N1>
__device__ __forceinline__ void turn(cplx *acc, const Phase &delta) {
    Phase ph = delta;
#pragma unroll
    for (int m = 1; m <= N1; ++m) {
#pragma unroll
        for (int n = m > N0 ? m : N0; n <= N1; ++n) {
            cplx &f = acc[tri(n, m) - tri(N0, 0)];
            const double re = f.re;
            f.re = re * ph.c + f.im * ph.s;
            f.im = f.im * ph.c - re * ph.s;
        }
        if (m < N1) ph.advance(delta);
    }
}

// the terms of M'_K^L = a + ib in the outputs of the pass
template <int P, int N0, int N1, int K, int L, class Rows>
__device__ __forceinline__ void contract(cplx *acc, const Rows &g, double a, double b) {
    const double a2 = 2.0 * a;
    auto degree = [&]<int n>() {
        const double *th = g.template row<n + K>();
#pragma unroll
        for (int m = 0; m <= n; ++m) {
            cplx &f = acc[tri(n, m) - tri(N0, 0)];
            if constexpr (L == 0) {
                f.re = fma(a, th[m], f.re);
            } else if (m == 0) {
                f.re = fma(a2, th[L], f.re);
            } else {
                const double tp = th[m + L], tm = th[m > L ? m - L : L - m];
                const bool neg = m >= L ? (L & 1) : (m & 1);
                f.re = fma(a, tp, f.re);
                f.re = fma(neg ? -a : a, tm, f.re);
                f.im = fma(-b, tp, f.im);
                f.im = fma(neg ? -b : b, tm, f.im);
            }
        }
    };
    Unroll<N0, (N1 < P - K ? N1 : P - K)>::run(degree);
}

// one source's terms of a pass in its own frame; Ma: its multipoles, phi: its
// azimuth
template <int P, int N0, int N1, class Rows>
__device__ __forceinline__ void source_terms(cplx *acc, Rows &g, const cplx *Ma,
                                             const Phase &phi) {
    constexpr int KMAX = P - N0, COUNT = tri(KMAX + 1, 0);
    cplx ring[M2L_AHEAD];
#pragma unroll
    for (int i = 0; i < M2L_AHEAD; ++i)
        if (i < COUNT) ring[i] = Ma[i];
    auto first = [&]<int J>() { g.template next<J>(); };
    Unroll<1, N1>::run(first);
    auto degree = [&]<int k>() {
        if constexpr (k > 0 && N1 + k <= P) g.template next<N1 + k>();
        Phase ph{1.0, 0.0};
        auto order = [&]<int l>() {
            constexpr int i = tri(k, l);
            const cplx v = ring[i % M2L_AHEAD];
            if constexpr (i + M2L_AHEAD < COUNT) ring[i % M2L_AHEAD] = Ma[i + M2L_AHEAD];
            double a = v.re, b = v.im;
            if constexpr (l > 0) {
                ph.advance(phi);
                a = v.re * ph.c + v.im * ph.s;
                b = v.im * ph.c - v.re * ph.s;
            }
            contract<P, N0, N1, k, l>(acc, g, a, b);
            // loads stay where they are issued
            __asm__ volatile("" ::: "memory");
        };
        Unroll<0, k>::run(order);
    };
    Unroll<0, KMAX>::run(degree);
}

// azimuth of (x, y) and its distance from the z axis.  On the axis any azimuth
// does (0), and so close to it that x^2 + y^2 is denormal x/rho and y/rho would
// not be the cosine and sine of an angle: they would scale the accumulators that
// they turn.  So within 1e-145 of the axis is on it (a separation as short as that
// has no finite Theta_2 anyway).
__device__ __forceinline__ Phase azimuth(double x, double y, double &rho) {
    const double r2 = fma(x, x, y * y);
    const bool off = r2 > 1e-290;
    const double ri = off ? rsqrt_nr(r2) : 0.0;
    rho = r2 * ri;
    return off ? Phase{x * ri, y * ri} : Phase{1.0, 0.0};
}

// outputs N0..N1 of order P from multipoles of `stride` complex numbers per cell
template <int P, int N0, int N1>
__device__ __forceinline__ void m2l_pass(int B, int e0, int e1, const uint64_t *list,
                                         uint64_t mask, const TreeArrays &t, const cplx *M,
                                         int stride, cplx *out) {
    constexpr int NACC = tri(N1 + 1, 0) - tri(N0, 0);
    cplx acc[NACC];
#pragma unroll
    for (int i = 0; i < NACC; ++i) acc[i] = {0.0, 0.0};
    const double4 cb = t.cen[B];
    int A = (int)(list[e0] & mask);
    double4 ca = t.cen[A];
    Phase at{1.0, 0.0};      // azimuth of the accumulators' frame
    for (int e = e0; e < e1; ++e) {
        // the next source's index and centre, ahead of its turn
        const int An = (int)(list[e + 1 < e1 ? e + 1 : e] & mask);
        const double4 can = t.cen[An];
        const double x = cb.x - ca.x, y = cb.y - ca.y, z = cb.z - ca.z;
        double rho;
        const Phase phi = azimuth(x, y, rho);
        turn<N0, N1>(acc, Phase{phi.c * at.c + phi.s * at.s, phi.s * at.c - phi.c * at.s});
        at = phi;
        RealTheta<P, (N1 > N0 ? N1 - N0 + 1 : 2)> g;
        g.start(rho, z);
        source_terms<P, N0, N1>(acc, g, M + (size_t)A * stride, phi);
        A = An;
        ca = can;
    }
    turn<N0, N1>(acc, Phase{at.c, -at.s});
#pragma unroll
    for (int n = N0; n <= N1; ++n)
#pragma unroll
        for (int m = 0; m <= n; ++m)
            out[tri(n, m)] = {acc[tri(n, m) - tri(N0, 0)].re,
                              m == 0 ? 0.0 : acc[tri(n, m) - tri(N0, 0)].im};
}

// the pass with index `pass` (the same in every lane)
template <int P, int N0>
__device__ __forceinline__ void m2l_passes(int pass, int B, int e0, int e1, const uint64_t *list,
                                           uint64_t mask, const TreeArrays &t, const cplx *M,
                                           cplx *out) {
    constexpr int N1 = pass_end(P, N0);
    if (pass == 0)
        m2l_pass<P, N0, N1>(B, e0, e1, list, mask, t, M, tri(P + 1, 0), out);
    else if constexpr (N1 < P)
        m2l_passes<P, N1 + 1>(pass - 1, B, e0, e1, list, mask, t, M, out);
}

// blocks of 64 chunks, rounded up to the XCD count
__host__ __device__ constexpr int m2l_blocks(int nchunks) {
    return ((nchunks + 63) / 64 + FMM_NXCD - 1) / FMM_NXCD * FMM_NXCD;
}

// the chunk of this lane, or -1.  The grid is sized by a bound of the chunk
// count; each XCD takes a contiguous eighth of the blocks that hold chunks.
__device__ __forceinline__ int my_chunk(int nchunks) {
    const int nb = m2l_blocks(nchunks);
    if ((int)blockIdx.x >= nb) return -1;
    const int ch = xcd_block(blockIdx.x, nb) * 64 + threadIdx.x;
    return ch < nchunks ? ch : -1;
}

// One lane per chunk and pass: the grid's y dimension takes the passes, so that
// a short list still has several wavefronts per 64 chunks.  gridDim.x is a
// multiple of the XCD count, so that a chunk's passes share an L2.
template <int P>
__global__ void __launch_bounds__(64) __attribute__((amdgpu_waves_per_eu(2)))
k_m2l(const int *nchunks, const int4 *chunks, const uint64_t *list, uint64_t mask, TreeArrays t,
      const double *M, double *Fpart) {
    const int ch = my_chunk(*nchunks);
    if (ch < 0) return;
    const int4 c = chunks[ch];
    cplx *out = reinterpret_cast<cplx *>(Fpart) + (size_t)ch * tri(P + 1, 0);
    m2l_passes<P, 0>(blockIdx.y, c.x, c.y, c.z, list, mask, t, reinterpret_cast<const cplx *>(M),
                     out);
}


}  // namespace m2l_detail
}  // namespace fmm

// launcher of the order-P register kernel (defined in the m2l_p*.hip units)
#define FMM_M2L_FIXED_DEFINE(P)                                                              \
    namespace fmm {                                                                          \
    hipError_t launch_m2l_fixed_##P(int bound, const int *nchunks, const int4 *chunks,    \
                                    const uint64_t *list, uint64_t mask, const TreeArrays &t, \
                                    const double *M, double *Fpart, hipStream_t s) {         \
        hipLaunchKernelGGL(m2l_detail::k_m2l<P>,                                             \
                           dim3(m2l_detail::m2l_blocks(bound), m2l_detail::pass_count(P)),   \
                           dim3(64), 0, s, nchunks, chunks, list, mask, t, M, Fpart);       \
        return hipGetLastError();                                                            \
    }                                                                                        \
    }
