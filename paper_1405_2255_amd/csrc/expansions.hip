// Upward and downward passes: P2M (eq:P2M), M2M (eq:M2M), multipole power
// P_n (eq:def:PA), L2L (eq:L2L), L2P (eq:L2P:Psi, eq:L2P), and the low-order
// estimate of the sink scale (Sec. 5.4.2).
//
// Storage: per cell the complex X_n^m for 0 <= m <= n <= p at complex index
// tri(n, m) = n(n+1)/2 + m, (Re, Im) adjacent, Im = 0 for m = 0.
#include "internal.h"
#include "harmonics.h"
#include "near.h"
#include "p2m_impl.h"

namespace fmm {

namespace {

// ---- P2M: M_n^m(z) = sum_a mu_a Upsilon_n^m(x_a - z), a wavefront per leaf -----
template <int P>
__global__ void __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(P <= 15 ? 3 : 2)))
k_p2m(TreeArrays t, const int *leaf_cell, int nleaves, const double *x, const double *y,
      const double *z, const double *m, double *M) {
    __shared__ typename P2MLeaf<P>::Steps step;
    P2MLeaf<P>::fill(step);
    const int leaf = blockIdx.x * 4 + threadIdx.x / FMM_WAVE;
    if (leaf >= nleaves) return;
    const int c = leaf_cell[leaf];
    double *Mc = M + (size_t)c * 2 * tri(P + 1, 0);
    P2MLeaf<P>::run(step, t.beg[c], t.end[c], t.cen[c], x, y, z, [&](int i) { return m[i]; },
                    [&](int n, int col, int half, double v) { Mc[2 * tri(n, col) + half] = v; });
}

__device__ __forceinline__ cplx ld(const cplx *X, int n, int q) {
    return sym(X[tri(n, q < 0 ? -q : q)], q);
}

// ---- shifts (M2M, L2L): three one-dimensional sums ---------------------------
// A shift by r = (x, y, z) is the sum over (k, l) of Upsilon_k^l(r) with the
// cell's coefficients, O(p^4) terms.  By the addition theorem (a polynomial
// identity, valid for complex vectors too) Upsilon(r) is the convolution of
// those of the three parts
//   (0, 0, z):              Upsilon_k^0  = z^k / k!,       all else 0,
//   (w, -i w, 0):           Upsilon_k^k  = w^k / k!,       all else 0,
//   (-w~, ...) = its mirror: Upsilon_k^-k = (-w~)^k / k!,  all else 0,
// with w = (x + i y) / 2 (the last two vectors have length 0 and add up to
// (x, y, 0)).  The shift is then three sums over one index each, O(p^3) terms:
// 4 x 10^2 complex multiply-adds per sum at p = 15 against 5 x 10^3.  Against
// extended precision its error equals that of the sum over (k, l).
//
// One wavefront per cell, four cells per block: R coefficients per lane in LDS,
// weight j in lane j.  Four terms of every sum are read together; a term that
// does not exist reads a zero, so that the wavefront never parts.  Bound by
// latency in the levels with few cells (7 us a level) and by bytes and the sums'
// instructions elsewhere.  At p = 15, 5 x 10^4 cells, the M2M levels take 342 us
// with P_n, where a block per cell over (k, l) took 476 us, after 73 us for the
// Upsilon of each cell and before 55 us for P_n.
constexpr int XF_CELLS = 4;                                  // per block

// LDS of one cell: stored coefficients, then a zero; all orders (at n^2 + n + m),
// then a zero
inline __host__ __device__ int shift_lds_cplx(int p) {
    return tri(p + 1, 0) + 1 + (p + 1) * (p + 1) + 1;
}

// what one lane wrote to LDS is there for the others of its wavefront
__device__ __forceinline__ void wave_fence() {
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    __builtin_amdgcn_wave_barrier();
}

// a^j / j! in lane j <= p (by repeated squaring), 0 in the others
__device__ __forceinline__ cplx power_weight(int p, cplx a) {
    const int j = lane_id();
    cplx v = {1.0, 0.0};
#pragma unroll
    for (int q = 0; q < 5; ++q) {
        if ((j >> q) & 1) v = cmul(v, a);
        a = cmul(a, a);
    }
    if (j > p) return {0.0, 0.0};
    const double f = 1.0 / kFact.v[j];
    return {v.re * f, v.im * f};
}
__device__ __forceinline__ double power_weight(int p, double a) {
    const int j = lane_id();
    double v = 1.0;
#pragma unroll
    for (int q = 0; q < 5; ++q) {
        if ((j >> q) & 1) v *= a;
        a *= a;
    }
    return j > p ? 0.0 : v / kFact.v[j];
}

__device__ __forceinline__ void add_term(double wz, cplx x, cplx &s) {
    s.re = fma(wz, x.re, s.re);
    s.im = fma(wz, x.im, s.im);
}
__device__ __forceinline__ void add_term(cplx w, cplx x, cplx &s) {
    s.re = fma(w.re, x.re, fma(-w.im, x.im, s.re));
    s.im = fma(w.re, x.im, fma(w.im, x.re, s.im));
}
__device__ __forceinline__ double from_lane(double v, int j) { return readlane_f64(v, j); }
__device__ __forceinline__ cplx from_lane(cplx v, int j) {
    return {readlane_f64(v.re, j), readlane_f64(v.im, j)};
}

// degree and order of coefficient index e = tri(n, m)
__device__ __forceinline__ void nm_of(int e, int &n, int &m) {
    n = (int)((sqrtf(8.0f * (float)e + 1.0f) - 1.0f) * 0.5f);
    if (tri(n + 1, 0) <= e) ++n;
    if (tri(n, 0) > e) --n;
    m = e - tri(n, 0);
}

// One of the three sums for the R coefficients of a lane: terms j = 0 .. last[r]
// at index i, i + step, i + 2 step + grow, ... of X; jmax: the largest last.
template <int R, class W>
__device__ __forceinline__ void shift_sum(W weight, const cplx *X, int zero, int jmax, int grow,
                                          const int *first, const int *step0, const int *last,
                                          cplx *s) {
    int i[R], step[R];
#pragma unroll
    for (int r = 0; r < R; ++r) {
        i[r] = first[r];
        step[r] = step0[r];
        s[r] = {0.0, 0.0};
    }
    for (int j0 = 0; j0 <= jmax; j0 += 4) {
        cplx x[4][R];
#pragma unroll
        for (int q = 0; q < 4; ++q)
#pragma unroll
            for (int r = 0; r < R; ++r) {
                x[q][r] = X[j0 + q <= last[r] ? i[r] : zero];
                i[r] += step[r];
                step[r] += grow;
            }
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            const W wj = from_lane(weight, j0 + q);
#pragma unroll
            for (int r = 0; r < R; ++r) add_term(wj, x[q][r], s[r]);
        }
    }
}

struct Binomials {
    double v[FMM_PMAX + 1];
};

// ---- M2M and the multipole power --------------------------------------------
// Level by level from the bottom.  The wavefront of cell c first completes
// M(c): for an internal cell the sum, in child order, of the children's shifted
// expansions T(child) written by the previous level's launch (a leaf keeps its
// P2M result); then the power P_n^2 = sum_m (n-m)!(n+m)! |M_n^m|^2, stored as
// C(p, n) P_n, as the walk's error estimate uses it (P not null); then, unless
// c is a root, the shift of M(c) to the parent's centre,
//   T_n^m(c) = sum_{k=0}^{n} sum_{l=-k}^{k} Upsilon_k^l(z_c - z_parent) M_{n-k}^{m-l}(c).
template <int R>
__global__ void __launch_bounds__(XF_CELLS * FMM_WAVE)
k_m2m_level(int p, TreeArrays t, int c0, int c1, double *M, double *T, Binomials binom,
            double *P) {
    extern __shared__ double lds[];
    const int w = threadIdx.x / FMM_WAVE, lane = lane_id();
    const int c = c0 + blockIdx.x * XF_CELLS + w;
    if (c >= c1) return;
    const int nc = tri(p + 1, 0), nf = (p + 1) * (p + 1);
    cplx *half = reinterpret_cast<cplx *>(lds) + w * shift_lds_cplx(p), *full = half + nc + 1;
    const int4 info = t.info[c];
    const int nch = info.w, pc = t.parent[c];
    const double4 ca = t.cen[c], cb = t.cen[max(pc, 0)];
    cplx *Mc = reinterpret_cast<cplx *>(M) + (size_t)c * nc;
    const cplx *Tb = reinterpret_cast<const cplx *>(T) + (size_t)info.z * nc;
    int n[R], m[R], first[R], step[R], last[R];
    cplx v[R];
    double f2[R];
#pragma unroll
    for (int r = 0; r < R; ++r) {
        const int e = r * FMM_WAVE + lane, ee = min(e, nc - 1);
        nm_of(ee, n[r], m[r]);
        f2[r] = kFact.v[n[r] - m[r]] * kFact.v[n[r] + m[r]];
        if (nch > 0) {
            // the (at most 8) children's terms loaded together, added in order
            v[r] = {0.0, 0.0};
            cplx xs[8];
#pragma unroll
            for (int j = 0; j < 8; ++j) xs[j] = Tb[(size_t)(j < nch ? j : 0) * nc + ee];
#pragma unroll
            for (int j = 0; j < 8; ++j) {
                if (j < nch) {
                    v[r].re += xs[j].re;
                    v[r].im += xs[j].im;
                }
            }
            if (e < nc) Mc[e] = v[r];
        } else {
            v[r] = Mc[ee];
        }
        if (e < nc) half[e] = v[r];
    }
    if (lane == 0) half[nc] = full[nf] = {0.0, 0.0};
    if (P) {
        double *term = reinterpret_cast<double *>(full);
#pragma unroll
        for (int r = 0; r < R; ++r) {
            const int e = r * FMM_WAVE + lane;
            const double q = f2[r] * (v[r].re * v[r].re + v[r].im * v[r].im);
            if (e < nc) term[e] = m[r] == 0 ? q : 2.0 * q;
        }
        wave_fence();
        if (lane <= p) {
            double q = 0.0;
#pragma unroll 4
            for (int i = 0; i <= lane; ++i) q += term[tri(lane, i)];
            P[(size_t)c * power_stride(p) + lane] = binom.v[lane] * sqrt(q);
        }
    }
    if (pc < 0) return;
    const cplx wp = {0.5 * (ca.x - cb.x), 0.5 * (ca.y - cb.y)};
    const double wz = power_weight(p, ca.z - cb.z);
    const cplx wplus = power_weight(p, wp), wminus = power_weight(p, cplx{-wp.re, wp.im});
    wave_fence();
    cplx s[R];
    // along z: sum_j z^j/j! M_{n-j}^m
#pragma unroll
    for (int r = 0; r < R; ++r) {
        first[r] = tri(n[r], m[r]);
        step[r] = -n[r];
        last[r] = n[r] - m[r];
    }
    shift_sum<R>(wz, half, nc, p, 1, first, step, last, s);
#pragma unroll
    for (int r = 0; r < R; ++r) {
        if (r * FMM_WAVE + lane >= nc) continue;
        cplx *f = full + n[r] * n[r] + n[r];
        f[m[r]] = s[r];
        if (m[r] > 0) f[-m[r]] = sym(s[r], -m[r]);
    }
    wave_fence();
    // sum_j w^j/j! X_{n-j}^{m-j}
#pragma unroll
    for (int r = 0; r < R; ++r) {
        first[r] = n[r] * n[r] + n[r] + m[r];
        step[r] = -2 * n[r] - 1;
        last[r] = (n[r] + m[r]) / 2;
    }
    shift_sum<R>(wplus, full, nf, p, 2, first, step, last, s);
#pragma unroll
    for (int r = 0; r < R; ++r)
        if (r * FMM_WAVE + lane < nc) half[r * FMM_WAVE + lane] = s[r];
    wave_fence();
    // sum_j (-w~)^j/j! X_{n-j}^{m+j}
#pragma unroll
    for (int r = 0; r < R; ++r) {
        first[r] = tri(n[r], m[r]);
        step[r] = 1 - n[r];
        last[r] = (n[r] - m[r]) / 2;
    }
    shift_sum<R>(wminus, half, nc, p / 2, 1, first, step, last, s);
    cplx *Tc = reinterpret_cast<cplx *>(T) + (size_t)c * nc;
#pragma unroll
    for (int r = 0; r < R; ++r)
        if (r * FMM_WAVE + lane < nc)
            Tc[r * FMM_WAVE + lane] = {s[r].re, m[r] == 0 ? 0.0 : s[r].im};
}

// ---- L2L ---------------------------------------------------------------------
// F_n^m(s') += sum_{k=0}^{p-n} sum_l conj(Upsilon_k^l(s - s')) F_{n+k}^{m+l}(s),
// as three sums over degrees upwards (the parts commute; the one that raises
// the order comes last, so that the sums need orders m >= 0 only).
template <int R>
__global__ void __launch_bounds__(XF_CELLS * FMM_WAVE)
k_l2l_level(int p, TreeArrays t, int c0, int c1, double *F, const uint8_t *active) {
    extern __shared__ double lds[];
    const int w = threadIdx.x / FMM_WAVE, lane = lane_id();
    const int c = c0 + blockIdx.x * XF_CELLS + w;
    if (c >= c1) return;
    if (active && !active[c]) return;      // no listed sink below c
    const int pc = t.parent[c];
    if (pc < 0) return;
    const int nc = tri(p + 1, 0), nf = (p + 1) * (p + 1);
    cplx *half = reinterpret_cast<cplx *>(lds) + w * shift_lds_cplx(p), *full = half + nc + 1;
    const cplx *Fp = reinterpret_cast<const cplx *>(F) + (size_t)pc * nc;
    cplx *Fc = reinterpret_cast<cplx *>(F) + (size_t)c * nc;
    int n[R], m[R], first[R], step[R], last[R];
    cplx own[R], s[R];
#pragma unroll
    for (int r = 0; r < R; ++r) {
        const int e = r * FMM_WAVE + lane, ee = min(e, nc - 1);
        nm_of(ee, n[r], m[r]);
        s[r] = Fp[ee];
        own[r] = Fc[ee];
        if (e < nc) half[e] = s[r];
        last[r] = p - n[r];
    }
    if (lane == 0) half[nc] = full[nf] = {0.0, 0.0};
    const double4 ca = t.cen[pc], cb = t.cen[c];
    const cplx wp = {0.5 * (ca.x - cb.x), 0.5 * (ca.y - cb.y)};
    // conjugated weights
    const double wz = power_weight(p, ca.z - cb.z);
    const cplx wplus = power_weight(p, cplx{wp.re, -wp.im});
    const cplx wminus = power_weight(p, cplx{-wp.re, -wp.im});
    wave_fence();
#pragma unroll
    for (int r = 0; r < R; ++r) {
        first[r] = tri(n[r], m[r]);
        step[r] = n[r] + 1;
    }
    shift_sum<R>(wz, half, nc, p, 1, first, step, last, s);
#pragma unroll
    for (int r = 0; r < R; ++r) {
        if (r * FMM_WAVE + lane >= nc) continue;
        cplx *f = full + n[r] * n[r] + n[r];
        f[m[r]] = s[r];
        if (m[r] > 0) f[-m[r]] = sym(s[r], -m[r]);
    }
    wave_fence();
#pragma unroll
    for (int r = 0; r < R; ++r) {
        first[r] = n[r] * n[r] + n[r] + m[r];
        step[r] = 2 * n[r] + 1;
    }
    shift_sum<R>(wminus, full, nf, p, 2, first, step, last, s);
#pragma unroll
    for (int r = 0; r < R; ++r)
        if (r * FMM_WAVE + lane < nc) half[r * FMM_WAVE + lane] = s[r];
    wave_fence();
#pragma unroll
    for (int r = 0; r < R; ++r) {
        first[r] = tri(n[r], m[r]);
        step[r] = n[r] + 2;
    }
    shift_sum<R>(wplus, half, nc, p, 1, first, step, last, s);
#pragma unroll
    for (int r = 0; r < R; ++r)
        if (r * FMM_WAVE + lane < nc)
            Fc[r * FMM_WAVE + lane] = {own[r].re + s[r].re,
                                       m[r] == 0 ? own[r].im : own[r].im + s[r].im};
}

// ---- L2P: one thread per particle ------------------------------------------
// Psi_0^0 = sum_{k,l} conj(Upsilon_k^l(s - x)) F_k^l and
// Psi_1^m = sum_{k<=p-1,l} conj(Upsilon_k^l(s - x)) F_{k+1}^{m+l};
// a = grad Psi_0^0 = -(Re Psi_1^1, Im Psi_1^1, Psi_1^0).
template <int P>
__global__ void __launch_bounds__(256)
k_l2p(TreeArrays t, const int *leaf_of, const int *leaf_cell, int64_t n, const double *x,
      const double *y, const double *z, const double *F, double4 *out4, const uint8_t *active) {
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= n) return;
    const int c = leaf_cell[leaf_of[i]];
    if (active && !active[c]) return;      // a leaf without listed sinks
    const double4 cen = t.cen[c];
    const cplx *Fc = reinterpret_cast<const cplx *>(F) + (size_t)c * tri(P + 1, 0);
    RowGen<P> g;
    g.upsilon_start(cen.x - x[i], cen.y - y[i], cen.z - z[i]);
    double psi = 0.0;
    cplx p10 = {0.0, 0.0}, p11 = {0.0, 0.0};
    auto emit = [&]<int K>() {
        if constexpr (K > 0) g.template upsilon_row<K>();
        const cplx *u = g.template row<K>();
        // potential: Upsilon_k^0 F_k^0 + 2 sum_{l>0} Re(conj(U) F)
        {
            double s = u[0].re * Fc[tri(K, 0)].re;
#pragma unroll
            for (int l = 1; l <= K; ++l) {
                const cplx f = Fc[tri(K, l)];
                s += 2.0 * (u[l].re * f.re + u[l].im * f.im);
            }
            psi += s;
        }
        if constexpr (K < P) {
#pragma unroll
            for (int l = -K; l <= K; ++l) {
                const cplx ul = sym(u[l < 0 ? -l : l], l);
                const cplx cu = {ul.re, -ul.im};
                const cplx f0 = ld(Fc, K + 1, l), f1 = ld(Fc, K + 1, l + 1);
                p10 = cadd(p10, cmul(cu, f0));
                p11 = cadd(p11, cmul(cu, f1));
            }
        }
    };
    Unroll<0, P>::run(emit);
    out4[i] = make_double4(psi, -p11.re, -p11.im, -p10.re);
}

// ---- low-order estimate (p = 1 at the centre of mass, or the 1/r^2 monopole) --
// Fe = (Psi, F_1^0, Re F_1^1, Im F_1^1); for f only .x is used.  One wavefront
// per sink cell: lane j adds entries j, j + 64, ... of the cell's list, then
// the lanes are added in a fixed butterfly order (deterministic).
__global__ void __launch_bounds__(256)
k_est_m2l(int want_f, TreeArrays t, int nsinks, const int64_t *off, const uint64_t *list, int sh,
          double4 *Fe) {
    const int b = blockIdx.x * 4 + threadIdx.x / FMM_WAVE;
    if (b >= nsinks) return;
    const int lane = lane_id();
    const int64_t e0 = off[b], e1 = off[b + 1];
    const double4 sb = t.com[b];
    const uint64_t mask = (1ull << sh) - 1;
    double f0 = 0.0, f10 = 0.0, f11r = 0.0, f11i = 0.0;
    for (int64_t e = e0 + lane; e < e1; e += FMM_WAVE) {
        const int a = (int)(list[e] & mask);
        const double4 za = t.com[a];
        const double M = t.mass[a];
        const double dx = sb.x - za.x, dy = sb.y - za.y, dz = sb.z - za.z;
        const double r2 = fma(dx, dx, fma(dy, dy, dz * dz));
        if (want_f) {
            f0 += M / r2;
        } else {
            const double ri = rsqrt_nr(r2);
            const double q = M * ri, q3 = q * ri * ri;
            f0 += q;                       // M Theta_0^0
            f10 = fma(q3, dz, f10);        // M Theta_1^0 = M z / r^3
            f11r = fma(q3, dx, f11r);      // M Theta_1^1 = M (x + i y) / r^3
            f11i = fma(q3, dy, f11i);
        }
    }
    f0 = wave_sum(f0);
    f10 = wave_sum(f10);
    f11r = wave_sum(f11r);
    f11i = wave_sum(f11i);
    if (lane == 0) Fe[b] = make_double4(f0, f10, f11r, f11i);
}

// p = 1 shift: F_1^m is unchanged and F_0^0 is not needed for |a|, so a leaf's
// far field is the sum over its chain of ancestors, the same at every particle.
// EST_G lanes per leaf follow the chain together (one launch where a level by
// level pass takes one per level) and write its particles.
constexpr int EST_G = 16;
__global__ void __launch_bounds__(256)
k_est_down(int want_f, TreeArrays t, const int *leaf_cell, int nleaves, const double4 *Fe,
           double4 *out4) {
    const int64_t gt = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (gt / EST_G >= nleaves) return;
    const int c = leaf_cell[gt / EST_G];
    double4 f = Fe[c];
    for (int a = t.parent[c]; a >= 0; a = t.parent[a]) {
        const double4 v = Fe[a];
        f.x += v.x; f.y += v.y; f.z += v.z; f.w += v.w;
    }
    const double4 o = want_f ? make_double4(f.x, 0.0, 0.0, 0.0)
                             : make_double4(0.0, -f.z, -f.w, -f.y);
    const int e = t.end[c];
    for (int i = t.beg[c] + (int)(gt % EST_G); i < e; i += EST_G) out4[i] = o;
}

inline unsigned blocks(int64_t n, int b) { return (unsigned)((n + b - 1) / b); }

#define FMM_DISPATCH_P(p, CALL)                                                        \
    switch (p) {                                                                       \
    case 1: CALL(1); break;   case 2: CALL(2); break;   case 3: CALL(3); break;         \
    case 4: CALL(4); break;   case 5: CALL(5); break;   case 6: CALL(6); break;         \
    case 7: CALL(7); break;   case 8: CALL(8); break;   case 9: CALL(9); break;         \
    case 10: CALL(10); break; case 11: CALL(11); break; case 12: CALL(12); break;       \
    case 13: CALL(13); break; case 14: CALL(14); break; case 15: CALL(15); break;       \
    case 16: CALL(16); break; case 17: CALL(17); break; case 18: CALL(18); break;       \
    case 19: CALL(19); break; case 20: CALL(20); break;                                 \
    default: return hipErrorInvalidValue;                                              \
    }

}  // namespace

hipError_t launch_p2m(int p, const TreeArrays &t, const int *leaf_cell, int nleaves,
                      const double *x, const double *y, const double *z, const double *m,
                      double *M, hipStream_t s) {
    if (nleaves <= 0) return hipSuccess;
#define CALL(P) hipLaunchKernelGGL(k_p2m<P>, dim3(blocks(nleaves, 4)), dim3(256), 0, s, t, \
                                   leaf_cell, nleaves, x, y, z, m, M)
    FMM_DISPATCH_P(p, CALL)
#undef CALL
    return hipGetLastError();
}

// coefficients per lane of a wavefront: 1 up to p = 9, 2 up to 14, 3 up to 18
#define FMM_DISPATCH_R(p, CALL)                                 \
    switch ((ncplx(p) + FMM_WAVE - 1) / FMM_WAVE) {             \
    case 1: CALL(1); break;   case 2: CALL(2); break;           \
    case 3: CALL(3); break;   case 4: CALL(4); break;           \
    default: return hipErrorInvalidValue;                       \
    }

hipError_t launch_m2m_level(int p, const TreeArrays &t, int c0, int c1, double *M, double *T,
                            double *P, hipStream_t s) {
    if (c1 <= c0) return hipSuccess;
    Binomials b;
    b.v[0] = 1.0;
    for (int k = 1; k <= p; ++k) b.v[k] = b.v[k - 1] * (double)(p - k + 1) / (double)k;
#define CALL(R)                                                                                \
    hipLaunchKernelGGL(k_m2m_level<R>, dim3(blocks(c1 - c0, XF_CELLS)),                        \
                       dim3(XF_CELLS * FMM_WAVE), XF_CELLS * shift_lds_cplx(p) * sizeof(cplx), \
                       s, p, t, c0, c1, M, T, b, P)
    FMM_DISPATCH_R(p, CALL)
#undef CALL
    return hipGetLastError();
}

hipError_t launch_l2l_level(int p, const TreeArrays &t, int c0, int c1, double *F,
                            const uint8_t *active, hipStream_t s) {
    if (c1 <= c0) return hipSuccess;
#define CALL(R)                                                                                \
    hipLaunchKernelGGL(k_l2l_level<R>, dim3(blocks(c1 - c0, XF_CELLS)),                        \
                       dim3(XF_CELLS * FMM_WAVE), XF_CELLS * shift_lds_cplx(p) * sizeof(cplx), \
                       s, p, t, c0, c1, F, active)
    FMM_DISPATCH_R(p, CALL)
#undef CALL
    return hipGetLastError();
}

hipError_t launch_l2p(int p, const TreeArrays &t, const int *leaf_of, const int *leaf_cell,
                      int64_t n, const double *x, const double *y, const double *z,
                      const double *F, double4 *out4, hipStream_t s, const uint8_t *active) {
#define CALL(P) hipLaunchKernelGGL(k_l2p<P>, dim3(blocks(n, 256)), dim3(256), 0, s, t, leaf_of, \
                                   leaf_cell, n, x, y, z, F, out4, active)
    FMM_DISPATCH_P(p, CALL)
#undef CALL
    return hipGetLastError();
}

hipError_t launch_est_m2l(int want_f, const TreeArrays &t, int nsinks, const int64_t *off,
                          const uint64_t *list, int sh, double4 *Fe, hipStream_t s) {
    hipLaunchKernelGGL(k_est_m2l, dim3(blocks(nsinks, 4)), dim3(256), 0, s, want_f, t, nsinks,
                       off, list, sh, Fe);
    return hipGetLastError();
}

hipError_t launch_est_down(int want_f, const TreeArrays &t, const int *leaf_cell, int nleaves,
                           const double4 *Fe, double4 *out4, hipStream_t s) {
    hipLaunchKernelGGL(k_est_down, dim3(blocks((int64_t)nleaves * EST_G, 256)), dim3(256), 0, s,
                       want_f, t, leaf_cell, nleaves, Fe, out4);
    return hipGetLastError();
}

}  // namespace fmm
