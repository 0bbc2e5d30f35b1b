// Jerk kernels (Sec. 7, jerk; eqs:fmm:dot).
//
// Rates of the regular harmonics for dr/dt = v (App. A.5): in the variables
// xi = (x+iy)/2, eta = -(x-iy)/2 (eq:xi:eta) and z, eq:dUnm gives
// d/dxi Upsilon_n^m = Upsilon_{n-1}^{m-1}, d/deta Upsilon_n^m = Upsilon_{n-1}^{m+1}
// and d/dz Upsilon_n^m = Upsilon_{n-1}^m, so
//   d/dt Upsilon_n^m = xidot Upsilon_{n-1}^{m-1} + vz Upsilon_{n-1}^m
//                      + etadot Upsilon_{n-1}^{m+1},
// xidot = (vx + i vy)/2, etadot = -(vx - i vy)/2 (Upsilon_1^1 = xi has rate
// xidot, which fixes the pairing of xidot with m-1).  Every rate of degree n
// is a combination of degree n-1 harmonics, so the P2M and L2P kernels form
// the rates from the row or column they already generate.
#include "jerk.h"
#include "harmonics.h"
#include "near.h"
#include "p2m_impl.h"

namespace fmm {

namespace {

inline unsigned blocks(int64_t n, int b) { return (unsigned)((n + b - 1) / b); }

// xidot X + etadot Y for the velocity (vx, vy)
__device__ __forceinline__ cplx rate_xy(double vx, double vy, cplx X, cplx Y) {
    // (vx + i vy)/2 X - (vx - i vy)/2 Y
    return {0.5 * (vx * (X.re - Y.re) - vy * (X.im + Y.im)),
            0.5 * (vx * (X.im - Y.im) + vy * (X.re + Y.re))};
}

// ---- gather -----------------------------------------------------------------
__global__ void k_gather_vel(int64_t n, const uint32_t *perm, const double *vel, double4 *v4) {
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= n) return;
    const int64_t j = perm[i];
    v4[i] = make_double4(vel[3 * j], vel[3 * j + 1], vel[3 * j + 2], 0.0);
}

// ---- P2M rates: one wavefront per leaf ------------------------------------------
// d/dt Upsilon_n^m(x) = xidot Upsilon_{n-1}^{m-1} + etadot Upsilon_{n-1}^{m+1}
// + zdot Upsilon_{n-1}^m is linear in the velocity, so the rates are P2M of degree
// P - 1 three times, weighted by mu v_x, mu v_y and mu v_z, into LDS, and one
// combination per coefficient (xidot = (v_x + i v_y)/2, etadot = -(v_x - i v_y)/2).
// 2 x 10^5 bodies, p = 15: 134 us; with neighbouring columns exchanged for every
// particle and degree, at one wavefront per SIMD, 400 us.
template <int P>
__global__ void __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(P <= 15 ? 3 : 2)))
k_p2m_dot(TreeArrays t, const int *leaf_cell, int nleaves, const double *x, const double *y,
          const double *z, const double *m, const double4 *v4, double *Md) {
    typedef P2MLeaf<P - 1> Leaf;
    constexpr int NC = tri(P, 0);              // coefficients up to degree P - 1
    __shared__ typename Leaf::Steps step;
    __shared__ double mom[4][3][2 * NC];
    Leaf::fill(step);
    const int w = threadIdx.x / FMM_WAVE, leaf = blockIdx.x * 4 + w;
    if (leaf >= nleaves) return;               // whole wavefronts leave together
    const int c = leaf_cell[leaf];
    const int beg = t.beg[c], end = t.end[c];
    const double4 cen = t.cen[c];
    const double *vel = reinterpret_cast<const double *>(v4);
    for (int d = 0; d < 3; ++d)
        Leaf::run(step, beg, end, cen, x, y, z, [&](int i) { return m[i] * vel[4 * (size_t)i + d]; },
                  [&](int n, int col, int half, double v) {
                      mom[w][d][2 * tri(n, col) + half] = v;
                  });
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    __builtin_amdgcn_wave_barrier();
    const cplx *X = reinterpret_cast<const cplx *>(mom[w][0]),
               *Y = reinterpret_cast<const cplx *>(mom[w][1]),
               *Z = reinterpret_cast<const cplx *>(mom[w][2]);
    // coefficient (n, q) of a set of moments, 0 beyond its orders
    auto at = [](const cplx *A, int n, int q) {
        const int a = q < 0 ? -q : q;
        return a <= n ? sym(A[tri(n, a)], q) : cplx{0.0, 0.0};
    };
    cplx *Mc = reinterpret_cast<cplx *>(Md) + (size_t)c * tri(P + 1, 0);
    for (int e = lane_id(); e < tri(P + 1, 0); e += FMM_WAVE) {
        int n = (int)((sqrtf(8.0f * (float)e + 1.0f) - 1.0f) * 0.5f);
        if (tri(n + 1, 0) <= e) ++n;
        if (tri(n, 0) > e) --n;
        const int q = e - tri(n, 0);
        cplx r = {0.0, 0.0};
        if (n > 0) {
            const cplx xl = at(X, n - 1, q - 1), xr = at(X, n - 1, q + 1);
            const cplx yl = at(Y, n - 1, q - 1), yr = at(Y, n - 1, q + 1);
            const cplx zz = at(Z, n - 1, q);
            r = {0.5 * ((xl.re - yl.im) - (xr.re + yr.im)) + zz.re,
                 0.5 * ((xl.im + yl.re) - (xr.im - yr.re)) + zz.im};
        }
        Mc[e] = {r.re, q == 0 ? 0.0 : r.im};
    }
}

// ---- L2P rates: one thread per particle --------------------------------------
// Psidot_1^m = sum_{k <= p-1, l} [conj(Upsilon_k^l(s - x)) Fdot_{k+1}^{m+l}
//              + conj(d/dt Upsilon_k^l(s - x)) F_{k+1}^{m+l}], d(s - x)/dt = -v,
// jerk = -(Re Psidot_1^1, Im Psidot_1^1, Psidot_1^0).  Rows of Upsilon come
// one degree at a time; row k's rates use row k-1, which the generator still
// holds.
__device__ __forceinline__ cplx ldc(const cplx *X, int n, int q) {
    return sym(X[tri(n, q < 0 ? -q : q)], q);
}

template <int P>
__global__ void __launch_bounds__(256)
k_l2p_dot(TreeArrays t, const int *leaf_of, const int *leaf_cell, int64_t n, const double *x,
          const double *y, const double *z, const double4 *v4, const double *F,
          const double *Fd, double4 *jo4, const uint8_t *active) {
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= n) return;
    const int c = leaf_cell[leaf_of[i]];
    if (active && !active[c]) return;      // a leaf without listed sinks
    const double4 cen = t.cen[c];
    const cplx *Fc = reinterpret_cast<const cplx *>(F) + (size_t)c * tri(P + 1, 0);
    const cplx *Gc = reinterpret_cast<const cplx *>(Fd) + (size_t)c * tri(P + 1, 0);
    const double4 v = v4[i];
    const double wx = -v.x, wy = -v.y, wz = -v.z;   // rate of s - x
    RowGen<P> g;
    g.upsilon_start(cen.x - x[i], cen.y - y[i], cen.z - z[i]);
    cplx p10 = {0.0, 0.0}, p11 = {0.0, 0.0};
    auto emit = [&]<int K>() {
        if constexpr (K > 0) g.template upsilon_row<K>();
        const cplx *u = g.template row<K>();
#pragma unroll
        for (int l = -K; l <= K; ++l) {
            const cplx ul = sym(u[l < 0 ? -l : l], l);
            const cplx cu = {ul.re, -ul.im};
            p10 = cadd(p10, cmul(cu, ldc(Gc, K + 1, l)));
            p11 = cadd(p11, cmul(cu, ldc(Gc, K + 1, l + 1)));
        }
        if constexpr (K > 0) {
            const cplx *w = g.template row<K - 1>();
#pragma unroll
            for (int l = -K; l <= K; ++l) {
                const int a = l - 1, b = l + 1;     // columns of degree K-1
                const cplx X = (a >= -(K - 1) && a <= K - 1) ? sym(w[a < 0 ? -a : a], a)
                                                             : cplx{0.0, 0.0};
                const cplx Y = (b >= -(K - 1) && b <= K - 1) ? sym(w[b < 0 ? -b : b], b)
                                                             : cplx{0.0, 0.0};
                const cplx Z = (l >= -(K - 1) && l <= K - 1) ? sym(w[l < 0 ? -l : l], l)
                                                             : cplx{0.0, 0.0};
                const cplx r = rate_xy(wx, wy, X, Y);
                const cplx ud = {fma(wz, Z.re, r.re), fma(wz, Z.im, r.im)};
                const cplx cud = {ud.re, -ud.im};
                p10 = cadd(p10, cmul(cud, ldc(Fc, K + 1, l)));
                p11 = cadd(p11, cmul(cud, ldc(Fc, K + 1, l + 1)));
            }
        }
    };
    Unroll<0, P - 1>::run(emit);
    jo4[i] = make_double4(0.0, -p11.re, -p11.im, -p10.re);
}

// ---- near field: potential, acceleration and jerk in one pass ---------------
// d/dt [mu (x_a - x_b)/r^3] = mu [v_ab/r^3 - 3 (r . v_ab) r/r^5],
// r = x_a - x_b, v_ab = v_a - v_b.  Same slices, lanes and summation order as
// the force-only FP64 direct sums (near.h), so the potential and acceleration
// are bit for bit those of the force-only call; the jerk reuses each pair's
// separation and 1/r^3.
//
// Summed with 2/|r| in place of 1/|r|, as the force-only direct sums are:
// potential times 2, acceleration and jerk times 8, scaled back once per sink.
constexpr double JERK_POT_BACK = 0.5, JERK_ACC_BACK = 0.125;

struct Moving {
    double4 x, v;            // position and mass, velocity
};

struct SinkSum {
    double pot, ax, ay, az, jx, jy, jz;
};

__device__ __forceinline__ void pair_jerk(const Moving &s, double xb, double yb, double zb,
                                          double ub, double vb, double wb, bool skip,
                                          SinkSum &k) {
    const double dx = s.x.x - xb, dy = s.x.y - yb, dz = s.x.z - zb;
    const double r2 = skip ? 1.0 : fma(dx, dx, fma(dy, dy, dz * dz));
    const double mu = skip ? 0.0 : s.x.w;
    const double ri = rsqrt2_nr(r2);            // 2/|r|
    const double q = mu * ri;
    const double q3 = q * ri * ri;
    k.pot += q;
    k.ax = fma(q3, dx, k.ax);
    k.ay = fma(q3, dy, k.ay);
    k.az = fma(q3, dz, k.az);
    const double ux = s.v.x - ub, uy = s.v.y - vb, uz = s.v.z - wb;
    // 3 (r.u)/r^2 = 0.75 (r.u) (2/|r|)^2
    const double rv = 0.75 * fma(dx, ux, fma(dy, uy, dz * uz)) * (ri * ri);
    k.jx = fma(q3, fma(-rv, dx, ux), k.jx);
    k.jy = fma(q3, fma(-rv, dy, uy), k.jy);
    k.jz = fma(q3, fma(-rv, dz, uz), k.jz);
}

template <int R>
__device__ __forceinline__ void near_jerk(const NearTask &q, const int2 *entry,
                                          const double4 *xyzm, const double4 *v4, double4 *out4,
                                          double4 *jo4, double4 *row, double4 *jrow) {
    const int lane = lane_id();
    const double4 mx = xyzm[q.sb + (lane < R ? lane : 0)];
    const double4 mv = v4[q.sb + (lane < R ? lane : 0)];
    double sx[R], sy[R], sz[R], su[R], sv[R], sw[R];
    SinkSum f[R];
#pragma unroll
    for (int k = 0; k < R; ++k) {
        sx[k] = readlane_f64(mx.x, k);
        sy[k] = readlane_f64(mx.y, k);
        sz[k] = readlane_f64(mx.z, k);
        su[k] = readlane_f64(mv.x, k);
        sv[k] = readlane_f64(mv.y, k);
        sw[k] = readlane_f64(mv.z, k);
        f[k] = {0.0, 0.0, 0.0, 0.0, 0.0, 0.0, 0.0};
    }
    near_sources(
        entry, q, [&](uint32_t i) { return Moving{load32(xyzm, i), load32(v4, i)}; },
        [&](const Moving &a) {
#pragma unroll
            for (int k = 0; k < R; ++k) {
                pair_jerk(a, sx[k], sy[k], sz[k], su[k], sv[k], sw[k], false, f[k]);
                if (k % 2 == 1) __builtin_amdgcn_sched_barrier(0);
            }
        },
        [&](Moving a, uint32_t i, bool on) {
            if (!on) a.x = a.v = make_double4(0.0, 0.0, 0.0, 0.0);
#pragma unroll
            for (int k = 0; k < R; ++k) {
                pair_jerk(a, sx[k], sy[k], sz[k], su[k], sv[k], sw[k],
                          !on || i == (uint32_t)(q.sb + k), f[k]);
                __builtin_amdgcn_sched_barrier(0);
            }
        });
    // lane i of each row of 16 lanes takes one component of sink i
    double v = 0.0, vj = 0.0;
#pragma unroll
    for (int k = 0; k < R; ++k) {
        const double w = wave_sum4(f[k].pot, f[k].ax, f[k].ay, f[k].az);
        const double wj = wave_sum4(0.0, f[k].jx, f[k].jy, f[k].jz);
        v = (lane & 15) == k ? w : v;
        vj = (lane & 15) == k ? wj : vj;
    }
    const int comp = wave_sum4_component(), s = lane & 15;
    v *= comp == 0 ? JERK_POT_BACK : JERK_ACC_BACK;
    vj *= JERK_ACC_BACK;
    if (s >= R) return;
    if (q.single) {
        reinterpret_cast<double *>(out4 + q.sb + s)[comp] += v;
        reinterpret_cast<double *>(jo4 + q.sb + s)[comp] += vj;
    } else {
        reinterpret_cast<double *>(row + s)[comp] = v;
        reinterpret_cast<double *>(jrow + s)[comp] = vj;
    }
}

__global__ void __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(3)))
k_p2p_jerk(int ntasks, const int4 *tasks, const int2 *entry, const double4 *xyzm,
           const double4 *v4, double4 *out4, double4 *jo4, double4 *partial, double4 *jpartial) {
    const int task = blockIdx.x * 4 + threadIdx.x / FMM_WAVE;
    if (task >= ntasks) return;                // whole wavefronts leave together
    const NearTask q = unpack_task(tasks[task]);
    double4 *row = partial + (size_t)task * NEAR_JERK_R;
    double4 *jrow = jpartial + (size_t)task * NEAR_JERK_R;
    static_assert(NEAR_JERK_R == 6, "the cases below");
#define FMM_NEAR(R) case R: near_jerk<R>(q, entry, xyzm, v4, out4, jo4, row, jrow); break
    switch (q.r) {
        FMM_NEAR(1); FMM_NEAR(2); FMM_NEAR(3); FMM_NEAR(4); FMM_NEAR(5); FMM_NEAR(6);
    }
#undef FMM_NEAR
}

// listed sinks: jerk[3 j + d] = G (far4 + jo4)[inv[act[j]]].(y, z, w) (indices out of
// range are skipped; the caller reports them)
__global__ void k_output_jerk_listed(int64_t n, int64_t nact, const int64_t *act, const int *inv,
                                     const double4 *far4, const double4 *jo4, double G,
                                     double *jerk, int *nonfinite) {
    const int64_t j = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (j >= nact) return;
    const int64_t idx = act[j];
    if (idx < 0 || idx >= n) return;
    const double4 f = far4[inv[idx]], v = jo4[inv[idx]];
    const double a = G * (f.y + v.y), b = G * (f.z + v.z), c = G * (f.w + v.w);
    jerk[3 * j] = a;
    jerk[3 * j + 1] = b;
    jerk[3 * j + 2] = c;
    if (!(isfinite(a) && isfinite(b) && isfinite(c))) atomicOr(nonfinite, 1);
}

__global__ void k_output_jerk(int64_t n, const uint32_t *perm, const double4 *far4,
                              const double4 *jo4, double G, double *jerk, int *nonfinite) {
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= n) return;
    const double4 f = far4[i], v = jo4[i];
    const int64_t j = perm[i];
    const double a = G * (f.y + v.y), b = G * (f.z + v.z), c = G * (f.w + v.w);
    jerk[3 * j] = a;
    jerk[3 * j + 1] = b;
    jerk[3 * j + 2] = c;
    if (!(isfinite(a) && isfinite(b) && isfinite(c))) atomicOr(nonfinite, 1);
}

// exact jerk of listed sinks against all n sources, as the exact forces are
// summed (DIRECT_R sinks per wavefront, the sources cut into chunks whose rows
// of part are added in order); *bad = 1 for an index outside [0, n).  2048
// sinks of 10^6: 2.2 ms; one thread per sink against all sources, on 8 compute
// units, took 211 ms.
__global__ void __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(3)))
k_direct_jerk_sinks(int64_t n, const double *pos, const double *vel, const double *mass,
                    double G, int64_t nsinks, const int64_t *sinks, int64_t chunk, double *jerk,
                    double4 *part, int *bad) {
    const int64_t wave = (int64_t)blockIdx.x * 4 + threadIdx.x / FMM_WAVE;
    if (wave * DIRECT_R >= nsinks) return;     // whole wavefronts leave together
    const int k = blockIdx.y, lane = lane_id();
    const DirectSinks d = direct_sinks(wave, n, nsinks, sinks, k == 0 ? bad : nullptr);
    double sx[DIRECT_R], sy[DIRECT_R], sz[DIRECT_R], su[DIRECT_R], sv[DIRECT_R], sw[DIRECT_R];
    double f[DIRECT_R][3];
#pragma unroll
    for (int q = 0; q < DIRECT_R; ++q) {
        const double *x = pos + 3 * d.idx[q], *v = vel + 3 * d.idx[q];
        sx[q] = readlane_f64(x[0], 0);
        sy[q] = readlane_f64(x[1], 0);
        sz[q] = readlane_f64(x[2], 0);
        su[q] = readlane_f64(v[0], 0);
        sv[q] = readlane_f64(v[1], 0);
        sw[q] = readlane_f64(v[2], 0);
        f[q][0] = f[q][1] = f[q][2] = 0.0;
    }
    const int64_t j0 = (int64_t)k * chunk, j1 = min(n, j0 + chunk);
    const double *px = pos + 3 * j0, *pv = vel + 3 * j0, *pm = mass + j0;
    auto source = [&](uint32_t o) {
        const size_t i = 3 * (size_t)o;
        return Moving{make_double4(px[i], px[i + 1], px[i + 2], pm[o]),
                      make_double4(pv[i], pv[i + 1], pv[i + 2], 0.0)};
    };
    auto add = [&](const Moving &a, int q, bool skip) {
        SinkSum s = {0.0, 0.0, 0.0, 0.0, f[q][0], f[q][1], f[q][2]};
        pair_jerk(a, sx[q], sy[q], sz[q], su[q], sv[q], sw[q], skip, s);
        f[q][0] = s.jx;
        f[q][1] = s.jy;
        f[q][2] = s.jz;
    };
    direct_steps(
        d, j0, j1,
        [&](uint32_t o) {
            const Moving a = source(o);
#pragma unroll
            for (int q = 0; q < DIRECT_R; ++q) {
                add(a, q, false);
                if (q % 2 == 1) __builtin_amdgcn_sched_barrier(0);
            }
        },
        [&](uint32_t o, bool on) {
            Moving a{make_double4(0.0, 0.0, 0.0, 0.0), make_double4(0.0, 0.0, 0.0, 0.0)};
            if (on) a = source(o);
#pragma unroll
            for (int q = 0; q < DIRECT_R; ++q) {
                add(a, q, !on || j0 + o == d.idx[q]);
                __builtin_amdgcn_sched_barrier(0);
            }
        });
    double v = 0.0;
#pragma unroll
    for (int q = 0; q < DIRECT_R; ++q) {
        const double w = wave_sum4(0.0, f[q][0], f[q][1], f[q][2]);
        v = (lane & 15) == q ? w : v;
    }
    const int comp = wave_sum4_component(), s = lane & 15;
    if (s >= DIRECT_R || !((d.valid >> s) & 1u)) return;
    v *= JERK_ACC_BACK;
    const int64_t t = d.t0 + s;
    if (part) reinterpret_cast<double *>(part + (int64_t)k * nsinks + t)[comp] = v;
    else if (comp > 0) jerk[3 * t + comp - 1] = G * v;
}

__global__ void k_direct_jerk_reduce(int64_t n, double G, int64_t nsinks, const int64_t *sinks,
                                     int nchunk, const double4 *part, double *jerk) {
    const int64_t t = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (t >= nsinks) return;
    const int64_t ii = sinks[t];
    if (ii < 0 || ii >= n) return;
    double4 v = part[t];
    for (int k = 1; k < nchunk; ++k) {
        const double4 q = part[(int64_t)k * nsinks + t];
        v.y += q.y; v.z += q.z; v.w += q.w;
    }
    jerk[3 * t] = G * v.y;
    jerk[3 * t + 1] = G * v.z;
    jerk[3 * t + 2] = G * v.w;
}

#define FMM_JERK_DISPATCH_P(p, CALL)                                                   \
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

hipError_t launch_gather_vel(int64_t n, const uint32_t *perm, const double *vel, double4 *v4,
                             hipStream_t s) {
    if (n <= 0) return hipSuccess;
    hipLaunchKernelGGL(k_gather_vel, dim3(blocks(n, 256)), dim3(256), 0, s, n, perm, vel, v4);
    return hipGetLastError();
}

hipError_t launch_p2m_dot(int p, const TreeArrays &t, const int *leaf_cell, int nleaves,
                          const double *x, const double *y, const double *z, const double *m,
                          const double4 *v4, double *Md, hipStream_t s) {
    if (nleaves <= 0) return hipSuccess;
#define CALL(P) hipLaunchKernelGGL(k_p2m_dot<P>, dim3(blocks(nleaves, 4)), dim3(256), 0, s, t, \
                                   leaf_cell, nleaves, x, y, z, m, v4, Md)
    FMM_JERK_DISPATCH_P(p, CALL)
#undef CALL
    return hipGetLastError();
}

hipError_t launch_l2p_dot(int p, const TreeArrays &t, const int *leaf_of, const int *leaf_cell,
                          int64_t n, const double *x, const double *y, const double *z,
                          const double4 *v4, const double *F, const double *Fd, double4 *jo4,
                          hipStream_t s, const uint8_t *active) {
    if (n <= 0) return hipSuccess;
#define CALL(P) hipLaunchKernelGGL(k_l2p_dot<P>, dim3(blocks(n, 256)), dim3(256), 0, s, t,   \
                                   leaf_of, leaf_cell, n, x, y, z, v4, F, Fd, jo4, active)
    FMM_JERK_DISPATCH_P(p, CALL)
#undef CALL
    return hipGetLastError();
}

hipError_t launch_p2p_jerk(int ntasks, const int4 *tasks, const int2 *entry,
                           const double4 *xyzm, const double4 *v4, double4 *out4, double4 *jo4,
                           double4 *partial, double4 *jpartial, hipStream_t s) {
    if (ntasks <= 0) return hipSuccess;
    hipLaunchKernelGGL(k_p2p_jerk, dim3(blocks(ntasks, 4)), dim3(256), 0, s, ntasks, tasks, entry,
                       xyzm, v4, out4, jo4, partial, jpartial);
    return hipGetLastError();
}

hipError_t launch_direct_jerk_sinks(int64_t n, const double *pos, const double *vel,
                                   const double *mass, double G, int64_t nsinks,
                                   const int64_t *sinks, int nchunk, double *jerk, double4 *part,
                                   int *bad, hipStream_t s) {
    if (nsinks <= 0) return hipSuccess;
    if (nchunk < 1 || (nchunk > 1 && !part)) return hipErrorInvalidValue;
    const int64_t chunk = row_length(n, nchunk);
    hipLaunchKernelGGL(k_direct_jerk_sinks, dim3(blocks(nsinks, 4 * DIRECT_R), (unsigned)nchunk),
                       dim3(256), 0, s, n, pos, vel, mass, G, nsinks, sinks, chunk, jerk,
                       nchunk > 1 ? part : nullptr, bad);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess || nchunk == 1) return e;
    hipLaunchKernelGGL(k_direct_jerk_reduce, dim3(blocks(nsinks, 256)), dim3(256), 0, s, n, G,
                       nsinks, sinks, nchunk, (const double4 *)part, jerk);
    return hipGetLastError();
}

hipError_t launch_output_jerk_listed(int64_t n, int64_t nact, const int64_t *act, const int *inv,
                                     const double4 *far4, const double4 *jo4, double G,
                                     double *jerk, int *nonfinite,
                                     hipStream_t s) {
    if (nact <= 0) return hipSuccess;
    hipLaunchKernelGGL(k_output_jerk_listed, dim3(blocks(nact, 256)), dim3(256), 0, s, n, nact, act,
                       inv, far4, jo4, G, jerk, nonfinite);
    return hipGetLastError();
}

hipError_t launch_output_jerk(int64_t n, const uint32_t *perm, const double4 *far4,
                              const double4 *jo4, double G, double *jerk, int *nonfinite, hipStream_t s) {
    if (n <= 0) return hipSuccess;
    hipLaunchKernelGGL(k_output_jerk, dim3(blocks(n, 256)), dim3(256), 0, s, n, perm, far4, jo4, G,
                       jerk, nonfinite);
    return hipGetLastError();
}

}  // namespace fmm
