// Direct sums: the near field (P2P, eq. 1 restricted to the walk's direct
// pairs), the all-pairs GPU direct summation used as a comparison baseline,
// and the final un-permute / scale / finiteness check.
//
// P2P: the sources of a sink leaf are the merged particle ranges listed for
// the leaf and for each of its ancestors (a direct sum accepted for a cell
// applies to all particles below it).  A leaf's work is cut into tasks of a few
// sinks x P2P_TASK sources - a sparse leaf far out in an untruncated halo can
// be summed against every particle, and as one wavefront's serial loop it
// would set the kernel time; short tasks also even out the load of the compute
// units at the end of a launch.  One wavefront per task.  FP64 sums hold up to
// NEAR_R sinks in scalar registers and one source per lane (near.h).
// Mixed-precision sums hold up to 64 sinks of a leaf, two per lane, lanes being
// (sink group, phase) pairs that stride through each range; the phases are
// summed through LDS at the end.  A leaf with one task adds into the output
// directly; otherwise each task writes a row of partial sums that a second
// kernel adds in task order (deterministic).
// Source particles are read as (x, y, z, m) double4 from the key-sorted copy.
#include <algorithm>

#include "internal.h"
#include "dev.h"
#include "near.h"
#include "range_loads.h"

namespace fmm {

namespace {

// sinks per lane of the mixed-precision kernel (two halves the source loads
// per pair; more costs occupancy)
constexpr int P2P_R = 2;

// up[c] = the nearest proper ancestor of c that has direct-sum ranges (or -1),
// so that a leaf visits only the cells of its chain that hold work instead of
// every ancestor (each step is a dependent load).
__global__ void k_range_up(int ncells, const int *parent, const int64_t *off, int *up) {
    const int c = blockIdx.x * blockDim.x + threadIdx.x;
    if (c >= ncells) return;
    int a = parent[c];
    while (a >= 0 && off[a + 1] == off[a]) a = parent[a];
    up[c] = a;
}

__device__ __forceinline__ int first_with_ranges(int c, const int *up, const int64_t *off) {
    return off[c + 1] > off[c] ? c : up[c];
}

// Work of one sink leaf: the number of source particles in its direct-sum
// ranges and those of its ancestors (one concatenated list); every lane of
// the wavefront ends with it.  Lanes take the range entries in turn.
__device__ __forceinline__ int64_t leaf_sources(int c, const int *up, const int64_t *off,
                                                const int2 *range) {
    int64_t s = 0;
    for (int anc = first_with_ranges(c, up, off); anc >= 0; anc = up[anc])
        for (int64_t r = off[anc] + lane_id(); r < off[anc + 1]; r += FMM_WAVE)
            s += range[r].y - range[r].x;
#pragma unroll
    for (int o = FMM_WAVE / 2; o > 0; o >>= 1) s += __shfl_xor(s, o, FMM_WAVE);
    return s;
}

// plan of the mixed-precision sums, per leaf (one wavefront each): tasks = sink
// chunks of 64 x source chunks of P2P_TASK sources; mtask = tasks that need a partial-sum row (leaves with
// more than one task) (active: when not null, leaves whose cell holds no
// listed sink get no task); entry nleaves is zeroed for the scans.  Also the
// leaf's chain of ancestors with ranges, so that the direct-sum tasks load it
// at once instead of following it one dependent load at a time.
__global__ void k_p2p_count(int nleaves, const int *leaf_cell, const int64_t *off,
                            const int2 *range, const int *up, TreeArrays t,
                            const uint8_t *active, int *ntask, int *mtask, int *nsrc_tasks,
                            int *chain) {
    const int leaf = (int)(((int64_t)blockIdx.x * blockDim.x + threadIdx.x) / FMM_WAVE);
    if (leaf > nleaves) return;
    const bool head = lane_id() == 0;
    if (leaf == nleaves) {
        if (head) {
            ntask[leaf] = 0;
            mtask[leaf] = 0;
        }
        return;
    }
    const int c = leaf_cell[leaf];
    int *ch = chain + (size_t)leaf * P2P_CHAIN;
    if (active && !active[c]) {
        if (head) {
            nsrc_tasks[leaf] = 1;
            ntask[leaf] = 0;
            mtask[leaf] = 0;
            ch[0] = 0;
        }
        return;
    }
    if (head) {
        int k = 0;
        for (int anc = first_with_ranges(c, up, off); anc >= 0; anc = up[anc]) ch[1 + k++] = anc;
        ch[0] = k;
    }
    const int64_t S = leaf_sources(c, up, off, range);
    if (!head) return;
    const int nsc = (t.end[c] - t.beg[c] + FMM_WAVE - 1) / FMM_WAVE;
    const int nts = (int)max((int64_t)1, (S + P2P_TASK - 1) / P2P_TASK);
    nsrc_tasks[leaf] = nts;
    ntask[leaf] = nsc * nts;
    mtask[leaf] = nsc * nts > 1 ? nsc * nts : 0;
}

// the task list: (leaf, index within the leaf), one wavefront per leaf
__global__ void k_p2p_tasks(int nleaves, const int *task_off, int2 *tasks) {
    const int leaf = (int)(((int64_t)blockIdx.x * blockDim.x + threadIdx.x) / FMM_WAVE);
    if (leaf >= nleaves) return;
    const int k0 = task_off[leaf], k1 = task_off[leaf + 1];
    for (int k = k0 + lane_id(); k < k1; k += FMM_WAVE) tasks[k] = make_int2(leaf, k - k0);
}

// Potentials and accelerations are summed with 2/|r| in place of 1/|r|
// (rsqrt2_nr), that is times 2 and times 8; the sums of a sink are scaled back
// once, before they leave the kernel (exact: powers of two).
constexpr double P2P_POT_BACK = 0.5, P2P_ACC_BACK = 0.125;

template <int WANT_F, int WITH_POT>
__device__ __forceinline__ void pair(const double4 s, double xb, double yb, double zb, bool skip,
                                     double &pot, double &ax, double &ay, double &az) {
    const double dx = s.x - xb, dy = s.y - yb, dz = s.z - zb;
    const double r2 = skip ? 1.0 : fma(dx, dx, fma(dy, dy, dz * dz));
    const double mu = skip ? 0.0 : s.w;
    if (WANT_F) {
        pot += mu / r2;
    } else {
        const double ri = rsqrt2_nr(r2);        // 2/|r|
        const double q = mu * ri;
        const double q3 = q * ri * ri;
        if (WITH_POT) pot += q;
        ax = fma(q3, dx, ax);
        ay = fma(q3, dy, ay);
        az = fma(q3, dz, az);
    }
}

// Mixed precision: the separation is formed in FP64 and rounded once; the
// squared distance, reciprocal square root, products and the running sums
// are FP32 (every pair's contribution carries a relative error of a few
// FP32 units).  Only ranges without the sinks themselves come here: no
// self-pair test.
__device__ __forceinline__ void pair32(const double4 s, const double4 xb, float &pot, float &ax,
                                       float &ay, float &az) {
    const float dx = (float)(s.x - xb.x), dy = (float)(s.y - xb.y), dz = (float)(s.z - xb.z);
    const float r2 = fmaf(dx, dx, fmaf(dy, dy, dz * dz));
    const float mu = (float)s.w;
    const float ri = __builtin_amdgcn_rsqf(r2);
    const float q = mu * ri;
    const float q3 = q * ri * ri;
    pot += q;
    ax = fmaf(q3, dx, ax);
    ay = fmaf(q3, dy, ay);
    az = fmaf(q3, dz, az);
}

// FP32 partial sums run over at most this many sources per lane before they
// are added into the FP64 sums
constexpr int P2P_CHUNK32 = 32;

// One lane's share of a source range that overlaps its R sinks' own leaf:
// sources p[0], p[stride], ... below pe (the sinks themselves skipped by
// address), the next source loaded before the current one is summed.  Always
// FP64.
template <int R>
__device__ __forceinline__ void sum_own(const double4 *p, const double4 *pe, int stride,
                                        const double4 (&xb)[R], const double4 *const (&self)[R],
                                        double4 (&f)[R]) {
    if (p >= pe) return;
    double4 a = p[0];
    for (;;) {
        const double4 *q = p + stride;
        const bool more = q < pe;
        const double4 b = (more ? q : p)[0];
#pragma unroll
        for (int k = 0; k < R; ++k)
            pair<0, 1>(a, xb[k].x, xb[k].y, xb[k].z, p == self[k], f[k].x, f[k].y, f[k].z, f[k].w);
        if (!more) break;
        p = q;
        a = b;
    }
}

static_assert((int64_t)P2P_TASK * sizeof(double4) < (int64_t(1) << 32),
              "byte offsets within a task's source range fit 32 bits");

// One lane's share of a source range that holds none of its sinks: sources
// base[i], base[i + stride], ... below base[n] (n <= P2P_TASK), FP32 partial
// sums over at most P2P_CHUNK32 sources per lane, then added into the FP64 sums.
template <int R>
__device__ __forceinline__ void sum_far32(const double4 *base, uint32_t i, uint32_t n,
                                          uint32_t stride, const double4 (&xb)[R],
                                          double4 (&f)[R]) {
    gchar *b = uniform_base(base);
    const uint32_t oe = n * 32u, st = stride * 32u;
    uint32_t o = i * 32u;
    while (o < oe) {
        float4 g[R];
#pragma unroll
        for (int k = 0; k < R; ++k) g[k] = make_float4(0.f, 0.f, 0.f, 0.f);
        for (int it = 0; it < P2P_CHUNK32 && o < oe; ++it, o += st) {
            const double4 a = load_source(b + o);
#pragma unroll
            for (int k = 0; k < R; ++k)
                pair32(a, xb[k], g[k].x, g[k].y, g[k].z, g[k].w);
        }
        constexpr double sp = 1.0 / P2P_POT_BACK, sa = 1.0 / P2P_ACC_BACK;
#pragma unroll
        for (int k = 0; k < R; ++k) {
            f[k].x = fma((double)g[k].x, sp, f[k].x);
            f[k].y = fma((double)g[k].y, sa, f[k].y);
            f[k].z = fma((double)g[k].z, sa, f[k].z);
            f[k].w = fma((double)g[k].w, sa, f[k].w);
        }
    }
}

// R sinks per lane: ng = ceil(nb / R) lane groups, group g holds sink slots
// g, g + ng, g + 2 ng, ... (a slot past the leaf repeats slot g and is
// discarded); lanes [0, ng * S) are (group, phase) with S = floor(64 / ng).
template <int R>
__global__ void __launch_bounds__(256)
k_p2p_mixed(int ntasks, const int2 *tasks, const int *leaf_cell, const int *nsrc_tasks,
      const int *moff, const int64_t *off, const int2 *range, const int *chain, TreeArrays t,
      const double4 *xyzm, double4 *out4, double4 *partial) {
    __shared__ double4 red[4][R * FMM_WAVE];
    // blocks in task order: the hardware deals them to the XCDs in turn, which
    // spreads the uneven task lengths evenly (a contiguous eighth of the tasks
    // per XCD left the shorter launches unbalanced)
    const int task = blockIdx.x * 4 + threadIdx.x / FMM_WAVE;
    if (task >= ntasks) return;
    const int lane = lane_id(), w = threadIdx.x / FMM_WAVE;
    const int2 tk = tasks[task];
    const int leaf = tk.x;
    const int c = leaf_cell[leaf];
    const int nts = nsrc_tasks[leaf];
    const int sc = tk.y / nts, ts = tk.y % nts;
    const int beg = t.beg[c], end = t.end[c];
    const int sb = beg + sc * FMM_WAVE;
    const int nb = min(end - sb, FMM_WAVE);
    const int ng = (nb + R - 1) / R;
    const int S = FMM_WAVE / ng;
    const int g = lane % ng, phase = lane / ng;
    const bool active = phase < S;
    double4 xb[R], f[R];
    const double4 *self[R];
#pragma unroll
    for (int k = 0; k < R; ++k) {
        const int slot = g + k * ng < nb ? g + k * ng : g;
        self[k] = xyzm + sb + slot;
        xb[k] = *self[k];
        f[k] = make_double4(0.0, 0.0, 0.0, 0.0);
    }
    // the chain of ancestors with ranges and their list offsets, one per lane
    const int *ch = chain + (size_t)leaf * P2P_CHAIN;
    const int nchain = ch[0];
    const int myanc = lane < nchain ? ch[1 + lane] : 0;
    const int64_t mr0 = lane < nchain ? off[myanc] : 0, mr1 = lane < nchain ? off[myanc + 1] : 0;
    // sources [ts * P2P_TASK, (ts + 1) * P2P_TASK) of the leaf's list; the range
    // descriptors are read 64 at a time (one per lane) and broadcast in turn
    int64_t skip = (int64_t)ts * P2P_TASK, left = P2P_TASK;
    for (int ci = 0; ci < nchain && left > 0; ++ci) {
        const int64_t r0 = readlane64(mr0, ci), r1 = readlane64(mr1, ci);
        for (int64_t rb = r0; rb < r1 && left > 0; rb += FMM_WAVE) {
          const int2 mine = rb + lane < r1 ? range[rb + lane] : make_int2(0, 0);
          const int nbat = (int)min((int64_t)FMM_WAVE, r1 - rb);
          for (int j = 0; j < nbat && left > 0; ++j) {
            int2 rg = make_int2(__builtin_amdgcn_readlane(mine.x, j),
                                __builtin_amdgcn_readlane(mine.y, j));
            const int len = rg.y - rg.x;
            if (skip >= len) {
                skip -= len;
                continue;
            }
            rg.x += (int)skip;
            skip = 0;
            if (rg.y - rg.x > left) rg.y = rg.x + (int)left;
            left -= rg.y - rg.x;
            if (!active) continue;
            const bool own = rg.x < sb + nb && rg.y > sb;   // overlaps the task's sinks
            // the sinks' own leaf holds their nearest neighbours, the largest
            // terms: summed in FP64 also in mixed precision
            const uint32_t nr = (uint32_t)(rg.y - rg.x);
            if (own)
                sum_own<R>(xyzm + rg.x + phase, xyzm + rg.y, S, xb, self, f);
            else
                sum_far32<R>(xyzm + rg.x, phase, nr, S, xb, f);
          }
        }
    }
    // sum the phases of each sink through LDS: red[w][slot + phase * R * ng];
    // active lanes cover every index below R * ng * S <= R * 64 exactly once
    if (active) {
#pragma unroll
        for (int k = 0; k < R; ++k) red[w][g + k * ng + phase * R * ng] = f[k];
    }
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
    if (lane >= nb) return;
    double4 v = red[w][lane];
    for (int ph = 1; ph < S; ++ph) {
        const double4 q = red[w][lane + ph * R * ng];
        v.x += q.x; v.y += q.y; v.z += q.z; v.w += q.w;
    }
    v.x *= P2P_POT_BACK;
    v.y *= P2P_ACC_BACK;
    v.z *= P2P_ACC_BACK;
    v.w *= P2P_ACC_BACK;
    const int bi = sb + lane;
    if (moff[leaf + 1] == moff[leaf]) {          // the leaf's only task
        double4 o = out4[bi];
        o.x += v.x; o.y += v.y; o.z += v.z; o.w += v.w;
        out4[bi] = o;
    } else {
        partial[((int64_t)moff[leaf] + tk.y) * FMM_WAVE + lane] = v;
    }
}

// *out += row[0] + row[stride] + ... (n rows): eight rows' loads in flight at a
// time, added in order
__device__ __forceinline__ void add_rows(double4 *out, const double4 *row, int64_t stride, int n) {
    double4 v = *out;
    for (int t0 = 0; t0 < n; t0 += 8) {
        double4 q[8];
#pragma unroll
        for (int j = 0; j < 8; ++j) q[j] = row[min(t0 + j, n - 1) * stride];
#pragma unroll
        for (int j = 0; j < 8; ++j) {
            if (t0 + j < n) {
                v.x += q[j].x; v.y += q[j].y; v.z += q[j].z; v.w += q[j].w;
            }
        }
    }
    *out = v;
}

// FP64 sums of one task: R sinks in scalar registers, a source per lane.  The
// pairs of a step are scheduled four at a time, which is enough to cover the
// latency of a dependent operation and keeps the kernel within 128 registers
// (four wavefronts per SIMD).
template <int R, int WANT_F, int WITH_POT>
__device__ __forceinline__ void near_sum(const NearTask &q, const int2 *entry,
                                         const double4 *xyzm, double4 *out4, double4 *row) {
    const int lane = lane_id();
    const double4 mine = xyzm[q.sb + (lane < R ? lane : 0)];
    double sx[R], sy[R], sz[R], f[R][4];
#pragma unroll
    for (int k = 0; k < R; ++k) {
        sx[k] = readlane_f64(mine.x, k);
        sy[k] = readlane_f64(mine.y, k);
        sz[k] = readlane_f64(mine.z, k);
        f[k][0] = f[k][1] = f[k][2] = f[k][3] = 0.0;
    }
    near_sources(
        entry, q, [&](uint32_t i) { return load32(xyzm, i); },
        [&](const double4 &a) {
#pragma unroll
            for (int k = 0; k < R; ++k) {
                pair<WANT_F, WITH_POT>(a, sx[k], sy[k], sz[k], false, f[k][0], f[k][1], f[k][2],
                                       f[k][3]);
                if (k % 4 == 3) __builtin_amdgcn_sched_barrier(0);
            }
        },
        [&](double4 a, uint32_t i, bool on) {
            if (!on) a = make_double4(0.0, 0.0, 0.0, 0.0);
#pragma unroll
            for (int k = 0; k < R; ++k) {
                pair<WANT_F, WITH_POT>(a, sx[k], sy[k], sz[k], !on || i == (uint32_t)(q.sb + k),
                                       f[k][0], f[k][1], f[k][2], f[k][3]);
                __builtin_amdgcn_sched_barrier(0);
            }
        });
    // lane i of each row of 16 lanes takes one component of sink i
    double v = 0.0;
#pragma unroll
    for (int k = 0; k < R; ++k) {
        const double w = wave_sum4(f[k][0], f[k][1], f[k][2], f[k][3]);
        v = (lane & 15) == k ? w : v;
    }
    const int comp = wave_sum4_component(), s = lane & 15;
    if (!WANT_F) v *= comp == 0 ? P2P_POT_BACK : P2P_ACC_BACK;
    if (s >= R) return;
    if (q.single) reinterpret_cast<double *>(out4 + q.sb + s)[comp] += v;
    else reinterpret_cast<double *>(row + s)[comp] = v;
}

template <int WANT_F, int WITH_POT>
__global__ void __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(4)))
k_p2p(int ntasks, const int4 *tasks, const int2 *entry, const double4 *xyzm, double4 *out4,
      double4 *partial) {
    const int task = blockIdx.x * 4 + threadIdx.x / FMM_WAVE;
    if (task >= ntasks) return;                  // whole wavefronts leave together
    const NearTask q = unpack_task(tasks[task]);
    double4 *row = partial + (size_t)task * NEAR_R;
    static_assert(NEAR_R == 8, "the cases below");
#define FMM_NEAR(R) case R: near_sum<R, WANT_F, WITH_POT>(q, entry, xyzm, out4, row); break
    switch (q.r) {
        FMM_NEAR(1); FMM_NEAR(2); FMM_NEAR(3); FMM_NEAR(4);
        FMM_NEAR(5); FMM_NEAR(6); FMM_NEAR(7); FMM_NEAR(8);
    }
#undef FMM_NEAR
}

// Plan of the FP64 direct sums, one wavefront per leaf.  Count: the leaf's
// tasks (groups of at most `width` sinks x slices of NEAR_TASK sources), its
// slices and its list entries (its and its ancestors' ranges, and the closing
// entry); active: when not null, leaves whose cell holds no listed sink get
// none.  Entry nleaves is zeroed for the scans.
__global__ void k_near_count(int nleaves, int width, const int *leaf_cell, const int64_t *off,
                             const int2 *range, const int *up, TreeArrays t,
                             const uint8_t *active, int *ntask, int *nslice, int *nentry) {
    const int leaf = (int)(((int64_t)blockIdx.x * blockDim.x + threadIdx.x) / FMM_WAVE);
    if (leaf > nleaves) return;
    int slices = 0;
    int64_t tasks = 0, entries = 0;
    const int c = leaf < nleaves ? leaf_cell[leaf] : -1;
    if (c >= 0 && (!active || active[c])) {
        for (int a = first_with_ranges(c, up, off); a >= 0; a = up[a])
            entries += off[a + 1] - off[a];
        const int64_t S = leaf_sources(c, up, off, range);
        slices = (int)max((int64_t)1, (S + NEAR_TASK - 1) / NEAR_TASK);
        tasks = (int64_t)slices * ((t.end[c] - t.beg[c] + width - 1) / width);
        ++entries;
    }
    if (lane_id() != 0) return;
    // (a count past 32 bits makes a total that the host refuses)
    ntask[leaf] = (int)min(tasks, (int64_t)INT_MAX);
    nentry[leaf] = (int)entries;
    if (leaf < nleaves) nslice[leaf] = slices;
}

// the bounds of the parts, one thread each
__global__ void k_near_parts(int nleaves, const int64_t *task_off, const int64_t *entry_off,
                             int parts, NearPart *bounds) {
    const int k = blockIdx.x * blockDim.x + threadIdx.x;
    if (k > parts) return;
    const int64_t l = k < parts ? near_part_begin(entry_off, nleaves, k) : nleaves;
    bounds[k] = {l, task_off[l], entry_off[l]};
}

// Fill: the list entries (shift, end) of the leaves [l0, l1), from entry offset
// first_entry on, and their tasks, slice by slice (the groups of a slice next to
// each other, so that the wavefronts of a block read the same sources).
__global__ void k_near_fill(int l0, int l1, int width, const int *leaf_cell, const int64_t *off,
                            const int2 *range, const int *up, TreeArrays t, const int *nslice,
                            const int64_t *task_off, const int64_t *entry_off,
                            int64_t first_entry, int4 *tasks, int2 *entry) {
    const int leaf = l0 + (int)(((int64_t)blockIdx.x * blockDim.x + threadIdx.x) / FMM_WAVE);
    if (leaf >= l1) return;
    const int e0 = (int)(entry_off[leaf] - first_entry), k0 = (int)task_off[leaf];
    if (task_off[leaf + 1] == k0) return;
    const int lane = lane_id(), c = leaf_cell[leaf], nts = nslice[leaf];
    const int beg = t.beg[c], nb = t.end[c] - beg, ng = (nb + width - 1) / width;
    // the leaf's position count is known only at the end; a slice is full
    // unless it is the last one, which is written then
    int pos = 0, d = 0, last_first = e0;
    for (int a = first_with_ranges(c, up, off); a >= 0; a = up[a]) {
        const int64_t r1 = off[a + 1];
        for (int64_t rb = off[a]; rb < r1; rb += FMM_WAVE) {
            const int2 rg = rb + lane < r1 ? range[rb + lane] : make_int2(0, 0);
            const int len = rg.y - rg.x;
            const int end = pos + wave_incl_scan(len), begin = end - len;
            if (rb + lane < r1) entry[e0 + d + lane] = make_int2(rg.x - begin, end);
            // slices that begin in this lane's range
            const int s0 = (begin + NEAR_TASK - 1) / NEAR_TASK;
            const int s1 = len > 0 ? (end - 1) / NEAR_TASK : s0 - 1;
            unsigned long long who = __ballot(s1 >= s0);
            while (who) {
                const int l = __ffsll((long long)who) - 1;
                who &= who - 1;
                const int t0 = __builtin_amdgcn_readlane(s0, l);
                const int t1 = __builtin_amdgcn_readlane(s1, l);
                const int first = e0 + d + l;
                const int m = (min(t1, nts - 2) - t0 + 1) * ng;
                for (int k = lane; k < m; k += FMM_WAVE) {
                    const int ts = t0 + k / ng, g = k % ng;
                    const int b0 = group_begin(nb, ng, g), b1 = group_begin(nb, ng, g + 1);
                    tasks[k0 + ts * ng + g] =
                        pack_task(beg + b0, first, ts * NEAR_TASK, b1 - b0, NEAR_TASK, false);
                }
                if (t1 == nts - 1) last_first = first;
            }
            d += (int)min((int64_t)FMM_WAVE, r1 - rb);
            pos = __builtin_amdgcn_readlane(end, FMM_WAVE - 1);
        }
    }
    const int ts = nts - 1;
    for (int g = lane; g < ng; g += FMM_WAVE) {
        const int b0 = group_begin(nb, ng, g), b1 = group_begin(nb, ng, g + 1);
        tasks[k0 + ts * ng + g] = pack_task(beg + b0, last_first, ts * NEAR_TASK, b1 - b0,
                                            pos - ts * NEAR_TASK, nts == 1);
    }
    if (lane == 0) entry[e0 + d] = make_int2(-pos, INT_MAX);
}

// add the slices' sums of leaves with more than one, in slice order
__global__ void k_near_reduce(int64_t n, int width, const int *leaf_of, const int *leaf_cell,
                              const int *nslice, const int64_t *task_off, TreeArrays t,
                              const double4 *partial, double4 *out4) {
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= n) return;
    const int leaf = leaf_of[i], nts = nslice[leaf];
    if (nts <= 1) return;
    const int c = leaf_cell[leaf];
    const int k = (int)(i - t.beg[c]), nb = t.end[c] - t.beg[c], ng = (nb + width - 1) / width;
    const int g = group_of(nb, ng, k);
    add_rows(out4 + i, partial + (task_off[leaf] + g) * width + (k - group_begin(nb, ng, g)),
             (int64_t)ng * width, nts);
}

// the same for the mixed-precision sums, whose groups are consecutive runs of
// 64 sinks, numbered before the slices
__global__ void k_p2p_reduce(int64_t n, const int *leaf_of, const int *leaf_cell,
                             const int *nsrc_tasks, const int *moff, TreeArrays t,
                             const double4 *partial, double4 *out4) {
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= n) return;
    const int leaf = leaf_of[i];
    if (moff[leaf + 1] == moff[leaf]) return;
    const int k = (int)(i - t.beg[leaf_cell[leaf]]), nts = nsrc_tasks[leaf];
    add_rows(out4 + i,
             partial + ((int64_t)moff[leaf] + k / FMM_WAVE * nts) * FMM_WAVE + k % FMM_WAVE,
             FMM_WAVE, nts);
}

// Exact sums of listed sinks (sinks null: of every particle).  A wavefront
// takes DIRECT_R sinks in scalar registers against the sources of its grid row,
// [k chunk, min(n, (k + 1) chunk)), one per lane (near.h), so that a few
// thousand sinks still fill the chip.  With one chunk it writes the results;
// otherwise it writes row k of part (nsinks double4 per row: Psi, a without G)
// and k_direct_sinks_reduce adds the rows of each sink in chunk order, so the
// result does not depend on the order in which blocks run.  An index outside
// [0, n) sets *bad (by the blocks of chunk 0) and its outputs are not written.
// Bound by VALU issue like the near field: 4096 sinks of 10^6 in 2.4 ms (1.7e12
// pairs/s), all of 30,000 in 0.57 ms.  A sink per lane, with the sources read as
// scalars and a self test per pair (25 issue slots), took 5.5 ms and, on 118 of
// the 256 compute units, 5.3 ms.
__global__ void __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(4)))
k_direct_sinks(int64_t n, const double *pos, const double *mass, double G, int64_t nsinks,
               const int64_t *sinks, int64_t chunk, double *pot, double *acc, double4 *part,
               int *bad) {
    const int64_t wave = (int64_t)blockIdx.x * 4 + threadIdx.x / FMM_WAVE;
    if (wave * DIRECT_R >= nsinks) return;       // whole wavefronts leave together
    const int k = blockIdx.y, lane = lane_id();
    const DirectSinks d = direct_sinks(wave, n, nsinks, sinks, k == 0 ? bad : nullptr);
    double sx[DIRECT_R], sy[DIRECT_R], sz[DIRECT_R], f[DIRECT_R][4];
#pragma unroll
    for (int q = 0; q < DIRECT_R; ++q) {
        const double *x = pos + 3 * d.idx[q];
        sx[q] = readlane_f64(x[0], 0);
        sy[q] = readlane_f64(x[1], 0);
        sz[q] = readlane_f64(x[2], 0);
        f[q][0] = f[q][1] = f[q][2] = f[q][3] = 0.0;
    }
    const int64_t j0 = (int64_t)k * chunk, j1 = min(n, j0 + chunk);
    const double *px = pos + 3 * j0, *pm = mass + j0;
    auto source = [&](uint32_t o) {
        const size_t i = 3 * (size_t)o;
        return make_double4(px[i], px[i + 1], px[i + 2], pm[o]);
    };
    direct_steps(
        d, j0, j1,
        [&](uint32_t o) {
            const double4 a = source(o);
#pragma unroll
            for (int q = 0; q < DIRECT_R; ++q) {
                pair<0, 1>(a, sx[q], sy[q], sz[q], false, f[q][0], f[q][1], f[q][2], f[q][3]);
                if (q % 4 == 3) __builtin_amdgcn_sched_barrier(0);
            }
        },
        [&](uint32_t o, bool on) {
            double4 a = make_double4(0.0, 0.0, 0.0, 0.0);
            if (on) a = source(o);
#pragma unroll
            for (int q = 0; q < DIRECT_R; ++q) {
                pair<0, 1>(a, sx[q], sy[q], sz[q], !on || j0 + o == d.idx[q], f[q][0], f[q][1],
                           f[q][2], f[q][3]);
                __builtin_amdgcn_sched_barrier(0);
            }
        });
    double v = 0.0;
#pragma unroll
    for (int q = 0; q < DIRECT_R; ++q) {
        const double w = wave_sum4(f[q][0], f[q][1], f[q][2], f[q][3]);
        v = (lane & 15) == q ? w : v;
    }
    const int comp = wave_sum4_component(), s = lane & 15;
    if (s >= DIRECT_R || !((d.valid >> s) & 1u)) return;
    v *= comp == 0 ? P2P_POT_BACK : P2P_ACC_BACK;
    const int64_t t = d.t0 + s;
    if (part) reinterpret_cast<double *>(part + (int64_t)k * nsinks + t)[comp] = v;
    else if (comp == 0) pot[t] = -G * v;
    else acc[3 * t + comp - 1] = G * v;
}

__global__ void k_direct_sinks_reduce(int64_t n, double G, int64_t nsinks, const int64_t *sinks,
                                      int nchunk, const double4 *part, double *pot, double *acc) {
    const int64_t t = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (t >= nsinks) return;
    const int64_t ii = sinks ? sinks[t] : t;
    if (ii < 0 || ii >= n) return;
    double4 v = part[t];
    for (int k = 1; k < nchunk; ++k) {
        const double4 q = part[(int64_t)k * nsinks + t];
        v.x += q.x; v.y += q.y; v.z += q.z; v.w += q.w;
    }
    pot[t] = -G * v.x;
    acc[3 * t] = G * v.y;
    acc[3 * t + 1] = G * v.z;
    acc[3 * t + 2] = G * v.w;
}

__global__ void k_fill_int(int *p, int64_t count, int v) {
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i < count) p[i] = v;
}

__global__ void k_zero(double4 *p, int64_t n) {
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i < n) p[i] = {0.0, 0.0, 0.0, 0.0};
}

__device__ __forceinline__ double4 add4(const double4 &a, const double4 &b) {
    return {a.x + b.x, a.y + b.y, a.z + b.z, a.w + b.w};
}

// far + near field of every particle in input order
__global__ void k_output(int64_t n, const uint32_t *perm, const double4 *far4,
                         const double4 *near4, double G, double *pot, double *acc,
                         int *nonfinite) {
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= n) return;
    const double4 v = add4(far4[i], near4[i]);
    const int64_t j = perm[i];
    const double p = -G * v.x, a = G * v.y, b = G * v.z, c = G * v.w;
    pot[j] = p;
    acc[3 * j] = a;
    acc[3 * j + 1] = b;
    acc[3 * j + 2] = c;
    if (!(isfinite(p) && isfinite(a) && isfinite(b) && isfinite(c))) atomicOr(nonfinite, 1);
}

// ---- forces for a listed subset of sinks (Sec. 7.1) ------------------------
// flag_in[act[j]] = 1 (input order, zeroed by the caller); *bad = 1 for an
// index outside [0, n)
__global__ void k_mark_listed(int64_t n, int64_t nact, const int64_t *act, int *flag_in,
                              int *bad) {
    const int64_t j = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (j >= nact) return;
    const int64_t i = act[j];
    if (i < 0 || i >= n) atomicOr(bad, 1);
    else flag_in[i] = 1;
}

// key order: f[i] = flag of the particle at sorted position i, inv[input] = i
__global__ void k_sorted_flags(int64_t n, const uint32_t *perm, const int *flag_in, int *f,
                               int *inv) {
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i > n) return;
    if (i == n) {
        f[n] = 0;
        return;
    }
    const uint32_t j = perm[i];
    f[i] = flag_in[j];
    inv[j] = (int)i;
}

// a cell is active if it holds a listed particle: pre is the exclusive scan of f
__global__ void k_cell_active(int ncells, const int *beg, const int *end, const int *pre,
                              uint8_t *active) {
    const int c = blockIdx.x * blockDim.x + threadIdx.x;
    if (c >= ncells) return;
    active[c] = pre[end[c]] > pre[beg[c]] ? 1 : 0;
}

// results of the listed particles, in list order (indices out of range are skipped)
__global__ void k_output_listed(int64_t n, int64_t nact, const int64_t *act, const int *inv,
                                const double4 *far4, const double4 *near4, double G,
                                double *pot, double *acc, int *nonfinite) {
    const int64_t j = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (j >= nact) return;
    const int64_t idx = act[j];
    if (idx < 0 || idx >= n) return;
    const double4 v = add4(far4[inv[idx]], near4[inv[idx]]);
    const double p = -G * v.x, a = G * v.y, b = G * v.z, c = G * v.w;
    pot[j] = p;
    acc[3 * j] = a;
    acc[3 * j + 1] = b;
    acc[3 * j + 2] = c;
    if (!(isfinite(p) && isfinite(a) && isfinite(b) && isfinite(c))) atomicOr(nonfinite, 1);
}

// ---- individual accuracy parameters (Sec. 7) ------------------------------
// every eps_b must be > 0 and finite (*bad = 1 otherwise); the smallest one as
// the bit pattern of a positive double (which orders like the value)
__global__ void __launch_bounds__(256)
k_eps_min(int64_t n, const double *eps_b, unsigned long long *minbits, int *bad) {
    __shared__ unsigned long long red[256 / FMM_WAVE];
    unsigned long long mine = ~0ull;
    int fail = 0;
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n;
         i += (int64_t)gridDim.x * blockDim.x) {
        const double v = eps_b[i];
        if (!(v > 0.0 && isfinite(v))) fail = 1;
        else mine = min(mine, (unsigned long long)__double_as_longlong(v));
    }
    if (__any(fail) && lane_id() == 0) atomicOr(bad, 1);
#pragma unroll
    for (int off = FMM_WAVE / 2; off > 0; off >>= 1) mine = min(mine, __shfl_xor(mine, off));
    if (lane_id() == 0) red[threadIdx.x / FMM_WAVE] = mine;
    __syncthreads();
    if (threadIdx.x == 0) {
        unsigned long long b = red[0];
        for (int w = 1; w < 256 / FMM_WAVE; ++w) b = min(b, red[w]);
        atomicMin(minbits, b);
    }
}

// scale[i] *= eps_b of the particle at sorted position i: the cell minimum
// then is min_B{eps_b a_b} (or f_b) and the criterion compares with it alone
__global__ void k_scale_eps(int64_t n, const uint32_t *perm, const double *eps_b, double *scale) {
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= n) return;
    scale[i] *= eps_b[perm[i]];
}

// sink scale of the acceptance test from the estimate: |a| (criterion a) or f
__global__ void k_scale(int want_f, int64_t n, const double4 *est4, double *scale) {
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= n) return;
    const double4 v = est4[i];
    scale[i] = want_f ? v.x : sqrt(fma(v.y, v.y, fma(v.z, v.z, v.w * v.w)));
}

inline unsigned blocks(int64_t n, int b) { return (unsigned)((n + b - 1) / b); }

}  // namespace

hipError_t launch_range_up(int ncells, const int *parent, const int64_t *off, int *up,
                           hipStream_t s) {
    hipLaunchKernelGGL(k_range_up, dim3(blocks(ncells, 256)), dim3(256), 0, s, ncells, parent,
                       off, up);
    return hipGetLastError();
}

hipError_t launch_p2p_plan(int nleaves, const int *leaf_cell, const int64_t *off,
                           const int2 *range, const int *up, const TreeArrays &t,
                           const uint8_t *active, int *ntask, int *mtask, int *nsrc_tasks,
                           int *task_off, int *moff, int *chain, int *tmp, int *totals,
                           hipStream_t s) {
    hipLaunchKernelGGL(k_p2p_count, dim3(blocks((int64_t)(nleaves + 1) * FMM_WAVE, 256)),
                       dim3(256), 0, s, nleaves, leaf_cell, off, range, up, t, active, ntask,
                       mtask, nsrc_tasks, chain);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    e = exclusive_scan(ntask, task_off, nleaves + 1, tmp, totals, s);
    if (e != hipSuccess) return e;
    return exclusive_scan(mtask, moff, nleaves + 1, tmp, totals + 1, s);
}

hipError_t launch_p2p_tasks(int nleaves, const int *task_off, int2 *tasks, hipStream_t s) {
    hipLaunchKernelGGL(k_p2p_tasks, dim3(blocks((int64_t)nleaves * FMM_WAVE, 256)), dim3(256), 0,
                       s, nleaves, task_off, tasks);
    return hipGetLastError();
}

hipError_t launch_p2p_mixed(int ntasks, const int2 *tasks, const int *leaf_cell,
                            const int *nsrc_tasks, const int *moff, const int64_t *off,
                            const int2 *range, const int *chain, const TreeArrays &t,
                            const double4 *xyzm, double4 *out4, double4 *partial, hipStream_t s) {
    if (ntasks <= 0) return hipSuccess;
    hipLaunchKernelGGL(k_p2p_mixed<P2P_R>, dim3(blocks(ntasks, 4)), dim3(256), 0, s, ntasks, tasks,
                       leaf_cell, nsrc_tasks, moff, off, range, chain, t, xyzm, out4, partial);
    return hipGetLastError();
}

hipError_t launch_p2p_reduce(int64_t n, const int *leaf_of, const int *leaf_cell,
                             const int *nsrc_tasks, const int *moff, const TreeArrays &t,
                             const double4 *partial, double4 *out4, hipStream_t s) {
    hipLaunchKernelGGL(k_p2p_reduce, dim3(blocks(n, 256)), dim3(256), 0, s, n, leaf_of, leaf_cell,
                       nsrc_tasks, moff, t, partial, out4);
    return hipGetLastError();
}

hipError_t launch_near_count(int nleaves, int width, const int *leaf_cell, const int64_t *off,
                             const int2 *range, const int *up, const TreeArrays &t,
                             const uint8_t *active, int *ntask, int *nslice, int *nentry,
                             int64_t *task_off, int64_t *entry_off, int64_t *tmp, int64_t *totals,
                             hipStream_t s) {
    hipLaunchKernelGGL(k_near_count, dim3(blocks((int64_t)(nleaves + 1) * FMM_WAVE, 256)),
                       dim3(256), 0, s, nleaves, width, leaf_cell, off, range, up, t, active,
                       ntask, nslice, nentry);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    e = exclusive_scan(ntask, task_off, nleaves + 1, tmp, totals, s);
    if (e != hipSuccess) return e;
    return exclusive_scan(nentry, entry_off, nleaves + 1, tmp, totals + 1, s);
}

hipError_t launch_near_parts(int nleaves, const int64_t *task_off, const int64_t *entry_off,
                             int parts, NearPart *bounds, hipStream_t s) {
    hipLaunchKernelGGL(k_near_parts, dim3(blocks(parts + 1, 256)), dim3(256), 0, s, nleaves,
                       task_off, entry_off, parts, bounds);
    return hipGetLastError();
}

hipError_t launch_near_fill(int l0, int l1, int width, const int *leaf_cell, const int64_t *off,
                            const int2 *range, const int *up, const TreeArrays &t,
                            const int *nslice, const int64_t *task_off, const int64_t *entry_off,
                            int64_t e0, int4 *tasks, int2 *entry, hipStream_t s) {
    if (l1 <= l0) return hipSuccess;
    hipLaunchKernelGGL(k_near_fill, dim3(blocks((int64_t)(l1 - l0) * FMM_WAVE, 256)), dim3(256), 0,
                       s, l0, l1, width, leaf_cell, off, range, up, t, nslice, task_off, entry_off,
                       e0, tasks, entry);
    return hipGetLastError();
}

hipError_t launch_near(int want_f, int with_pot, int ntasks, const int4 *tasks, const int2 *entry,
                       const double4 *xyzm, double4 *out4, double4 *partial, hipStream_t s) {
    if (ntasks <= 0) return hipSuccess;
#define FMM_P2P_LAUNCH(F, P)                                                                  \
    hipLaunchKernelGGL((k_p2p<F, P>), dim3(blocks(ntasks, 4)), dim3(256), 0, s, ntasks, tasks, \
                       entry, xyzm, out4, partial)
    if (want_f) FMM_P2P_LAUNCH(1, 0);
    else if (with_pot) FMM_P2P_LAUNCH(0, 1);
    else FMM_P2P_LAUNCH(0, 0);
#undef FMM_P2P_LAUNCH
    return hipGetLastError();
}

hipError_t launch_near_reduce(int64_t n, int width, const int *leaf_of, const int *leaf_cell,
                              const int *nslice, const int64_t *task_off, const TreeArrays &t,
                              const double4 *partial, double4 *out4, hipStream_t s) {
    hipLaunchKernelGGL(k_near_reduce, dim3(blocks(n, 256)), dim3(256), 0, s, n, width, leaf_of,
                       leaf_cell, nslice, task_off, t, partial, out4);
    return hipGetLastError();
}

hipError_t launch_zero(double4 *p, int64_t n, hipStream_t s) {
    hipLaunchKernelGGL(k_zero, dim3(blocks(n, 256)), dim3(256), 0, s, p, n);
    return hipGetLastError();
}

hipError_t launch_output(int64_t n, const uint32_t *perm, const double4 *far4,
                         const double4 *near4, double G, double *pot, double *acc,
                         int *nonfinite, hipStream_t s) {
    hipLaunchKernelGGL(k_output, dim3(blocks(n, 256)), dim3(256), 0, s, n, perm, far4, near4, G,
                       pot, acc, nonfinite);
    return hipGetLastError();
}

hipError_t launch_mark_listed(int64_t n, int64_t nact, const int64_t *act, int *flag_in, int *bad,
                             hipStream_t s) {
    if (nact <= 0) return hipSuccess;
    hipLaunchKernelGGL(k_mark_listed, dim3(blocks(nact, 256)), dim3(256), 0, s, n, nact, act,
                       flag_in, bad);
    return hipGetLastError();
}

hipError_t launch_cell_active(int64_t n, const uint32_t *perm, const int *flag_in, int *f,
                              int *inv, int *pre, int *tmp, int *total, int ncells, const int *beg,
                              const int *end, uint8_t *active, hipStream_t s) {
    hipLaunchKernelGGL(k_sorted_flags, dim3(blocks(n + 1, 256)), dim3(256), 0, s, n, perm,
                       flag_in, f, inv);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    e = exclusive_scan(f, pre, n + 1, tmp, total, s);
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(k_cell_active, dim3(blocks(ncells, 256)), dim3(256), 0, s, ncells, beg, end,
                       pre, active);
    return hipGetLastError();
}

hipError_t launch_output_listed(int64_t n, int64_t nact, const int64_t *act, const int *inv,
                                const double4 *far4, const double4 *near4, double G,
                                double *pot, double *acc, int *nonfinite, hipStream_t s) {
    if (nact <= 0) return hipSuccess;
    hipLaunchKernelGGL(k_output_listed, dim3(blocks(nact, 256)), dim3(256), 0, s, n, nact, act, inv,
                       far4, near4, G, pot, acc, nonfinite);
    return hipGetLastError();
}

hipError_t launch_eps_min(int64_t n, const double *eps_b, unsigned long long *minbits, int *bad,
                         hipStream_t s) {
    if (n <= 0) return hipSuccess;
    const unsigned nb = (unsigned)std::min<int64_t>(256, (n + 255) / 256);
    hipLaunchKernelGGL(k_eps_min, dim3(nb), dim3(256), 0, s, n, eps_b, minbits, bad);
    return hipGetLastError();
}

hipError_t launch_scale_eps(int64_t n, const uint32_t *perm, const double *eps_b, double *scale,
                           hipStream_t s) {
    hipLaunchKernelGGL(k_scale_eps, dim3(blocks(n, 256)), dim3(256), 0, s, n, perm, eps_b, scale);
    return hipGetLastError();
}

hipError_t launch_scale(int want_f, int64_t n, const double4 *est4, double *scale,
                        hipStream_t s) {
    hipLaunchKernelGGL(k_scale, dim3(blocks(n, 256)), dim3(256), 0, s, want_f, n, est4, scale);
    return hipGetLastError();
}

hipError_t launch_direct_sinks(int64_t n, const double *pos, const double *mass, double G,
                               int64_t nsinks, const int64_t *sinks, int nchunk, double *pot,
                               double *acc, double4 *part, int *bad, hipStream_t s) {
    if (nsinks <= 0) return hipSuccess;
    if (nchunk < 1 || (nchunk > 1 && !part)) return hipErrorInvalidValue;
    const int64_t chunk = row_length(n, nchunk);
    hipLaunchKernelGGL(k_direct_sinks, dim3(blocks(nsinks, 4 * DIRECT_R), (unsigned)nchunk),
                       dim3(256), 0, s, n, pos, mass, G, nsinks, sinks, chunk, pot, acc,
                       nchunk > 1 ? part : nullptr, bad);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess || nchunk == 1) return e;
    hipLaunchKernelGGL(k_direct_sinks_reduce, dim3(blocks(nsinks, 256)), dim3(256), 0, s, n, G,
                       nsinks, sinks, nchunk, (const double4 *)part, pot, acc);
    return hipGetLastError();
}

hipError_t launch_fill_int(int *p, int64_t count, int v, hipStream_t s) {
    if (count <= 0) return hipSuccess;
    hipLaunchKernelGGL(k_fill_int, dim3(blocks(count, 256)), dim3(256), 0, s, p, count, v);
    return hipGetLastError();
}

}  // namespace fmm
