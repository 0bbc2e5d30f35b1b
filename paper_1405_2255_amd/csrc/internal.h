// Host-side declarations shared by the libfmm translation units: launchers
// for each kernel group and the error-checking macro.  Every launcher takes
// the stream it is ordered on and returns hipSuccess or the launch error.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include "split.h"

#define FMM_KEYLEVELS 21                  // levels resolved by one 63-bit key
#define FMM_MAXLEVEL (2 * FMM_KEYLEVELS)  // levels 22..42 use the second key word
#define FMM_PMAX 20

namespace fmm {

// ---- sort.hip ---------------------------------------------------------
// Exclusive prefix sum of n int32 values (in may equal out).  tmp must hold
// scan_tmp_ints(n) ints.  *total (device, optional) receives the sum.
size_t scan_tmp_ints(int64_t n);
hipError_t exclusive_scan(const int *in, int *out, int64_t n, int *tmp, int *total,
                          hipStream_t s);
// The same with sums of 64 bits (tmp: scan_tmp_ints(n) of them).
hipError_t exclusive_scan(const int *in, int64_t *out, int64_t n, int64_t *tmp, int64_t *total,
                          hipStream_t s);
// Stable LSD radix sort of (key, value) by key bits [0, bits), 8 per pass.
// Buffers are ping-ponged; on return *keys/*vals point at the sorted data
// (one of the two given buffers).  vals may be null (key-only sort).  tmp must
// hold sort_tmp_ints(n) ints (split.h).
// (Only key bits [lo_bit, lo_bit + bits) are sorted.)
hipError_t radix_sort(uint64_t **keys, uint64_t **keys_alt, uint32_t **vals,
                      uint32_t **vals_alt, int64_t n, int bits, int *tmp, hipStream_t s,
                      int lo_bit = 0);

// ---- tree.hip ---------------------------------------------------------
struct TreeArrays {
    int *beg, *end, *parent, *child0, *nchild, *level;
    int *leaf_lo, *leaf_hi;     // leaves [leaf_lo, leaf_hi) in Morton leaf order
    int4 *info;                 // (begin, end, first child, child count) for the walk
    double4 *cen;               // (x, y, z, rho): expansion centre z = s, radius
    double4 *com;               // (x, y, z, rho_com): centre of mass, radius about it
    double *mass;
    double *lo, *hi;            // 3 per cell: bounding box of the cell's particles
    unsigned long long *rho2;   // 3 per cell: atomics scratch for squared radii
    double4 *bsph;              // (x, y, z, R): enclosing-sphere candidate and cover radius
    double *smin;               // min over the cell's particles of the sink scale
};

// K clusters: particles [off[k], off[k+1]) (device int64 offsets); bb holds
// 6 max(K, 1 + BBOX_WAVES) keys (the box of cluster k in bb[6k..6k+5]; with
// K = 1 the rest is per-wavefront scratch)
#define BBOX_WAVES 1024
hipError_t launch_bbox(const double *pos, int64_t n, int K, const int64_t *off,
                       unsigned long long *bb, hipStream_t s);
hipError_t launch_keys(const double *pos, int64_t n, int K, const int64_t *off,
                       const unsigned long long *bb, uint64_t *key, uint32_t *idx,
                       hipStream_t s);
hipError_t launch_cluster_keys(const uint32_t *idx, int64_t n, int K, const int64_t *off,
                               uint64_t *ckey, uint32_t *order, hipStream_t s);
hipError_t launch_apply_order(const uint32_t *order, const uint64_t *key, const uint32_t *idx,
                              int64_t n, uint64_t *key_out, uint32_t *idx_out, hipStream_t s);
// Second key word (levels 22..42) of sorted position i, for particles whose
// level-21 cell (a run of equal first keys inside one cluster) holds more
// than leaf_size particles, else 0; runstart[i] = first position of that run;
// *any (device int, zeroed by the caller) set to 1 if some run is overfull.
hipError_t launch_deep_keys(const double *pos, const uint32_t *perm, const uint64_t *key,
                            int64_t n, int K, const int64_t *off, const unsigned long long *bb,
                            int leaf_size, uint64_t *key2, uint64_t *runstart, uint32_t *iota,
                            int *any, hipStream_t s);
// out[i] = in[order[i]]
hipError_t launch_gather_u64(const uint32_t *order, const uint64_t *in, int64_t n, uint64_t *out,
                             hipStream_t s);
// key_out[i] = key[order[i]], key2_out[i] = key2[order[i]], idx_out[i] = idx[order[i]]
hipError_t launch_apply_order2(const uint32_t *order, const uint64_t *key, const uint64_t *key2,
                               const uint32_t *idx, int64_t n, uint64_t *key_out,
                               uint64_t *key2_out, uint32_t *idx_out, hipStream_t s);
hipError_t launch_gather(const double *pos, const double *mass, const uint32_t *perm,
                         int64_t n, double *x, double *y, double *z, double *m,
                         double4 *xyzm, hipStream_t s);
// The octree in one pass over the key-sorted particles (key: levels 1..21,
// key2: levels 22..42, zero outside refined level-21 cells): g, pre, suf hold
// n ints of scratch; cnt (n + 1 ints) receives the number of cells whose first
// particle is each particle (cnt[n] = 0).  After an exclusive scan of cnt,
// launch_tree_emit writes the cells as (level << 32) | first particle in
// particle order; stably sorted by level (key bits 32..37) they are numbered
// level by level and in key order within a level.  launch_tree_levels writes
// ls[L], L = 0..43, the first cell of each level (ncells past the last), and
// launch_tree_cells fills begin, end, level, parent, first child and child
// count of every cell (t sized for ncells).
hipError_t launch_tree(const uint64_t *key, const uint64_t *key2, int64_t n, int K,
                       const int64_t *off, int leaf_size, int *g, int *pre, int *suf, int *cnt,
                       hipStream_t s);
hipError_t launch_tree_emit(const uint64_t *key, const uint64_t *key2, int64_t n, int K,
                            const int64_t *off, int leaf_size, const int *pre, const int *suf,
                            const int *base, uint64_t *cell, hipStream_t s);
hipError_t launch_tree_levels(const uint64_t *cell, int ncells, int *ls, hipStream_t s);
hipError_t launch_tree_cells(const uint64_t *key, const uint64_t *key2, int64_t n, int K,
                             const int64_t *off, const uint64_t *cell, int ncells, const int *ls,
                             const TreeArrays &t, hipStream_t s);
hipError_t launch_leaf_flags(const TreeArrays &t, int ncells, int *flags, hipStream_t s);
hipError_t launch_leaf_ranges(const TreeArrays &t, int ncells, const int *leafscan,
                              int *leaf_cell, int *leaf_of, int64_t n, hipStream_t s);
// first cell of each level; levels without cells start where the next one does
struct LevelStart {
    int first[FMM_MAXLEVEL + 3];
};
#define LEVEL_SMALL 256   // cells of a level that one block can take
hipError_t launch_geometry(const TreeArrays &t, const LevelStart &ls, int depth, int nleaves,
                           const int *leaf_cell, const double *x, const double *y,
                           const double *z, const double *m, hipStream_t s);
// enclosing-sphere candidates of every cell
hipError_t launch_enclosing(const TreeArrays &t, const LevelStart &ls, int depth, int nleaves,
                            const int *leaf_cell, const double *x, const double *y,
                            const double *z, hipStream_t s);
// squared radii of every cell: candidate = false about the box midpoint and
// the centre of mass (rho2 slots 0, 1), true about the enclosing-sphere
// candidate (slot 2)
hipError_t launch_radii(const TreeArrays &t, int64_t n, const int *leaf_of,
                        const int *leaf_cell, int maxlevel, const double *x, const double *y,
                        const double *z, bool candidate, hipStream_t s);
// cen.w and com.w from slots 0, 1; smin = infinity
hipError_t launch_radii_finish(const TreeArrays &t, int ncells, hipStream_t s);
// the candidate replaces the midpoint where its radius (slot 2) is smaller
hipError_t launch_centre_select(const TreeArrays &t, int ncells, hipStream_t s);
// minimum sink scale of every cell (smin infinite before)
hipError_t launch_smin(const TreeArrays &t, int nleaves, const int *leaf_cell,
                       const double *scale, hipStream_t s);

// ---- expansions.hip ---------------------------------------------------
// Internal expansion layout: for each cell, the complex coefficients X_n^m,
// 0 <= m <= n <= p, at complex index n(n+1)/2 + m (Re, Im adjacent); the
// m < 0 half follows from X_n^{-m} = (-1)^m conj(X_n^m).
inline int ncplx(int p) { return (p + 1) * (p + 2) / 2; }
hipError_t launch_p2m(int p, const TreeArrays &t, const int *leaf_cell, int nleaves,
                      const double *x, const double *y, const double *z, const double *m,
                      double *M, hipStream_t s);
// C(p, n) P_n per cell: rows of power_stride(p) doubles (16-byte aligned)
inline __host__ __device__ int power_stride(int p) { return (p + 2) & ~1; }
// Cells [c0, c1) of one level: complete M (internal cells: sum of the
// children's T), write P (when not null) and T = M shifted to the parent's
// centre (not for roots).  Run from the deepest level up to level 0.
hipError_t launch_m2m_level(int p, const TreeArrays &t, int c0, int c1, double *M, double *T,
                            double *P, hipStream_t s);
// (active: when not null, cells / leaves without listed sinks are skipped)
hipError_t launch_l2l_level(int p, const TreeArrays &t, int c0, int c1, double *F,
                            const uint8_t *active, hipStream_t s);
// far field at every particle of every leaf: out4[i] = (Psi, ax, ay, az)
hipError_t launch_l2p(int p, const TreeArrays &t, const int *leaf_of, const int *leaf_cell,
                      int64_t n, const double *x, const double *y, const double *z,
                      const double *F, double4 *out4, hipStream_t s,
                      const uint8_t *active = nullptr);
// low-order estimate: monopole M2L into per-cell (Psi, a) at com (gravity)
// or the 1/r^2 sum (f); L2L of the same; evaluation at particles.
hipError_t launch_est_m2l(int want_f, const TreeArrays &t, int nsinks, const int64_t *off,
                          const uint64_t *list, int sh, double4 *Fe, hipStream_t s);
hipError_t launch_est_down(int want_f, const TreeArrays &t, const int *leaf_cell, int nleaves,
                           const double4 *Fe, double4 *out4, hipStream_t s);

// ---- walk.hip -----------------------------------------------------------
struct WalkParams {
    int mode;          // 0 main (criterion a/f), 1 main (theta), 2 estimate (theta<1 on com)
    int p;
    double eps;
    double theta_crit;
    double p2p_pairs;  // accepted with N_A N_B < p2p_pairs -> direct
    int nroots;        // the walk starts from (r, r) for every root r < nroots
    int sh;            // M2L keys are (sink << sh) | source cell
    int pb;            // direct-sum keys are (sink << pb) | first source particle
    int pack;          // nonzero: direct-sum keys carry the range end too,
                       // (sink << 2pb) | (first << pb) | end (needs sh + 2 pb <= 64)
    const uint8_t *active;   // not null: pairs whose sink cell holds no listed
                             // particle are dropped (forces for a subset, Sec. 7.1)
};
struct WalkBuffers {
    uint2 *front[2]; int64_t cap_out;   // sweep i reads front[i & 1] and writes the other
                                        // (both hold cap_out pairs)
    uint64_t *m2l; int64_t cap_m2l;
    uint64_t *p2p; uint32_t *p2p_end; int64_t cap_p2p;   // key, end of the source range
    unsigned long long *counters;   // [0] m2l, [1] direct entries, [2] direct particle
                                    // pairs, [3] overflow, [4 + i] frontier after sweep i,
                                    // [WALK_CUM + 2 i + k] the first two before sweep i,
                                    // [WALK_CUR + j] the sweep that launch j begins with,
                                    // [WALK_TICKETS + i] tiles of sweep i drawn,
                                    // [WALK_ENTRIES + 3 j + k] what tile j has published
    uint16_t *code;                 // cap_out: each input pair's decision (count -> write)
};
// Launch j takes the sweep in counters[WALK_CUR + j] (launch 0: sweep 0) and
// leaves the next one in counters[WALK_CUR + j + 1]; sweep i reads its frontier
// size from counters[4 + i - 1] (sweep 0: the roots) and does nothing if it is 0.
// A small run takes sweeps as long as their frontiers hold at most WALK_SMALL pairs
// (none if the first is larger), a tile sweep one sweep of at most WALK_TILES
// tiles (none if it is larger), a full sweep any.  btmp holds walk_tmp_u64()
// entries of per-block scratch.
enum WalkHow : char { WALK_FULL_SWEEP, WALK_SMALL_RUN, WALK_TILE_SWEEP };
constexpr int WALK_TILES = 1024;                            // of 256 pairs
constexpr int64_t WALK_TILED = 65536;                       // pairs: see walk.hip
constexpr int WALK_SMALL = 4096;
constexpr int WALK_SWEEPS = 2 * FMM_MAXLEVEL + 4;           // most sweeps of a walk
constexpr int WALK_CUM = 4 + WALK_SWEEPS;
constexpr int WALK_CUR = WALK_CUM + 2 * (WALK_SWEEPS + 1);
constexpr int WALK_LAUNCHES = 4 * WALK_SWEEPS;              // most launches of a walk
constexpr int WALK_TICKETS = WALK_CUR + WALK_LAUNCHES + 1;
constexpr int WALK_ENTRIES = WALK_TICKETS + WALK_SWEEPS;
constexpr int WALK_COUNTERS = WALK_ENTRIES + 3 * WALK_TILES;
size_t walk_tmp_u64();
hipError_t launch_root_pairs(uint2 *f, int nroots, hipStream_t s);
hipError_t launch_walk(const WalkParams &wp, const TreeArrays &t, const double *P,
                       const WalkBuffers &wb, int launch, WalkHow how, unsigned long long *btmp,
                       hipStream_t s);
// offsets of the sorted (sink << sh | source) list per sink: off[c] for c in [0, nsinks]
// (count: device, the list's length in place of nlist where not null)
hipError_t launch_list_offsets(const uint64_t *list, int64_t nlist, int nsinks, int sh,
                               int64_t *off, hipStream_t s, const int *count = nullptr);
// merge key-sorted direct-sum entries into maximal particle ranges per sink:
// first call (write = false) flags and scans (flag: n + 1 ints, *total = runs);
// second call writes range[run] = (begin, end) and rkey[run] = (sink << pb) |
// begin.  packed: the keys carry the ends (WalkParams::pack), end is unused.
hipError_t launch_range_merge(const uint64_t *key, const uint32_t *end, int64_t n, int pb,
                              int packed, int *flag, int *tmp, int *total, int2 *range,
                              uint64_t *rkey, bool write, hipStream_t s);

// ---- m2l.hip ------------------------------------------------------------
// Chunk table of the sink-sorted M2L list: the chunks per cell counted into cnt
// and scanned into coff (ncells + 1 entries, the last one the number of chunks),
// then chunks[] = (sink, e0, e1).  A list of n entries has at most
// n / M2L_CHUNK + ncells chunks; the M2L launchers take such a bound (it sizes the grid and the
// buffers) and the number itself on the device.
#define M2L_CHUNK 16
hipError_t launch_chunks(int ncells, const int64_t *off, int *cnt, int *coff, int *tmp,
                         int4 *chunks, hipStream_t s);
// orders up to FMM_M2L_FIXED_MAX use register-resident kernels compiled per
// order; higher orders (or generic = true) use the LDS-staged generic kernel
#define FMM_M2L_FIXED_MAX 16
hipError_t launch_m2l(int p, int bound, const int *nchunks, const int4 *chunks, const uint64_t *list, int sh,
                      const TreeArrays &t, const double *M, double *Fpart, hipStream_t s,
                      bool generic = false);
// Mixed precision (orders up to FMM_M2L_FIXED_MAX): scaled FP32 multipoles,
// FP32 chunk sums Fh with their scale sigma, the FP64 terms of degree
// n + k <= FMM_M2L32_JLO per chunk (Flow: tri(min(p, JLO) + 1, 0) complex
// each), reduction to FP64 F.
#define FMM_M2L32_JLO 3
hipError_t launch_m2l32_multipoles(int p, int ncells, const TreeArrays &t, const double *M,
                                   float *M32, hipStream_t s);
hipError_t launch_m2l32(int p, int bound, const int *nchunks, const int4 *chunks, const uint64_t *list, int sh,
                        const TreeArrays &t, const double *M, const float *M32, float *Fpart,
                        double *Flow, double *sig, hipStream_t s);
hipError_t launch_m2l32_reduce(int p, int ncells, const int *coff, const float *Fpart,
                               const double *Flow, const double *sig, double *F, hipStream_t s);
hipError_t launch_m2l_reduce(int p, int ncells, const int *coff, const double *Fpart, double *F,
                             hipStream_t s);

// ---- m2l_rot.hip ---------------------------------------------------------
// Rotation-accelerated M2L (App. A), orders 1..FMM_M2L_ROT_MAX: one wavefront
// per 64 consecutive entries of the sink-sorted list; partial sums per piece
// (a run of one sink's entries inside one window) go to Fpart (2 tri(p+1, 0)
// doubles each) and launch_m2l_reduce adds them per sink.  Pieces: at most
// ceil(nlist / 64) + ncells; launch_rot_pieces counts them per cell into cnt
// and scans into coff (ncells + 1 entries, *total = pieces).
#define FMM_M2L_ROT_MAX 16
// The rotation kernel is switched off until its results on the device are
// established: FMM_M2L_AUTO never selects it (FMM_M2L_ROT_AUTO_MIN above
// FMM_M2L_ROT_MAX) and an explicit request fails with FMM_E_UNSUPPORTED.
#define FMM_M2L_ROT_ENABLED 0
#define FMM_M2L_ROT_AUTO_MIN (FMM_M2L_ROT_MAX + 1)
hipError_t launch_rot_pieces(int ncells, const int64_t *off, int *cnt, int *coff, int *tmp,
                             int *total, hipStream_t s);
hipError_t launch_m2l_rot(int p, int64_t nlist, const uint64_t *list, int sh, const int64_t *off,
                          const int *coff, const TreeArrays &t, const double *M, double *Fpart,
                          hipStream_t s);

// ---- p2p.hip ------------------------------------------------------------
// Near field of each sink leaf over its list, added to out4 (sorted order).
// off: ncells + 1 offsets into range (per sink cell).
// up[c]: nearest proper ancestor of c with direct-sum ranges (or -1)
hipError_t launch_range_up(int ncells, const int *parent, const int64_t *off, int *up,
                           hipStream_t s);
// FP64 sums: tasks of up to `width` sinks (NEAR_R; NEAR_JERK_R with the jerk,
// jerk.h) x NEAR_TASK sources (near.h).  Count and scan: tasks and list entries
// per leaf (ntask, nentry and their scans task_off, entry_off: nleaves + 1
// each), nslice (nleaves); totals[0] = tasks, totals[1] = entries.  The entries
// of all leaves together have no 32-bit bound (a leaf of one particle has
// hundreds), so the leaves are taken in parts of about NEAR_ENTRIES entries
// (near_parts, split.h): launch_near_parts finds the bounds of the parts
// (parts + 1 of them: leaf, its task and its entry offset).  Fill: the tasks of
// the leaves [l0, l1) and their entries, from entry offset e0 on (entry padded
// by 64).  Every task has a partial row of `width` entries, used by leaves with
// more than one slice; the reduction adds those.
#define NEAR_R 8
#define NEAR_JERK_R 6
#define NEAR_TASK 4096
#define NEAR_PAD 128    // particles past n that the sums may load (and drop)
struct NearPart {
    int64_t leaf, task, entry;
};
hipError_t launch_near_count(int nleaves, int width, const int *leaf_cell, const int64_t *off,
                             const int2 *range, const int *up, const TreeArrays &t,
                             const uint8_t *active, int *ntask, int *nslice, int *nentry,
                             int64_t *task_off, int64_t *entry_off, int64_t *tmp, int64_t *totals,
                             hipStream_t s);
hipError_t launch_near_parts(int nleaves, const int64_t *task_off, const int64_t *entry_off,
                             int parts, NearPart *bounds, hipStream_t s);
hipError_t launch_near_fill(int l0, int l1, int width, const int *leaf_cell, const int64_t *off,
                            const int2 *range, const int *up, const TreeArrays &t,
                            const int *nslice, const int64_t *task_off, const int64_t *entry_off,
                            int64_t e0, int4 *tasks, int2 *entry, hipStream_t s);
hipError_t launch_near(int want_f, int with_pot, int ntasks, const int4 *tasks, const int2 *entry,
                       const double4 *xyzm, double4 *out4, double4 *partial, hipStream_t s);
hipError_t launch_near_reduce(int64_t n, int width, const int *leaf_of, const int *leaf_cell,
                              const int *nslice, const int64_t *task_off, const TreeArrays &t,
                              const double4 *partial, double4 *out4, hipStream_t s);
// Mixed precision (FP32 pair arithmetic, separations in FP64, sums flushed to
// FP64; potential and acceleration): tasks of up to 64 sinks x P2P_TASK sources.
// Planning: per leaf the task counts (ntask, mtask, nsrc_tasks: nleaves + 1
// ints each) and their scans task_off, moff; totals[0] = tasks, totals[1] =
// partial rows (64 entries each).
#define P2P_TASK 2048
// chain: P2P_CHAIN ints per leaf, [0] = the number of cells on the leaf's
// chain of ancestors that hold direct-sum ranges (the leaf first), then their
// indices; written by the plan, read by the direct-sum kernel
#define P2P_CHAIN (FMM_MAXLEVEL + 2)
hipError_t launch_p2p_plan(int nleaves, const int *leaf_cell, const int64_t *off,
                           const int2 *range, const int *up, const TreeArrays &t,
                           const uint8_t *active, int *ntask, int *mtask, int *nsrc_tasks,
                           int *task_off, int *moff, int *chain, int *tmp, int *totals,
                           hipStream_t s);
hipError_t launch_p2p_tasks(int nleaves, const int *task_off, int2 *tasks, hipStream_t s);
hipError_t launch_p2p_mixed(int ntasks, const int2 *tasks, const int *leaf_cell,
                            const int *nsrc_tasks, const int *moff, const int64_t *off,
                            const int2 *range, const int *chain, const TreeArrays &t,
                            const double4 *xyzm, double4 *out4, double4 *partial, hipStream_t s);
hipError_t launch_p2p_reduce(int64_t n, const int *leaf_of, const int *leaf_cell,
                             const int *nsrc_tasks, const int *moff, const TreeArrays &t,
                             const double4 *partial, double4 *out4, hipStream_t s);
// pot, acc of every particle from its far and near field (sorted order)
hipError_t launch_output(int64_t n, const uint32_t *perm, const double4 *far4,
                         const double4 *near4, double G, double *pot, double *acc,
                         int *nonfinite, hipStream_t s);
hipError_t launch_zero(double4 *p, int64_t n, hipStream_t s);
// forces for a listed subset of sinks (Sec. 7.1): flag_in (n ints, zeroed by the
// caller) marks the listed input indices, *bad = 1 if one is outside [0, n);
// then per sorted position f (n + 1), inv (input -> sorted, n), the exclusive
// scan pre (n + 1, scratch tmp/total) and active[c] = 1 for cells holding a
// listed particle; the output kernel writes the listed particles in list order
hipError_t launch_mark_listed(int64_t n, int64_t nact, const int64_t *act, int *flag_in, int *bad,
                             hipStream_t s);
hipError_t launch_cell_active(int64_t n, const uint32_t *perm, const int *flag_in, int *f,
                              int *inv, int *pre, int *tmp, int *total, int ncells, const int *beg,
                              const int *end, uint8_t *active, hipStream_t s);
// individual accuracy parameters (Sec. 7): *bad = 1 unless every eps_b is
// > 0 and finite; *minbits (set to all ones by the caller) = bit pattern of the
// smallest; launch_scale_eps multiplies the key-ordered sink scale by eps_b
hipError_t launch_eps_min(int64_t n, const double *eps_b, unsigned long long *minbits, int *bad,
                         hipStream_t s);
hipError_t launch_scale_eps(int64_t n, const uint32_t *perm, const double *eps_b, double *scale,
                           hipStream_t s);
hipError_t launch_output_listed(int64_t n, int64_t nact, const int64_t *act, const int *inv,
                                const double4 *far4, const double4 *near4, double G,
                                double *pot, double *acc, int *nonfinite, hipStream_t s);
hipError_t launch_scale(int want_f, int64_t n, const double4 *est4, double *scale,
                        hipStream_t s);
// Exact sums for listed sinks (sinks null: nsinks = n, every particle; an index
// outside [0, n) sets *bad and its outputs are left alone).  The sources are cut
// into nchunk chunks of ceil(n / nchunk), one per grid row; with nchunk > 1 the
// partial sums go to part (nchunk * nsinks double4) and are added per sink in
// chunk order.  direct_rows (split.h) gives the library's choice.
hipError_t launch_direct_sinks(int64_t n, const double *pos, const double *mass, double G,
                               int64_t nsinks, const int64_t *sinks, int nchunk, double *pot,
                               double *acc, double4 *part, int *bad, hipStream_t s);
// p[0 .. count) = v (a kernel, so that no memset node enters a captured graph)
hipError_t launch_fill_int(int *p, int64_t count, int v, hipStream_t s);

}  // namespace fmm
