// Device-wide exclusive scan and stable LSD radix sort for gfx950.
//
// Scan: tiles of 2048 counts (256 threads x 8); one launch sums the tiles, a
// second scans each tile behind the sum of the tiles before it.
//
// Radix sort: 8-bit digits.  Up to RS_BLOCK_KEYS keys are sorted by one block
// that holds them in LDS over all passes.  Longer arrays take one launch per
// pass: the digit counts of every pass are known beforehand (they do not depend
// on the order), and a tile learns how many equal digits lie in the tiles
// before it from what those have published (each publishes its own counts at
// once and its running sum as soon as it knows it): the prefix scan by looking
// back of Merrill and Garland (2016), as Adinets and Merrill (2022) use it for
// digits.  A key's rank inside its
// tile comes from 64-wide ballot matching of equal digits.
#include "internal.h"
#include "dev.h"

#include <algorithm>
#include <utility>

namespace fmm {

namespace {

constexpr int SCAN_THREADS = 256;
constexpr int SCAN_ITEMS = 8;
constexpr int SCAN_TILE = SCAN_THREADS * SCAN_ITEMS;

template <class T>
__device__ T block_excl_scan(T v, T *total) {
    // 256 threads = 4 waves
    __shared__ T wsum[SCAN_THREADS / FMM_WAVE];
    const int lane = lane_id(), w = threadIdx.x / FMM_WAVE;
    const T inc = wave_incl_scan(v);
    if (lane == FMM_WAVE - 1) wsum[w] = inc;
    __syncthreads();
    T off = 0, tot = 0;
#pragma unroll
    for (int i = 0; i < SCAN_THREADS / FMM_WAVE; ++i) {
        if (i < w) off += wsum[i];
        tot += wsum[i];
    }
    __syncthreads();
    if (total) *total = tot;
    return off + inc - v;
}

template <class I, class T>
__global__ void __launch_bounds__(SCAN_THREADS) k_tile_sums(const I *in, int64_t n, T *sums) {
    const int64_t base = (int64_t)blockIdx.x * SCAN_TILE;
    T s = 0;
#pragma unroll
    for (int i = 0; i < SCAN_ITEMS; ++i) {
        const int64_t j = base + (int64_t)i * SCAN_THREADS + threadIdx.x;
        if (j < n) s += in[j];
    }
    T tot;
    block_excl_scan(s, &tot);
    if (threadIdx.x == 0) sums[blockIdx.x] = tot;
}

// Each tile behind the sum of the tiles before it: sums holds the tiles' sums,
// which each block adds up to its own (up to SCAN_TILES of them, from the
// cache, cost less than a launch that scans them), or their prefixes.
constexpr int SCAN_TILES = 8192;
template <class I, class T>
__global__ void __launch_bounds__(SCAN_THREADS)
k_tile_scan(const I *in, T *out, int64_t n, const T *sums, bool prefixes, T *total) {
    const int64_t base = (int64_t)blockIdx.x * SCAN_TILE + (int64_t)threadIdx.x * SCAN_ITEMS;
    I v[SCAN_ITEMS];
    T s = 0, off = 0;
    if (sums && prefixes) {
        off = sums[blockIdx.x];
    } else if (sums) {
        T q = 0;
#pragma unroll 4
        for (int i = threadIdx.x; i < (int)blockIdx.x; i += SCAN_THREADS) q += sums[i];
        block_excl_scan(q, &off);
    }
#pragma unroll
    for (int i = 0; i < SCAN_ITEMS; ++i) {
        const int64_t j = base + i;
        v[i] = j < n ? in[j] : 0;
        s += v[i];
    }
    T tot;
    T run = block_excl_scan(s, &tot) + off;
#pragma unroll
    for (int i = 0; i < SCAN_ITEMS; ++i) {
        const int64_t j = base + i;
        if (j < n) out[j] = run;
        run += v[i];
    }
    if (total && blockIdx.x == gridDim.x - 1 && threadIdx.x == SCAN_THREADS - 1) *total = run;
}

// One block scans an array of up to SCAN1_MAX ints in a single launch
// instead of two (5 to 9 us against 12): each thread sums a contiguous chunk, the block scans the
// chunk sums, and each thread writes its chunk's prefixes.  in and out may be
// the same array (each thread reads its chunk before it writes it).
constexpr int SCAN1_THREADS = 1024;
constexpr int64_t SCAN1_MAX = 1 << 14;

template <class I, class T>
__global__ void __launch_bounds__(SCAN1_THREADS)
k_scan_single(const I *in, T *out, int64_t n, T *total) {
    __shared__ T wsum[SCAN1_THREADS / FMM_WAVE];
    const int t = threadIdx.x, lane = lane_id(), w = t / FMM_WAVE;
    const int64_t chunk = (n + SCAN1_THREADS - 1) / SCAN1_THREADS;
    const int64_t lo = min(n, (int64_t)t * chunk), hi = min(n, lo + chunk);
    T s = 0;
#pragma unroll 8
    for (int64_t i = lo; i < hi; ++i) s += in[i];
    const T inc = wave_incl_scan(s);
    if (lane == FMM_WAVE - 1) wsum[w] = inc;
    __syncthreads();
    T run = inc - s;
    for (int i = 0; i < w; ++i) run += wsum[i];
    if (total && t == SCAN1_THREADS - 1) *total = run + s;
#pragma unroll 8
    for (int64_t i = lo; i < hi; ++i) {
        const I v = in[i];
        out[i] = run;
        run += v;
    }
}

// ---- radix sort -------------------------------------------------------
constexpr int RS_WINDOW = 4;              // entries of earlier tiles read at a time
constexpr int RS_DIGITS_THREADS = 256;
constexpr int RS_DIGITS_BLOCKS = 1024;
constexpr int RS_BLOCK_THREADS = 1024;
constexpr int RS_BLOCK_KEYS = RS_BLOCK_THREADS * RS_ITEMS;
// A tile's entry per digit: 0 (nothing yet), its own count + 1, or
// RS_RUNNING + the count of this and all earlier tiles.
constexpr unsigned RS_RUNNING = 1u << 16;

// what a sort keeps in its scratch: digit counts of every pass, a ticket per
// pass, and two arrays of tile entries (a pass clears the next one's)
struct SortTmp {
    int *digits;
    int *tickets;
    unsigned *entry[2];
};

template <int THREADS>
struct TileLds {
    int wcount[THREADS / FMM_WAVE][256];  // per wavefront: digit counts, then offsets
    int start[256];                       // first position of a digit in the tile
    int base[256];                        // and in the output, less start
    int wsum[2][4];
};

// exclusive prefix over the 256 digits of the first 256 threads' v (all threads
// call it; the others' result means nothing)
__device__ __forceinline__ int digit_scan(int v, int *wsum) {
    const int w = threadIdx.x / FMM_WAVE;
    const int inc = wave_incl_scan(v);
    if (w < 4 && lane_id() == FMM_WAVE - 1) wsum[w] = inc;
    __syncthreads();
    int off = 0;
#pragma unroll
    for (int i = 0; i < 3; ++i) off += i < w ? wsum[i] : 0;
    return off + inc - v;
}

// one round of a wavefront, a key per lane: the key's rank among the equal
// digits of the rounds so far, whose counts stand in wc (zeros at first)
__device__ __forceinline__ int wave_rank(uint64_t k, bool valid, int shift, int *wc) {
    const unsigned long long below = (1ull << lane_id()) - 1ull;
    const int d = (int)((k >> shift) & 255u);
    unsigned long long peers = __ballot(valid);
#pragma unroll
    for (int b = 0; b < 8; ++b) {
        const unsigned long long m = __ballot((d >> b) & 1);
        peers &= ((d >> b) & 1) ? m : ~m;
    }
    const int before = __popcll(peers & below);
    const int old = wc[d];
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    if (valid && before == 0) wc[d] = old + __popcll(peers);
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    return old + before;
}

// counts -> the wavefronts' offsets within a digit; the tile's count of digit
// threadIdx.x (first 256 threads)
template <int THREADS>
__device__ __forceinline__ int wave_offsets(TileLds<THREADS> &L) {
    int run = 0;
    if (threadIdx.x < 256) {
#pragma unroll
        for (int i = 0; i < THREADS / FMM_WAVE; ++i) {
            const int c = L.wcount[i][threadIdx.x];
            L.wcount[i][threadIdx.x] = run;
            run += c;
        }
    }
    return run;
}

template <int THREADS>
__device__ __forceinline__ void clear_counts(TileLds<THREADS> &L) {
    int *c = &L.wcount[0][0];
#pragma unroll
    for (int i = threadIdx.x; i < THREADS / FMM_WAVE * 256; i += THREADS) c[i] = 0;
}

__global__ void __launch_bounds__(256) k_rs_zero(int *a, int64_t n) {
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i < n) a[i] = 0;
}

// Digit counts of all passes.  Neighbouring keys share their upper digits, so
// that adds to one counter meet: there are RS_COPIES of each, taken by the
// lanes in turn, and a wavefront that holds one digit adds it at once.  Eight
// keys per thread are loaded together.
constexpr int RS_COPIES = 4;
__global__ void __launch_bounds__(RS_DIGITS_THREADS)
k_rs_digits(const uint64_t *keys, int64_t n, int lo, int passes, int *digits) {
    __shared__ int h[RS_MAX_PASSES * 256 * RS_COPIES];
    for (int i = threadIdx.x; i < passes * 256 * RS_COPIES; i += RS_DIGITS_THREADS) h[i] = 0;
    __syncthreads();
    const int lane = lane_id();
    constexpr int64_t TILE = RS_DIGITS_THREADS * RS_ITEMS;
    for (int64_t j0 = (int64_t)blockIdx.x * TILE; j0 < n; j0 += (int64_t)gridDim.x * TILE) {
        uint64_t k[RS_ITEMS];
#pragma unroll
        for (int r = 0; r < RS_ITEMS; ++r) {
            const int64_t j = j0 + r * RS_DIGITS_THREADS + threadIdx.x;
            k[r] = keys[min(j, n - 1)] >> lo;
        }
#pragma unroll
        for (int r = 0; r < RS_ITEMS; ++r) {
            const bool valid = j0 + r * RS_DIGITS_THREADS + threadIdx.x < n;
            const int on = __popcll(__ballot(valid));
            for (int q = 0; q < passes; ++q) {
                const int d = (int)((k[r] >> (8 * q)) & 255u);
                int *c = h + (q * 256 + d) * RS_COPIES;
                if (__all(d == __builtin_amdgcn_readfirstlane(d))) {
                    if (lane == 0) atomicAdd(c, on);
                } else if (valid) {
                    atomicAdd(c + lane % RS_COPIES, 1);
                }
            }
        }
    }
    __syncthreads();
    for (int i = threadIdx.x; i < passes * 256; i += RS_DIGITS_THREADS) {
        int v = 0;
#pragma unroll
        for (int j = 0; j < RS_COPIES; ++j) v += h[i * RS_COPIES + j];
        if (v) atomicAdd(&digits[i], v);
    }
}

__device__ __forceinline__ unsigned entry_load(const unsigned *p) {
    return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ void entry_store(unsigned *p, unsigned v) {
    __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// equal digits in the tiles before this one: backwards over the published
// entries, RS_WINDOW at a time, until a running sum.  A tile's number is a ticket
// drawn at its start, so every earlier tile has started, and it publishes its
// counts before it waits for anything: the wait ends.
__device__ __forceinline__ int tiles_before(const unsigned *entry, int tile, int digit) {
    unsigned sum = 0;
    int t = tile - 1;
    while (t >= 0) {
        unsigned e[RS_WINDOW];
#pragma unroll
        for (int j = 0; j < RS_WINDOW; ++j)
            e[j] = entry_load(entry + (size_t)max(t - j, 0) * 256 + digit);
#pragma unroll
        for (int j = 0; j < RS_WINDOW; ++j) {
            if (t < 0) break;
            if (e[j] == 0) {
                __builtin_amdgcn_s_sleep(1);
                break;
            }
            if (e[j] >= RS_RUNNING) {
                sum += e[j] - RS_RUNNING;
                t = -1;
            } else {
                sum += e[j] - 1;
                --t;
            }
        }
    }
    return (int)sum;
}

// One pass.  Bound by the bytes of the keys once read and once written for long
// arrays and by latency for short ones: the tile is put in order in LDS first,
// so that the writes of a digit are one run.  10^6 keys with values: 17.5 us a
// pass; with counts, three launches of scans and a scatter it was 58 us of
// which the kernels ran 32.
template <int THREADS, bool HAS_VAL>
__global__ void __launch_bounds__(THREADS)
k_rs_pass(const uint64_t *keys, const uint32_t *vals, uint64_t *okeys, uint32_t *ovals,
          int64_t n, int shift, const int *digits, int *ticket, unsigned *entry,
          unsigned *next) {
    constexpr int TILE = THREADS * RS_ITEMS;
    __shared__ TileLds<THREADS> L;
    __shared__ uint64_t skey[TILE];
    __shared__ uint32_t sval[HAS_VAL ? TILE : 1];
    __shared__ int stile;
    const int tid = threadIdx.x, lane = lane_id(), w = tid / FMM_WAVE;
    if (tid == 0) stile = atomicAdd(ticket, 1);
    clear_counts(L);
    __syncthreads();
    const int tile = stile;
    const int64_t tbase = (int64_t)tile * TILE;
    const int count = (int)min((int64_t)TILE, n - tbase);
    const int first = w * FMM_WAVE * RS_ITEMS;
    uint64_t k[RS_ITEMS];
    uint32_t v[HAS_VAL ? RS_ITEMS : 1];
#pragma unroll
    for (int r = 0; r < RS_ITEMS; ++r) {
        const int i = min(first + r * FMM_WAVE + lane, count - 1);
        k[r] = keys[tbase + i];
        if (HAS_VAL) v[r] = vals[tbase + i];
    }
    const int all = tid < 256 ? digits[tid] : 0;
    int rank[RS_ITEMS];
#pragma unroll
    for (int r = 0; r < RS_ITEMS; ++r)
        rank[r] = wave_rank(k[r], first + r * FMM_WAVE + lane < count, shift, L.wcount[w]);
    __syncthreads();
    const int mine = wave_offsets(L);
    if (tid < 256) {
        next[(size_t)tile * 256 + tid] = 0;
        entry_store(entry + (size_t)tile * 256 + tid,
                    tile == 0 ? RS_RUNNING + (unsigned)mine : (unsigned)mine + 1u);
    }
    const int st = digit_scan(mine, L.wsum[0]);
    const int gst = digit_scan(all, L.wsum[1]);
    if (tid < 256) L.start[tid] = st;
    __syncthreads();
#pragma unroll
    for (int r = 0; r < RS_ITEMS; ++r) {
        if (first + r * FMM_WAVE + lane < count) {
            const int d = (int)((k[r] >> shift) & 255u);
            const int pos = L.start[d] + L.wcount[w][d] + rank[r];
            skey[pos] = k[r];
            if (HAS_VAL) sval[pos] = v[r];
        }
    }
    if (tid < 256) {
        const int before = tiles_before(entry, tile, tid);
        if (tile > 0)
            entry_store(entry + (size_t)tile * 256 + tid, RS_RUNNING + (unsigned)(before + mine));
        L.base[tid] = gst + before - st;
    }
    __syncthreads();
    for (int i = tid; i < count; i += THREADS) {
        const uint64_t q = skey[i];
        const int pos = L.base[(int)((q >> shift) & 255u)] + i;
        okeys[pos] = q;
        if (HAS_VAL) ovals[pos] = sval[i];
    }
}

// All passes of a short array in one block: 2000 keys with values in eight
// passes 24 us, where 24 launches took 150.
template <bool HAS_VAL>
__global__ void __launch_bounds__(RS_BLOCK_THREADS)
k_rs_block(const uint64_t *keys, const uint32_t *vals, uint64_t *okeys, uint32_t *ovals, int n,
           int lo, int passes) {
    __shared__ TileLds<RS_BLOCK_THREADS> L;
    __shared__ uint64_t skey[RS_BLOCK_KEYS];
    __shared__ uint32_t sval[HAS_VAL ? RS_BLOCK_KEYS : 1];
    const int tid = threadIdx.x, lane = lane_id(), w = tid / FMM_WAVE;
    // the wavefronts share the keys evenly
    const int rounds = (n + RS_BLOCK_THREADS - 1) / RS_BLOCK_THREADS;
    const int first = w * FMM_WAVE * rounds;
    uint64_t k[RS_ITEMS];
    uint32_t v[HAS_VAL ? RS_ITEMS : 1];
#pragma unroll
    for (int r = 0; r < RS_ITEMS; ++r) {
        const int i = min(first + r * FMM_WAVE + lane, n - 1);
        if (r < rounds) {
            k[r] = keys[i];
            if (HAS_VAL) v[r] = vals[i];
        }
    }
    for (int q = 0; q < passes; ++q) {
        const int shift = lo + 8 * q;
        clear_counts(L);
        __syncthreads();
        int rank[RS_ITEMS];
#pragma unroll
        for (int r = 0; r < RS_ITEMS; ++r)
            if (r < rounds)
                rank[r] = wave_rank(k[r], first + r * FMM_WAVE + lane < n, shift, L.wcount[w]);
        __syncthreads();
        const int mine = wave_offsets(L);
        const int st = digit_scan(mine, L.wsum[0]);
        if (tid < 256) L.start[tid] = st;
        __syncthreads();
#pragma unroll
        for (int r = 0; r < RS_ITEMS; ++r) {
            if (r < rounds && first + r * FMM_WAVE + lane < n) {
                const int d = (int)((k[r] >> shift) & 255u);
                const int pos = L.start[d] + L.wcount[w][d] + rank[r];
                skey[pos] = k[r];
                if (HAS_VAL) sval[pos] = v[r];
            }
        }
        __syncthreads();
#pragma unroll
        for (int r = 0; r < RS_ITEMS; ++r) {
            if (r < rounds) {
                const int i = min(first + r * FMM_WAVE + lane, n - 1);
                k[r] = skey[i];
                if (HAS_VAL) v[r] = sval[i];
            }
        }
    }
#pragma unroll
    for (int r = 0; r < RS_ITEMS; ++r) {
        const int i = first + r * FMM_WAVE + lane;
        if (r < rounds && i < n) {
            okeys[i] = k[r];
            if (HAS_VAL) ovals[i] = v[r];
        }
    }
}

}  // namespace

size_t scan_tmp_ints(int64_t n) {
    size_t total = 0;
    int64_t m = n;
    while (m > SCAN_TILE) {
        m = (m + SCAN_TILE - 1) / SCAN_TILE;
        total += (size_t)m;
    }
    return total + 1;
}

namespace {

template <class I, class T>
hipError_t scan(const I *in, T *out, int64_t n, T *tmp, T *total, hipStream_t s) {
    if (n <= 0) {
        if (total) return hipMemsetAsync(total, 0, sizeof(T), s);
        return hipSuccess;
    }
    const int64_t tiles = (n + SCAN_TILE - 1) / SCAN_TILE;
    if (tiles > 1 && n <= SCAN1_MAX) {
        hipLaunchKernelGGL((k_scan_single<I, T>), dim3(1), dim3(SCAN1_THREADS), 0, s, in, out, n,
                           total);
        return hipGetLastError();
    }
    if (tiles == 1) {
        hipLaunchKernelGGL((k_tile_scan<I, T>), dim3(1), dim3(SCAN_THREADS), 0, s, in, out, n,
                           (const T *)nullptr, false, total);
        return hipGetLastError();
    }
    T *sums = tmp;
    hipLaunchKernelGGL((k_tile_sums<I, T>), dim3((unsigned)tiles), dim3(SCAN_THREADS), 0, s, in, n,
                       sums);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    const bool prefixes = tiles > SCAN_TILES;
    if (prefixes) {
        e = scan(sums, sums, tiles, tmp + tiles, (T *)nullptr, s);
        if (e != hipSuccess) return e;
    }
    hipLaunchKernelGGL((k_tile_scan<I, T>), dim3((unsigned)tiles), dim3(SCAN_THREADS), 0, s, in,
                       out, n, (const T *)sums, prefixes, total);
    return hipGetLastError();
}

}  // namespace

hipError_t exclusive_scan(const int *in, int *out, int64_t n, int *tmp, int *total,
                          hipStream_t s) {
    return scan(in, out, n, tmp, total, s);
}

hipError_t exclusive_scan(const int *in, int64_t *out, int64_t n, int64_t *tmp, int64_t *total,
                          hipStream_t s) {
    return scan(in, out, n, tmp, total, s);
}

namespace {

template <bool HAS_VAL>
void launch_pass(int threads, int ntiles, const uint64_t *k, const uint32_t *v, uint64_t *ok,
                 uint32_t *ov, int64_t n, int shift, const SortTmp &T, int q, hipStream_t s) {
    const int *dg = T.digits + 256 * q;
    int *tk = T.tickets + q;
    unsigned *e = T.entry[q & 1], *e2 = T.entry[(q & 1) ^ 1];
    if (threads == 256)
        hipLaunchKernelGGL((k_rs_pass<256, HAS_VAL>), dim3(ntiles), dim3(256), 0, s, k, v, ok, ov,
                           n, shift, dg, tk, e, e2);
    else
        hipLaunchKernelGGL((k_rs_pass<512, HAS_VAL>), dim3(ntiles), dim3(512), 0, s, k, v, ok, ov,
                           n, shift, dg, tk, e, e2);
}

}  // namespace

hipError_t radix_sort(uint64_t **keys, uint64_t **keys_alt, uint32_t **vals,
                      uint32_t **vals_alt, int64_t n, int bits, int *tmp, hipStream_t s,
                      int lo_bit) {
    if (n <= 1 || bits <= 0) return hipSuccess;
    const int passes = (bits + 7) / 8;
    auto flip = [&] {
        std::swap(*keys, *keys_alt);
        if (vals) std::swap(*vals, *vals_alt);
    };
    if (n <= RS_BLOCK_KEYS) {
        if (vals)
            hipLaunchKernelGGL(k_rs_block<true>, dim3(1), dim3(RS_BLOCK_THREADS), 0, s, *keys,
                               *vals, *keys_alt, *vals_alt, (int)n, lo_bit, passes);
        else
            hipLaunchKernelGGL(k_rs_block<false>, dim3(1), dim3(RS_BLOCK_THREADS), 0, s, *keys,
                               (const uint32_t *)nullptr, *keys_alt, (uint32_t *)nullptr, (int)n,
                               lo_bit, passes);
        flip();
        return hipGetLastError();
    }
    const int threads = sort_threads(n);
    const int ntiles = (int)sort_tiles(n, threads);
    SortTmp T;
    T.digits = tmp;
    T.tickets = tmp + RS_MAX_PASSES * 256;
    T.entry[0] = reinterpret_cast<unsigned *>(T.tickets + RS_MAX_PASSES);
    T.entry[1] = T.entry[0] + (size_t)256 * ntiles;
    // the counts, the tickets and the first pass's entries lie side by side
    const int64_t nz = RS_MAX_PASSES * 257 + (int64_t)256 * ntiles;
    hipLaunchKernelGGL(k_rs_zero, dim3((unsigned)((nz + 255) / 256)), dim3(256), 0, s, tmp, nz);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    const int64_t db = (n + RS_DIGITS_THREADS * RS_ITEMS - 1) / (RS_DIGITS_THREADS * RS_ITEMS);
    hipLaunchKernelGGL(k_rs_digits, dim3((unsigned)std::min<int64_t>(db, RS_DIGITS_BLOCKS)),
                       dim3(RS_DIGITS_THREADS), 0, s, *keys, n, lo_bit, passes, T.digits);
    e = hipGetLastError();
    if (e != hipSuccess) return e;
    for (int q = 0; q < passes; ++q) {
        if (vals)
            launch_pass<true>(threads, ntiles, *keys, *vals, *keys_alt, *vals_alt, n,
                              lo_bit + 8 * q, T, q, s);
        else
            launch_pass<false>(threads, ntiles, *keys, nullptr, *keys_alt, nullptr, n,
                               lo_bit + 8 * q, T, q, s);
        e = hipGetLastError();
        if (e != hipSuccess) return e;
        flip();
    }
    return hipSuccess;
}

}  // namespace fmm
