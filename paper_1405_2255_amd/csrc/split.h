// How work is split: the keys of a sort over tiles, the sources of exact sums over
// grid rows, the leaves of the near field over parts (host and device; plain
// arithmetic, so that it can be checked without a device).
#pragma once

#include <algorithm>
#include <cstddef>
#include <cstdint>

namespace fmm {

// Radix sort, one launch per pass: tiles of 2048 keys (256 threads of RS_ITEMS);
// of 4096 above RS_WIDE keys, where the chip is full either way and half the tiles
// mean half the way back through their entries (10^6 keys 17.5 us a pass
// against 22; 10^5 keys 9 us with both).
constexpr int RS_ITEMS = 8;               // keys per thread of a tile
constexpr int RS_MAX_PASSES = 8;
constexpr int64_t RS_WIDE = 1 << 17;
constexpr int sort_threads(int64_t n) { return n > RS_WIDE ? 512 : 256; }
constexpr int64_t sort_tiles(int64_t n, int threads) {
    return (n + threads * RS_ITEMS - 1) / (threads * RS_ITEMS);
}
// scratch of a sort of n keys or fewer: digit counts and a ticket per pass, two
// arrays of 256 entries per tile.  2^17 keys have more tiles than a few more keys
// do, and a scratch made for the latter takes them too.
constexpr size_t sort_tmp_ints(int64_t n) {
    const int64_t narrow = sort_tiles(std::min(n, RS_WIDE), 256);
    const int64_t wide = n > RS_WIDE ? sort_tiles(n, 512) : 0;
    return RS_MAX_PASSES * 257 + 2 * 256 * (size_t)std::max(narrow, wide);
}

constexpr int DIRECT_R = 8;               // sinks of a wavefront
constexpr int64_t DIRECT_WAVES = 16384;
constexpr int64_t DIRECT_SOURCES = 512;

// sources per row: row k holds [k len, min(n, (k + 1) len))
constexpr int64_t row_length(int64_t n, int64_t rows) { return (n + rows - 1) / rows; }

// The library's number of rows: about DIRECT_WAVES wavefronts of DIRECT_R sinks
// (16 per SIMD, so that the last ones cost little), rows of at least
// DIRECT_SOURCES and at most 2^31 sources.  Rounding the length up would leave
// rows past the last source (10^6 sources in 1953 rows of 513 end in row
// 1949), so the rows are counted again from the length: each then holds at
// least one source.  With more than one row, rows * nsinks < 2 * DIRECT_WAVES *
// DIRECT_R.
constexpr int64_t direct_rows(int64_t n, int64_t nsinks) {
    const int64_t waves = (nsinks + DIRECT_R - 1) / DIRECT_R;
    const int64_t want = (DIRECT_WAVES + waves - 1) / waves;
    const int64_t rows = std::max(n / (int64_t(1) << 31) + 1, std::min(want, n / DIRECT_SOURCES));
    return row_length(n, row_length(n, rows));
}

// sources in [j0, j1) of a row; 0 where the row begins past its end
constexpr uint32_t slice_length(int64_t j0, int64_t j1) {
    return j1 > j0 ? (uint32_t)(j1 - j0) : 0u;
}

// The near field takes its leaves in parts of about NEAR_ENTRIES list entries (8
// bytes each; at most one leaf's entries more, which are fewer than its sources),
// so that offsets inside a part fit 32 bits and the list's memory is bounded:
// part k holds the leaves whose entries begin in [k NEAR_ENTRIES, (k + 1)
// NEAR_ENTRIES).  10^6 bodies in leaves of 80 have 4e6 entries, in leaves of one
// body 1.7e8 to 2.2e8 (2^31 would come at 10^7 bodies).
constexpr int64_t NEAR_ENTRIES = int64_t(1) << 27;
constexpr int near_parts(int64_t entries) {
    return (int)std::max<int64_t>(1, (entries + NEAR_ENTRIES - 1) / NEAR_ENTRIES);
}
// the first leaf of part k: entry_off holds nleaves + 1 offsets, not decreasing
constexpr int64_t near_part_begin(const int64_t *entry_off, int64_t nleaves, int64_t k) {
    int64_t lo = 0, hi = nleaves;
    while (lo < hi) {
        const int64_t mid = lo + (hi - lo) / 2;
        if (entry_off[mid] < k * NEAR_ENTRIES) lo = mid + 1;
        else hi = mid;
    }
    return lo;
}

}  // namespace fmm
