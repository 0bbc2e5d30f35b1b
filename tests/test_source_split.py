"""How work is split (split.h), checked on the CPU.

Rows of sources of the exact sums: every row begins inside [0, n), the rows
cover it, their number is what the partial sums have room for, and a row that
began past its end would be empty.

Parts of leaves of the near field, with totals past 32 bits: the parts cover the
leaves in order, and an offset inside a part fits 32 bits.

Scratch of a sort: what is enough for n keys is enough for fewer, also where the
tiles change their width."""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

ROWS = r"""
#include <cstdio>
#include "split.h"
int main() {
    const long long scratch = 16ll << 20;      // bytes of the fixed scratch's rows (n < 2^30)
    long long bad = 0, cases = 0;
    auto check = [&](int64_t n, int64_t k) {
        const int64_t rows = fmm::direct_rows(n, k), len = fmm::row_length(n, rows);
        const bool ok = rows >= 1 && rows <= 65535 && len >= 1 && len <= (int64_t(1) << 31) &&
                        (rows - 1) * len < n && rows * len >= n &&
                        (rows == 1 || n > 1073741823 || rows * k * 32 <= scratch);
        ++cases;
        if (!ok && bad++ < 5)
            std::printf("n %lld sinks %lld rows %lld of %lld\n", (long long)n, (long long)k,
                        (long long)rows, (long long)len);
    };
    for (int64_t n = 1; n <= 10000000; n += 1 + n / 97)
        for (int64_t k = 1; k <= 16384; k += 1 + k / 23) {
            check(n, k);
            check(n + 1, k);
        }
    for (int64_t n : {500000ll, 1000000ll, 1000001ll, 1999999ll, 10000000ll, 1073741823ll})
        for (int64_t k = 1; k <= 20000; ++k) check(n, k);
    for (int64_t n = 1; n <= 1073741823; n += 1 + n / 7) check(n, n);
    check(3ll << 31, 3ll << 31);
    if (fmm::slice_length(5, 5) != 0 || fmm::slice_length(6, 5) != 0 ||
        fmm::slice_length(5, 69) != 64)
        ++bad;
    std::printf("%lld cases, %lld bad\n", cases, bad);
    return bad != 0;
}
"""


PARTS = r"""
#include <cstdio>
#include <vector>
#include "split.h"
int main() {
    uint64_t x = 88172645463325252ull;
    auto random = [&]() { x ^= x << 13; x ^= x >> 7; x ^= x << 17; return x; };
    long long bad = 0;
    // leaves and the most entries of one
    const int64_t sizes[][2] = {{1, 1}, {1, 1 << 30}, {7, 100}, {1000, 1 << 28}, {100000, 500},
                                {100000, 100000}, {3000000, 2000}, {3000000, 40}, {5, 0}};
    for (auto &z : sizes) {
        const int64_t nl = z[0];
        std::vector<int64_t> off(nl + 1, 0);
        int64_t largest = 0;
        for (int64_t l = 0; l < nl; ++l) {
            // (leaves without sinks have none)
            const int64_t e = random() % 4 ? random() % (z[1] + 1) : 0;
            off[l + 1] = off[l] + e;
            largest = std::max(largest, e);
        }
        const int parts = fmm::near_parts(off[nl]);
        bad += parts < 1 || (off[nl] <= fmm::NEAR_ENTRIES) != (parts == 1);
        int64_t last = 0;
        for (int k = 0; k < parts; ++k) {
            const int64_t b = fmm::near_part_begin(off.data(), nl, k);
            const int64_t e = k + 1 < parts ? fmm::near_part_begin(off.data(), nl, k + 1) : nl;
            const int64_t size = off[e] - off[b];
            bad += (k == 0 && b != 0) || (k > 0 && b != last) || e < b;
            bad += size > fmm::NEAR_ENTRIES + largest || size >= (int64_t(1) << 31);
            last = e;
        }
        std::printf("%lld leaves, %lld entries, %d parts\n", (long long)nl, (long long)off[nl],
                    parts);
    }
    return bad != 0;
}
"""


SCRATCH = r"""
#include <cstdio>
#include "split.h"
int main() {
    long long bad = 0;
    size_t before = 0;
    for (int64_t n = 0; n <= (int64_t(1) << 31); n += n < 600000 ? 1 : n / 50) {
        const size_t have = fmm::sort_tmp_ints(n);
        const size_t used = fmm::RS_MAX_PASSES * 257 +
                            512 * (size_t)fmm::sort_tiles(n, fmm::sort_threads(n));
        if ((have < before || have < used) && bad++ < 5)
            std::printf("n %lld: %zu ints, used %zu, before %zu\n", (long long)n, have, used,
                        before);
        before = have;
    }
    return bad != 0;
}
"""


def _run(tmp_path, program):
    if shutil.which("g++") is None:
        pytest.skip("g++ not available")
    src, exe = tmp_path / "split.cpp", tmp_path / "split"
    src.write_text(program)
    r = subprocess.run(["g++", "-std=c++20", "-O1", "-Wall", "-Werror", "-fsanitize=undefined",
                        "-fno-sanitize-recover=undefined",
                        "-I", os.path.join(ROOT, "paper_1405_2255_amd", "csrc"), str(src), "-o",
                        str(exe)], capture_output=True, text=True)
    assert r.returncode == 0, r.stderr[-4000:]
    r = subprocess.run([str(exe)], capture_output=True, text=True)
    assert r.returncode == 0, r.stdout + r.stderr
    return r.stdout


def test_every_row_holds_sources(tmp_path):
    _run(tmp_path, ROWS)


def test_offsets_inside_a_part_fit_32_bits(tmp_path):
    out = _run(tmp_path, PARTS)
    # the largest totals are past what 32 bits hold
    assert max(int(line.split()[2]) for line in out.splitlines()) > 1 << 32


def test_scratch_of_a_sort_grows_with_the_keys(tmp_path):
    _run(tmp_path, SCRATCH)
