"""The rows that the exact sums cut their sources into (split.h), checked on the
CPU: every row begins inside [0, n), the rows cover it, their number is what the
partial sums have room for, and a row that began past its end would be empty."""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

PROGRAM = r"""
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


def test_every_row_holds_sources(tmp_path):
    if shutil.which("g++") is None:
        pytest.skip("g++ not available")
    src, exe = tmp_path / "split.cpp", tmp_path / "split"
    src.write_text(PROGRAM)
    r = subprocess.run(["g++", "-std=c++20", "-O1", "-Wall", "-Werror", "-fsanitize=undefined",
                        "-fno-sanitize-recover=undefined",
                        "-I", os.path.join(ROOT, "paper_1405_2255_amd", "csrc"), str(src), "-o",
                        str(exe)], capture_output=True, text=True)
    assert r.returncode == 0, r.stderr[-4000:]
    r = subprocess.run([str(exe)], capture_output=True, text=True)
    assert r.returncode == 0, r.stdout + r.stderr
