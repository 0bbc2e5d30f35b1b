"""The FP64 M2L kernel's lanes (m2l_impl.h) run on the CPU against the oracle's
M2L, on lists whose separations lie on the z axis, next to it, or anywhere.

The kernel turns each source's frame about z by the separation's azimuth.  Next
to the axis the squared distance from it underflows, and a cosine and a sine
made from it would not have length 1, which scales what the lane has summed
so far.  Bound: the summed F equals the oracle's to 1e-11 of its largest
coefficient."""
import os
import shutil
import subprocess

import numpy as np
import pytest

import oracle

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_1405_2255_amd", "csrc")
ORDERS = (3, 8, 15)

PROGRAM = r"""
#include <cstdio>
#include <vector>
#include "m2l_impl.h"
int __lane_id() { return 0; }
using namespace fmm;
template <int P>
void run(int ns, std::vector<double4> &cen, std::vector<cplx> &M, std::vector<cplx> &F) {
    std::vector<uint64_t> list(ns);
    for (int i = 0; i < ns; ++i) list[i] = i;
    TreeArrays t{};
    t.cen = cen.data();
    for (int q = 0; q < m2l_detail::pass_count(P); ++q)
        m2l_detail::m2l_passes<P, 0>(q, ns, 0, ns, list.data(), (1ull << 20) - 1, t, M.data(),
                                     F.data());
}
int main(int, char **argv) {
    long long h[2];
    FILE *f = std::fopen(argv[1], "rb");
    if (std::fread(h, 8, 2, f) != 2) return 1;
    const int p = (int)h[0], ns = (int)h[1], nc = (p + 1) * (p + 2) / 2;
    std::vector<double4> cen(ns + 1);
    std::vector<cplx> M((size_t)ns * nc), F(nc, cplx{0.0, 0.0});
    if (std::fread(cen.data(), sizeof(double4), ns + 1, f) != (size_t)ns + 1) return 1;
    if (std::fread(M.data(), sizeof(cplx), M.size(), f) != M.size()) return 1;
    std::fclose(f);
    switch (p) {
#define C(P) case P: run<P>(ns, cen, M, F); break;
    M2L_ORDERS
    default: return 1;
    }
    f = std::fopen(argv[2], "wb");
    std::fwrite(F.data(), sizeof(cplx), nc, f);
    std::fclose(f);
    return 0;
}
"""


@pytest.fixture(scope="module")
def emulator(tmp_path_factory):
    if shutil.which("g++") is None:
        pytest.skip("g++ not available")
    d = tmp_path_factory.mktemp("m2l")
    (d / "m2l.cpp").write_text(PROGRAM)
    orders = " ".join(f"C({p})" for p in ORDERS)
    r = subprocess.run(["g++", "-std=c++20", "-O1", "-Wno-attributes", f"-DM2L_ORDERS={orders}",
                        "-I", os.path.join(ROOT, "tests", "rotation_emu"), "-I", CSRC,
                        str(d / "m2l.cpp"), "-o", str(d / "m2l")], capture_output=True, text=True)
    assert r.returncode == 0, r.stderr[-4000:]
    return d / "m2l"


@pytest.mark.parametrize("p", ORDERS)
@pytest.mark.parametrize("offset", [0.0, 1e-300, 2e-162, 1e-160, 1e-157, 1e-154, 1e-150, 1e-100,
                                    1e-17, 1e-3])
def test_separations_next_to_the_axis(emulator, tmp_path, p, offset):
    rng = np.random.default_rng(17)
    ns = 7
    cen = np.zeros((ns + 1, 4))           # the sink, at the origin, is the last
    cen[:ns, :3] = rng.standard_normal((ns, 3))
    cen[:ns, :3] *= 4.0 / np.linalg.norm(cen[:ns, :3], axis=1)[:, None]
    for k, (x, y) in ((2, (offset, 0.3 * offset)), (3, (0.0, -offset)), (5, (offset, 0.0))):
        cen[k, :3] = (x, y, 4.0 if k != 3 else -4.0)
    NC = (p + 1) * (p + 2) // 2
    M = np.zeros((ns, NC), dtype=np.complex128)
    want = np.zeros((p + 1) ** 2, dtype=np.complex128)
    for k in range(ns):
        x = cen[k, :3] + 0.5 * rng.standard_normal((6, 3))
        full = oracle.p2m(x, rng.random(6), cen[k, :3], p)
        M[k] = [full[n * n + n + m] for n in range(p + 1) for m in range(n + 1)]
        want += oracle.m2l(full, cen[ns, :3] - cen[k, :3], p)
    want = np.array([want[n * n + n + m] for n in range(p + 1) for m in range(n + 1)])
    fin, fout = tmp_path / "in.bin", tmp_path / "out.bin"
    with open(fin, "wb") as f:
        np.array([p, ns], dtype=np.int64).tofile(f)
        cen.tofile(f)
        M.tofile(f)
    subprocess.run([str(emulator), str(fin), str(fout)], check=True)
    got = np.fromfile(fout, dtype=np.complex128)
    assert np.abs(got - want).max() < 1e-11 * np.abs(want).max()
