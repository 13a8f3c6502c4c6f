"""The partial sums of a chain always have room: a call that can lend a chain
nothing besides the workspace's partials region (an Euler step of several
substeps, the second half of a Runge-Kutta step) must fit one into it, for
every grid and every number of products, on devices of any size.

Host arithmetic only: a small program linked against libexpi.so asks the
library's own sizing functions.
"""
import os
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
PKG = os.path.join(ROOT, "paper_1309_4616_amd")

SOURCE = r"""
#include <cstdio>
#include "expi_internal.h"
using namespace expi;
int main() {
    long bad = 0, seen = 0;
    auto check = [&](Op& op, int n0, int n1, int cus) {
        op.n[0] = n0;
        op.n[1] = n1;
        op.size = (int64_t)n0 * n1;
        const size_t region = partials_bytes(op);
        const size_t rooms[] = {region, std::max(region, (size_t)op.size * 8)};
        for (size_t room : rooms)
            for (int n = 2; n <= 6; ++n) {
                if (!chain2d_length(op, n)) continue;
                const size_t b = chain2d_partials(op, n, cus, room);
                ++seen;
                if (b == 0 || b > room) {
                    if (bad++ < 10) std::printf("%d x %d, %d products, %d CUs: %zu of %zu bytes\n", n0, n1, n, cus, b, room);
                }
            }
    };
    Op op;
    op.kind = 0;
    op.dim = 2;
    op.n[2] = 1;
    for (int coef : {EXPI_COEF_CONST, EXPI_COEF_FIELD}) {
        op.coef = coef;
        for (int n0 = 1; n0 <= 1024; ++n0)
            for (int n1 = 1; n1 <= 4200; n1 += (n0 >= 110 && n0 <= 130) ? 1 : 7) check(op, n0, n1, 256);
        for (int cus : {1, 8, 64, 304})
            for (int n0 : {1, 63, 64, 65, 120, 125, 128, 129, 600, 5000, 300000})
                for (int n1 : {1, 2, 5, 12, 100, 999, 2048, 2050, 4000, 100000})
                    if ((int64_t)n0 * n1 < ((int64_t)1 << 28)) check(op, n0, n1, cus);
    }
    std::printf("%ld sizings, %ld without room\n", seen, bad);
    return bad != 0;
}
"""


SOURCE_3D = r"""
#include <cstdio>
#include "expi_internal.h"
using namespace expi;
int main() {
    long bad = 0, seen = 0;
    Op op;
    op.kind = 0;
    op.dim = 3;
    op.coef = EXPI_COEF_CONST;
    const int xs[] = {1, 2, 7, 16, 33, 63, 64, 65, 96, 120, 128, 129, 150, 200, 257, 512, 1000};
    const int ys[] = {1, 2, 3, 8, 9, 40, 64, 65, 130, 250, 256, 700};
    const int zs[] = {1, 3, 4, 5, 17, 32, 33, 111, 256};
    for (int x : xs) for (int y : ys) for (int z : zs) {
        op.n[0] = x; op.n[1] = y; op.n[2] = z;
        op.size = (int64_t)x * y * z;
        const size_t region = partials_bytes(op);
        for (int vec : {1, 2}) for (int waves : {1, 2, 4, 8}) for (int march : {4, 8, 32, 120}) {
            const Tiles t{vec, waves, march};
            if (!tiles_valid(op, t)) continue;
            ++seen;
            if ((size_t)make_geom(op, t).grid * 32 > region && bad++ < 10)
                std::printf("%d x %d x %d, tiles %d %d %d\n", x, y, z, vec, waves, march);
        }
    }
    std::printf("%ld settings, %ld without room\n", seen, bad);
    return bad != 0;
}
"""


def run_program(tmp_path, source):
    if not os.path.exists(os.path.join(PKG, "libexpi.so")):
        from paper_1309_4616_amd import build
        build.build()
    src = tmp_path / "room.cpp"
    src.write_text("#include <algorithm>\n" + source)
    exe = str(tmp_path / "room")
    subprocess.run(["hipcc", "-O2", "-std=c++17", str(src), "-I", os.path.join(PKG, "csrc"), "-I",
                    os.path.join(ROOT, "include"), "-L", PKG, "-lexpi", "-Wl,-rpath," + PKG, "-o", exe], check=True,
                   timeout=300)
    r = subprocess.run([exe], capture_output=True, text=True, timeout=300)
    print(r.stdout)
    assert r.returncode == 0, r.stdout


def test_one_chain_always_fits(tmp_path):
    run_program(tmp_path, SOURCE)


def test_products_fit_whichever_way_rows_are_laid_out(tmp_path):
    run_program(tmp_path, SOURCE_3D)
