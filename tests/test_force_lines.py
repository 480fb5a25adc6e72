"""The walk over the lines of an atom's truncation sphere (csrc/force_lines.hpp),
built for the CPU, against all points of the box: every point inside the sphere
is visited once, by one of the strides' walkers, and the walk ends.  Boxes with no,
one, two and three grid planes along an axis (cut-offs below the spacing), odd
strides, and cut-offs of up to 127 spacings, where single precision decides the
ends of the lines near the sphere's rim."""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

MAIN = r"""
#include <cstdio>
#include <cstdlib>
#include <set>
#include <tuple>
#include "force_lines.hpp"
using namespace sg;

// points inside but not visited, points visited twice, steps out of the box
static long check(const ForceBox& b, int stride) {
    std::set<std::tuple<int, int, int>> seen;
    long bad = 0;
    for (int w = 0; w < stride; ++w) {
        ForceStep s{w - stride, 0, 0, 0, 1, 0};
        long steps = 0;
        while (force_advance(b, s, stride, [](int v) { return v; })) {
            if (++steps > 1000000) return -1;
            if (s.j < 0 || s.j >= b.nyb || s.k < 0 || s.k >= b.nzb || s.n < 1 || s.n > kForcePoints) ++bad;
            for (int e = 0; e < s.n; ++e) {
                if (s.i0 + e < 0 || s.i0 + e >= b.nxb) ++bad;
                if (!seen.insert({s.i0 + e, s.j, s.k}).second) ++bad;
            }
        }
    }
    for (int k = 0; k < b.nzb; ++k)
        for (int j = 0; j < b.nyb; ++j)
            for (int i = 0; i < b.nxb; ++i) {
                const double x = (b.lx + i) * b.hx - b.cx, y = (b.ly + j) * b.hy - b.cy, z = (b.lz + k) * b.hz - b.cz;
                if (x * x + y * y + z * z <= b.rcut2 && !seen.count({i, j, k})) ++bad;
            }
    return bad;
}

static double uni(double lo, double hi) { return lo + (hi - lo) * drand48(); }

int main(int argc, char** argv) {
    srand48(7);
    long bad = 0, lost = 0, empty = 0, rim = 0;
    if (argv[1][0] == 'b') {
        for (int t = 0; t < 3000; ++t) {
            const double h = 0.3, rcut = h * uni(0.05, 1.6);
            const ForceBox b = force_box(uni(0, 9), uni(0, 9), uni(0, 9), h, 1.3 * h, 0.8 * h, rcut);
            empty += b.nxb <= 0 || b.nyb <= 0 || b.nzb <= 0;
            const long r = check(b, 1 + t % 5);
            if (r < 0) return printf("endless\n"), 1;
            bad += r;
        }
        for (int t = 0; t < 20; ++t)
            bad += check(force_box(uni(0, 9), uni(0, 9), uni(0, 9), 0.3, 0.25, 0.33, uni(1, 5)), 4);
    } else {
        // single lines that leave the sphere within a few hundredths of a spacing
        // of their middle, where a point lies
        for (int t = 0; t < 200000; ++t) {
            const double h = 0.05, rcut = h * uni(40, 127), u = uni(0.0, 0.06), cx = 3.0 + h * uni(-u, u);
            const double dy = sqrt(rcut * rcut - u * u * h * h);
            // the line y = 2 of the plane z = 0, the only one
            const ForceBox b = force_box(cx, 2.0 + dy, 0.0, h, 1.0, 8.0, rcut);
            const int j = 2 - b.ly, i = 60 - b.lx;
            const double x = 60 * h - cx, y = 2.0 - b.cy;
            if (j < 0 || j >= b.nyb || i < 0 || i >= b.nxb || x * x + y * y > b.rcut2) continue;
            ++rim;
            ForceStep s{j - b.nyb, 0, 0, 0, 1, 0};
            const bool hit = force_advance(b, s, b.nyb, [](int v) { return v; }) && s.j == j && s.k == 0 &&
                             s.i0 <= i && i < s.i0 + s.n;
            lost += !hit;
        }
    }
    printf("bad %ld empty %ld rim %ld lost %ld\n", bad, empty, rim, lost);
    return bad || lost || (argv[1][0] == 'b' ? empty < 100 : rim < 10000);
}
"""


@pytest.fixture(scope="module")
def walk(tmp_path_factory):
    cxx = shutil.which("g++")
    if cxx is None:
        pytest.skip("no host compiler")
    d = tmp_path_factory.mktemp("walk")
    (d / "main.cpp").write_text(MAIN)
    subprocess.run([cxx, "-O1", "-std=c++17", "-ffp-contract=fast", "-I", os.path.join(ROOT, "paper_2005_10431_amd", "csrc"),
                    "-o", str(d / "walk"), str(d / "main.cpp")], check=True)
    return lambda mode: subprocess.run([str(d / "walk"), mode], capture_output=True, text=True, timeout=20)


def test_walk_covers_small_and_empty_boxes(walk):
    r = walk("boxes")
    assert r.returncode == 0, r.stdout


def test_walk_keeps_points_at_the_rim(walk):
    r = walk("rim")
    assert r.returncode == 0, r.stdout
