// The x-lines of an atom's truncation sphere in the order in which the force
// projections take them.  Host code too, for the CPU test of the walk.
#pragma once

#include <cmath>

#ifndef __HIPCC__
#define __host__
#define __device__
#endif

namespace sg {

// The sphere's box in grid points, lx .. lx + nxb - 1 and so on around (cx, cy,
// cz); empty along an axis with no grid plane within rcut of the atom.
struct ForceBox {
    double cx, cy, cz, hx, hy, hz, rcut2;
    int lx, ly, lz, nxb, nyb, nzb;
    float fx, per_h, r2;   // the centre in points of the box, points per length, rcut2
};

__host__ __device__ inline ForceBox force_box(double cx, double cy, double cz, double hx, double hy, double hz,
                                              double rcut) {
    ForceBox b{cx, cy, cz, hx, hy, hz, rcut * rcut, 0, 0, 0, 0, 0, 0, 0, 0, 0};
    b.lx = (int)ceil((cx - rcut) / hx);
    b.ly = (int)ceil((cy - rcut) / hy);
    b.lz = (int)ceil((cz - rcut) / hz);
    b.nxb = (int)floor((cx + rcut) / hx) - b.lx + 1;
    b.nyb = (int)floor((cy + rcut) / hy) - b.ly + 1;
    b.nzb = (int)floor((cz + rcut) / hz) - b.lz + 1;
    b.fx = (float)((cx - b.lx * hx) / hx);
    b.per_h = (float)(1.0 / hx);
    b.r2 = (float)b.rcut2;
    return b;
}

constexpr int kForcePoints = 24;   // points of a step

// A step: n points i0, i0 + 1, ... of the box's line (j, k); next .. last is what
// is left of the line.  Start with j = (first line) - stride, next > last.
struct ForceStep {
    int j, k, i0, n, next, last;
};

// The next step of every stride-th line; false past the last.  The part of a line
// inside the sphere is found in single precision and made longer by more than
// its rounding (at most 4e-7 rcut2 under the root, 3e-5 points outside), so that
// no point inside is left out; the caller tests each point.  `uniform`: makes a
// value that all lanes share a scalar.
template <typename F>
__host__ __device__ inline bool force_advance(const ForceBox& b, ForceStep& s, int stride, F uniform) {
    if (b.nyb <= 0) return false;
    while (s.next > s.last) {
        s.j += stride;
        while (s.j >= b.nyb) {
            s.j -= b.nyb;
            ++s.k;
        }
        if (s.k >= b.nzb) return false;
        const float dy = (float)((b.ly + s.j) * b.hy - b.cy), dz = (float)((b.lz + s.k) * b.hz - b.cz);
        const float in2 = b.r2 - dy * dy - dz * dz + 1e-6f * b.r2;
        if (in2 < 0.0f) continue;
        const float half = sqrtf(in2) * b.per_h + 0.02f;
        const int lo = (int)ceilf(b.fx - half), hi = (int)floorf(b.fx + half);
        s.next = uniform(lo > 0 ? lo : 0);
        s.last = uniform(hi < b.nxb - 1 ? hi : b.nxb - 1);
    }
    s.i0 = s.next;
    s.n = s.last - s.i0 + 1 < kForcePoints ? s.last - s.i0 + 1 : kForcePoints;
    s.next += kForcePoints;
    return true;
}

}  // namespace sg
