// Nonlocal term of H (Sec. 2.1: applied through its outer products),
// V_nl x = sum_I sum_lm chi_Ilm D_Ilm with D = gamma dV chi^T x, and its Bloch
// form, whose passes are the same over the halves [Re; Im] of a column and whose
// phases enter with the sum over an atom's entries (k_nl_reduce_k).
//
// The projections D of a block and their application are products with a
// tall matrix that every orbital shares: chi on a tile of the grid, against
// 16 orbitals at a time, on MFMA.  One pass over the block does
//   apply    y += chi D     and / or     project    D' = alpha gamma dV chi^T y,
// so a filter step is one local sweep followed by one pass that completes
// its output and forms the projections the next step needs.
//
// Layout of the pass (one workgroup = one unit x up to 64 orbitals, 16 per
// wave):
//  - the points of a z-plane are cut into blocks of 16 consecutive points
//    (one 128-byte line in FP64, aligned whenever n_x n_y is a multiple of
//    16), so that a wave reads and writes whole lines of every orbital: on
//    24-point pieces of rows instead, a plain read and write of the block
//    ran at 2.9 instead of 4.3 TB/s at 120^3 x 1200;
//  - a pencil is up to kNlBlocks blocks that lie close together in x and y; a
//    unit is a pencil over a range of z, of which few columns take more and
//    shorter ones (nl_shape);
//  - along the unit's planes every (atom, image) pair that reaches it holds
//    one of S slots for its z extent.  A slot's 4 projections stay in
//    accumulators and its 4 coefficients in registers until it leaves, when
//    the sums are written as one partial entry (entry, orbital, lm); the
//    entries of an atom are added in a fixed order by k_nl_reduce, so results
//    are bitwise reproducible.  The order goes with the number of columns of the
//    call, not with the groups that they are taken in;
//  - per plane the workgroup tabulates chi of the plane's points x slots in
//    LDS, shared by its orbitals; slots go in groups of four (16 projectors,
//    one MFMA row tile) and a block skips the groups that do not touch it (a
//    block of a 4.5-Bohr lattice meets 5.3 pairs in 2.15 groups on average).
// The accumulator layout of the apply product is the operand layout of the
// projection product, so a value goes from its load through both without
// leaving its lane.
//
// The products run over whole blocks and groups of slots, with chi = 0 where a
// pair does not reach.  Zero times an infinity or a NaN would carry these past an
// atom's support, so they go round the products.  The sum over an atom's entries
// forms a projection that is not finite again from the atom's points alone
// (sum_support) and marks its 16 columns; in marked columns the pass applies what
// is not finite point by point (plane_odd).
#include <algorithm>
#include <array>
#include <cmath>
#include <map>
#include <mutex>
#include <type_traits>

#include "internal.hpp"
#include "mfma.hpp"

namespace sg {

namespace {

constexpr int kIdle = 255;          // slot without a pair
constexpr int kMaxLocal = 112;      // pairs of a unit (with 24 slots and 128 planes 106 KB of LDS in FP64)
constexpr int kMaxPlanes = 128;     // planes of a unit
constexpr int kMaxSlots = 24;
constexpr int kNlWaves = 4;         // waves of a workgroup, 16 orbitals each
constexpr int kNlSplit = 3;         // or three that share the blocks of 16 orbitals
constexpr double kNlSplitPlane = 0.65;   // and time of a plane then

template <typename T, int N>
struct NlVec {
    typedef T type __attribute__((ext_vector_type(N), aligned(sizeof(T))));
};

// The four points (of a block's 16) that lane group g holds when the products
// run in C, and the point of MFMA row i.  T: type in memory.
template <typename C>
struct Pts;
template <>
struct Pts<double> {
    static __device__ inline int of(int g, int r) { return 2 * g + (r & 1) + 8 * (r >> 1); }
    static __device__ inline int row(int i) { return 2 * (i & 3) + ((i >> 2) & 1) + 8 * (i >> 3); }
    // position of MFMA row i (slot i % 4, lm i / 4) among a group's 16 (slot, lm) values
    static __device__ inline int perm(int i) { return 4 * (i & 3) + (i >> 2); }
    template <typename T>
    static __device__ inline void load(const T* x, int p0, int g, T* q) {
        using v2 = typename NlVec<T, 2>::type;
        const v2 a = *reinterpret_cast<const v2*>(x + p0 + 2 * g);
        const v2 b = *reinterpret_cast<const v2*>(x + p0 + 2 * g + 8);
        q[0] = a.x;
        q[1] = a.y;
        q[2] = b.x;
        q[3] = b.y;
    }
    template <typename T>
    static __device__ inline void store(T* x, int p0, int g, const T* q) {
        using v2 = typename NlVec<T, 2>::type;
        *reinterpret_cast<v2*>(x + p0 + 2 * g) = v2{q[0], q[1]};
        *reinterpret_cast<v2*>(x + p0 + 2 * g + 8) = v2{q[2], q[3]};
    }
};
template <>
struct Pts<float> {
    static __device__ inline int of(int g, int r) { return 4 * g + r; }
    static __device__ inline int row(int i) { return i; }
    static __device__ inline int perm(int i) { return i; }
    static __device__ inline void load(const float* x, int p0, int g, float* q) {
        using v4 = typename NlVec<float, 4>::type;
        const v4 a = *reinterpret_cast<const v4*>(x + p0 + 4 * g);
        q[0] = a.x;
        q[1] = a.y;
        q[2] = a.z;
        q[3] = a.w;
    }
    static __device__ inline void store(float* x, int p0, int g, const float* q) {
        using v4 = typename NlVec<float, 4>::type;
        *reinterpret_cast<v4*>(x + p0 + 4 * g) = v4{q[0], q[1], q[2], q[3]};
    }
};

template <typename T, typename C>
struct NlArgs {
    T* y;
    long ldx;
    int halves;                  // 0: column j at j ldx; 1: at (j / 2) ldx + (j % 2) half (Bloch columns)
    long half;
    int by_pair;                 // D per (atom, image) pair (Bloch) or per atom
    int nx, ny, nz, nxy, ncol;
    int nwc, nchunk, nunit;      // MFMA waves per workgroup, column chunks, units
    int zlen, ncl;               // most planes and pairs of a unit
    const NlUnit* units;
    const int* blk;              // first points of the kNlBlocks blocks of each pencil, -1 pads
    int tail;                    // n_x n_y % 16
    T* dummy;                    // 256 values: where the places past a pencil's list store
    const uint8_t* occ;          // per unit zlen x S: pair (local index) in each slot
    const uint64_t* gm;          // per unit zlen: bit b S/4 + G: block b meets group G
    const int* ent_cand;         // pair of every entry
    const NlCand* cand;
    double hx, hy, hz, inv_rc2, N0, N1, rcut2;
    const C* D;                  // column j at D + j ldD, 4 per pair or atom
    long ldD;
    uint32_t* odd;               // per 16 columns: epoch if a coefficient is not finite
    uint32_t epoch;
    double* part;                // [(entry ncol + col) 4 + lm]
    const C* zero;               // coefficients of a slot without a pair
    double* alpha;               // project: alpha of the filter step (mode, step) that will apply D
    const double* params;
    int mode, step;
};

// Planes of the sums of one group: FP64 in the accumulators; in FP32 the MFMA
// sums of one plane (at most 96 points) are added to FP64 sums.
template <typename T>
struct GroupSum;
template <>
struct GroupSum<double> {
    typename Mfma<double>::acc_t p{0, 0, 0, 0};
    __device__ inline void plane() {}
    __device__ inline double get(int r) const { return p[r]; }
    __device__ inline void zero() { p = Mfma<double>::acc_t{0, 0, 0, 0}; }
};
template <>
struct GroupSum<float> {
    typename Mfma<float>::acc_t p{0, 0, 0, 0};
    double s[4] = {0, 0, 0, 0};
    __device__ inline void plane() {
#pragma unroll
        for (int r = 0; r < 4; ++r) s[r] += (double)p[r];
        p = Mfma<float>::acc_t{0, 0, 0, 0};
    }
    __device__ inline double get(int r) const { return s[r]; }
    __device__ inline void zero() {
        p = Mfma<float>::acc_t{0, 0, 0, 0};
#pragma unroll
        for (int r = 0; r < 4; ++r) s[r] = 0;
    }
};

struct NlLds {
    size_t gxy, ez, gm, cand, xy, occ, total;
};

__host__ __device__ inline NlLds nl_lds_layout(size_t ts, int S, int zlen, int ncl) {
    auto up = [](size_t v) { return (v + 15) & ~(size_t)15; };
    NlLds L{};
    const size_t np = 16 * kNlBlocks;
    size_t o = up(np * (4 * S + 4) * ts);   // chi of the current plane
    L.gxy = o;                              // per (slot, point): the Gaussian's x-y factor
    o += up(np * S * ts);
    L.ez = o;                               // per plane parity and slot: z factor, dz
    o += 2 * (size_t)S * 16;
    L.gm = o;
    o += up((size_t)zlen * 8);
    L.cand = o;
    o += up((size_t)ncl * sizeof(NlCand));
    L.xy = o;
    o += up(np * sizeof(int));
    L.occ = o;
    o += up((size_t)(zlen + 1) * S);
    L.total = o;
    return L;
}

// Offsets and squared distances of grid points from an image's centre in the
// host tables' own operations (dx^2 + dy^2, then + dz^2), so that a point is
// inside rcut exactly when the tables say so.
__device__ inline double off_x(const NlCand& c, int x, double hx) {
#pragma clang fp contract(off)
    return (x + c.bx) * hx - c.px;
}
__device__ inline double off_y(const NlCand& c, int y, double hy) {
#pragma clang fp contract(off)
    return (y + c.by) * hy - c.py;
}
__device__ inline double off_z(const NlCand& c, int z, double hz) {
#pragma clang fp contract(off)
    return (z + c.bz) * hz - c.pz;
}
__device__ inline double sum_sq(double u, double v) {
#pragma clang fp contract(off)
    return u * u + v * v;
}
__device__ inline double add_sq(double r2, double d) {
#pragma clang fp contract(off)
    return r2 + d * d;
}

// AP: y += chi D (1) or y = chi D (2).  PR: partial projections of (the completed)
// y.  WB: blocks of a wave: all of the pencil's, or a third of them, when the waves
// of a workgroup share 16 columns and leave a partial entry each (see nl_shape).
// Per plane: barrier; chi of the plane into LDS; barrier; the products.  Two
// workgroups of four waves fit a compute unit (71 KB of LDS each), so one's
// table overlaps the other's products.  A wave has the loads of a whole plane
// (12 KB in FP64) in flight: with half of that and six waves per workgroup
// the pass took 9.5 instead of 8.3 ms at 120^3 x 1200 in FP64.  With 24 slots in
// FP64 the LDS holds one workgroup, which has the registers of both (within half of
// them it spilled: 72^3 x 130, supports of 4.1 Bohr, a filter step 1130 us, now 820).
template <typename T, typename C, int S, int WB, int AP, bool PR, bool TAIL>
__global__ __launch_bounds__(64 * kNlWaves, S == kMaxSlots && sizeof(C) == 8 ? 1 : 2) void k_nl_pass(
    NlArgs<T, C> a) {
    using P = Pts<C>;
    using acc_t = typename Mfma<C>::acc_t;
    constexpr int NB = kNlBlocks, NG = S / 4, RS = 4 * S + 4, NP = 16 * NB;
    constexpr int NW = NB / WB;   // waves that share a unit's blocks
    extern __shared__ __align__(16) unsigned char smem_raw[];
    const NlLds L = nl_lds_layout(sizeof(C), S, a.zlen, a.ncl);
    C* chi = reinterpret_cast<C*>(smem_raw);
    C* gxy = reinterpret_cast<C*>(smem_raw + L.gxy);
    double* ezdz = reinterpret_cast<double*>(smem_raw + L.ez);
    uint64_t* gml = reinterpret_cast<uint64_t*>(smem_raw + L.gm);
    NlCand* cand = reinterpret_cast<NlCand*>(smem_raw + L.cand);
    int* xy = reinterpret_cast<int*>(smem_raw + L.xy);
    uint8_t* occ = reinterpret_cast<uint8_t*>(smem_raw + L.occ);

    // block b runs on XCD b % 8.  All units of 64 orbitals go before the next
    // orbitals, the last ones first, which the sweep before has left in the
    // last-level cache; an XCD takes a contiguous eighth of the units, a different
    // one each time, since some hold one more
    if (PR && blockIdx.x == 0 && threadIdx.x == 0) {
        double csh, beta;
        filter_coefs(a.params, a.mode, a.step, *a.alpha, csh, beta);
    }
    const int bslot = blockIdx.x / 8, per = (a.nunit + 7) / 8;
    const int chunk = a.nchunk - 1 - bslot / per, xr = (blockIdx.x + 3 * chunk) % 8;
    const int u = a.nunit / 8 * xr + min(xr, a.nunit % 8) + bslot % per;
    if (bslot % per >= a.nunit / 8 + (xr < a.nunit % 8 ? 1 : 0)) return;
    const NlUnit U = a.units[u];
    const int nzl = U.ze - U.zb;
    const int t = threadIdx.x, nt = blockDim.x;
    const int* blk = a.blk + (long)U.pencil * NB;
    // the last block of a plane whose points are no multiple of 16 starts
    // early; it sits in the last place and leaves the points that the block
    // before it owns alone
    const bool part5 = a.tail && blk[NB - 1] == a.nxy - 16;
    const int nb = U.nb - (part5 ? 1 : 0);   // blocks in the first places
    T* const dummy = a.dummy + 16 * (threadIdx.x & 15);

    // the unit's tables
    for (int j = t; j < nzl; j += nt) gml[j] = a.gm[(long)u * a.zlen + j];
    for (int j = t; j < (nzl + 1) * S; j += nt) occ[j] = j < nzl * S ? a.occ[(long)u * a.zlen * S + j] : (uint8_t)kIdle;
    for (int j = t; j < U.ncl; j += nt) cand[j] = a.cand[a.ent_cand[U.ebase + j]];
    for (int j = t; j < NP; j += nt) {
        const int p = blk[j / 16] + j % 16;
        const bool own = blk[j / 16] >= 0 && !(part5 && j / 16 == NB - 1 && j % 16 < 16 - a.tail);
        xy[j] = own ? (p % a.nx) | (p / a.nx) << 16 : -1;
    }
    __syncthreads();

    // z factor and dz of the slots' pairs at plane zl (by the wave without columns, if any)
    const int zt = NW > 1 ? t - 64 * NW : t;
    auto zfactor = [&](int zl) {
        if (zt >= 0 && zt < S) {
            const int o = occ[zl * S + zt];
            if (o != kIdle) {
                const double dz = off_z(cand[o], U.zb + zl, a.hz);
                double* e = ezdz + ((zl & 1) * S + zt) * 2;
                e[0] = exp(-dz * dz * a.inv_rc2);
                e[1] = dz;
            }
        }
    };
    // chi of plane zl: point-major rows of (slot, lm), zero where the pair
    // does not reach.  A thread keeps the same (slot, point) places through
    // the planes; it forms the x-y Gaussian when a pair enters the slot.  Waves that
    // share their columns leave registers for the places' offsets too (KEEP; one
    // column at 120^3, project and apply: 145 and 156 us without, 127 and 140 with).
    // With whole columns these cost the second workgroup's registers (FP32) or
    // give nothing (FP64).
    constexpr int NE = NP * S / (64 * kNlWaves);   // places of a thread
    constexpr bool KEEP = WB < NB && sizeof(C) == 8 && S <= 16;
    struct Place {
        double dx, dy;   // dx 1e150: no pair, or a point that the pencil does not own
        C g;
    };
    Place pl[KEEP ? NE : 1];
    auto build = [&](int zl) {
        const uint64_t gm = gml[zl];
        auto put_chi = [&](int s, int q, bool in, C gx, C dx, C dy, double ez, double dz) __attribute__((always_inline)) {
            const C ex = gx * (C)ez, e1 = (C)a.N1 * ex;
            C* r = chi + q * RS + 4 * s;
            r[0] = in ? (C)a.N0 * ex : (C)0;
            r[1] = in ? e1 * dx : (C)0;
            r[2] = in ? e1 * dy : (C)0;
            r[3] = in ? e1 * (C)dz : (C)0;
        };
        if constexpr (KEEP) {
            // opaque, so that the places' addresses are formed here again and not
            // kept in registers along the planes
            int tt = t;
            asm volatile("" : "+v"(tt));
            // the table reads of several places at a time, so that their waits are one
            constexpr int BT = AP && PR ? 3 : NE;
#pragma unroll
            for (int i0 = 0; i0 < NE; i0 += BT) {
                int s[BT], q[BT], on[BT], was[BT];
#pragma unroll
                for (int i = 0; i < BT; ++i) {
                    const int e = tt + 64 * kNlWaves * (i0 + i);
                    s[i] = e / NP;
                    q[i] = e - s[i] * NP;
                    on[i] = occ[zl * S + s[i]];
                    was[i] = occ[max(zl - 1, 0) * S + s[i]];
                }
                double z[BT][2];
#pragma unroll
                for (int i = 0; i < BT; ++i)
#pragma unroll
                    for (int j = 0; j < 2; ++j) z[i][j] = ezdz[((zl & 1) * S + s[i]) * 2 + j];
#pragma unroll
                for (int i = 0; i < BT; ++i) {
                    if (zl != 0 && on[i] == was[i]) continue;
                    Place& v = pl[i0 + i];
                    const int w = xy[q[i]];
                    v = Place{1e150, 0.0, 0};
                    if (on[i] != kIdle && w >= 0) {
                        v.dx = off_x(cand[on[i]], w & 0xFFFF, a.hx);
                        v.dy = off_y(cand[on[i]], w >> 16, a.hy);
                        v.g = (C)exp(-sum_sq(v.dx, v.dy) * a.inv_rc2);
                    }
                }
#pragma unroll
                for (int i = 0; i < BT; ++i) {
                    const Place& v = pl[i0 + i];
                    if ((gm >> ((q[i] >> 4) * NG + (s[i] >> 2))) & 1)
                        put_chi(s[i], q[i], add_sq(sum_sq(v.dx, v.dy), z[i][1]) <= a.rcut2, v.g, (C)v.dx, (C)v.dy, z[i][0],
                                z[i][1]);
                }
            }
        } else {
            for (int e = t; e < NP * S; e += nt) {
                const int s = e / NP, q = e - s * NP;
                const int o = occ[zl * S + s], w = xy[q];
                const bool live = o != kIdle && w >= 0;
                double dx = 0, dy = 0, r2 = 0;
                if (live) {
                    dx = off_x(cand[o], w & 0xFFFF, a.hx);
                    dy = off_y(cand[o], w >> 16, a.hy);
                    r2 = sum_sq(dx, dy);
                    if (zl == 0 || occ[(zl - 1) * S + s] != o) gxy[e] = (C)exp(-r2 * a.inv_rc2);
                }
                if (!((gm >> ((q >> 4) * NG + (s >> 2))) & 1)) continue;
                C v0 = 0, v1 = 0, v2 = 0, v3 = 0;
                if (live) {
                    const double* z = ezdz + ((zl & 1) * S + s) * 2;
                    if (add_sq(r2, z[1]) <= a.rcut2) {
                        const C ex = gxy[e] * (C)z[0];
                        const C e1 = (C)a.N1 * ex;
                        v0 = (C)a.N0 * ex;
                        v1 = e1 * (C)dx;
                        v2 = e1 * (C)dy;
                        v3 = e1 * (C)z[1];
                    }
                }
                C* r = chi + q * RS + 4 * s;
                r[0] = v0;
                r[1] = v1;
                r[2] = v2;
                r[3] = v3;
            }
        }
    };

    const int wv = t >> 6, lane = t & 63, li = lane & 15, g = lane >> 4;
    // waves without columns only help to build; lanes past the last column
    // repeat it (the same loads, results and stores)
    const int part = NW == 1 ? 0 : __builtin_amdgcn_readfirstlane(wv), b0 = WB * part;   // the wave's blocks: b0 ..
    const int tile = NW == 1 ? chunk * a.nwc + wv : chunk;                               // and 16 columns
    const bool mine = (NW == 1 ? wv < a.nwc : wv < NW) && 16 * tile < a.ncol;
    const int cl = 16 * tile + li, col = min(cl, a.ncol - 1);
    T* yc = a.y + (long)(col >> a.halves) * a.ldx + (long)(col & a.halves) * a.half;

    GroupSum<C> sum[NG];
    C d[NG][4];
    int oc[NG];
#pragma unroll
    for (int G = 0; G < NG; ++G) {
        oc[G] = kIdle;
#pragma unroll
        for (int j = 0; j < 4; ++j) d[G][j] = 0;
    }
    // the lane's slot of each group at plane zl: a pair that left leaves its
    // sums behind, one that came brings its coefficients
    auto slots = [&](int zl) {
#pragma unroll
        for (int G = 0; G < NG; ++G) {
            const int on = occ[zl * S + 4 * G + g];
            if (on == oc[G]) continue;
            if (PR) {
                if (oc[G] != kIdle && cl < a.ncol) {
                    double* q = a.part + (((long)(U.ebase + oc[G]) * NW + part) * a.ncol + col) * 4;
#pragma unroll
                    for (int r = 0; r < 4; ++r) q[r] = sum[G].get(r);
                }
                sum[G].zero();
            }
            if (AP) {
                // plain loads, nothing that would wait for them (and for those of the
                // next plane's blocks, which are in flight) before the next plane
                const C* Dc = a.zero;
                if (on != kIdle) Dc = a.D + (long)col * a.ldD + 4 * (a.by_pair ? cand[on].id : cand[on].atom);
#pragma unroll
                for (int j = 0; j < 4; ++j) d[G][j] = Dc[j];
            }
            oc[G] = on;
        }
    };
    // first point of each block (in scalar registers); places past the
    // pencil's list load the plane's first points and meet no group
    int pb0[WB];
#pragma unroll
    for (int b = 0; b < WB; ++b) pb0[b] = __builtin_amdgcn_readfirstlane(mine ? max(0, blk[b0 + b]) : 0);
    T q[WB][4];   // the blocks of a plane
    auto load = [&](T* v, int b, int z) {
        if constexpr (AP == 2) v[0] = v[1] = v[2] = v[3] = 0;
        else P::load(yc + (long)z * a.nxy, pb0[b], g, v);
    };
    // some coefficients of the wave's columns may not be finite
    const bool odd = AP && mine && a.odd[tile] == a.epoch;
    // a plane of such columns: block by block as in the loop below, with the
    // coefficients that are not finite at the points that their pairs reach only
    auto plane_odd = [&](int z, uint64_t gm) {
        const int zl = z - U.zb;
        const C* Dc = a.D + (long)col * a.ldD;
#pragma unroll
        for (int G = 0; G < NG; ++G)
            if (!(__builtin_isfinite(d[G][0]) && __builtin_isfinite(d[G][1]) && __builtin_isfinite(d[G][2]) &&
                  __builtin_isfinite(d[G][3])))
#pragma unroll
                for (int j = 0; j < 4; ++j) d[G][j] = 0;
#pragma unroll 1
        for (int b = b0; b < b0 + WB; ++b) {
            const bool tail = TAIL && b == NB - 1 && part5;
            if (b >= nb && !tail) continue;
            const uint32_t gb = (uint32_t)(gm >> (b * NG)) & ((1u << NG) - 1);
            T* yp = yc + (long)z * a.nxy + blk[b];
            T v[4] = {0, 0, 0, 0};
            if (AP != 2) P::load(yp, 0, g, v);
            acc_t acc = {(C)v[0], (C)v[1], (C)v[2], (C)v[3]};
            const C* cb = chi + 16 * b * RS;
#pragma unroll
            for (int G = 0; G < NG; ++G)
                if ((gb >> G) & 1)
#pragma unroll
                    for (int j = 0; j < 4; ++j)
                        acc = Mfma<C>::run(cb[P::row(li) * RS + 16 * G + 4 * g + j], d[G][j], acc);
#pragma unroll 1
            for (int s = 0; s < S; ++s) {
                const int o = occ[zl * S + s];
                if (o == kIdle || !((gb >> (s >> 2)) & 1)) continue;
                const C* e = Dc + 4 * (a.by_pair ? cand[o].id : cand[o].atom);
                const C e0 = e[0], e1 = e[1], e2 = e[2], e3 = e[3];
                if (__builtin_isfinite(e0) && __builtin_isfinite(e1) && __builtin_isfinite(e2) && __builtin_isfinite(e3))
                    continue;
                const double dz = ezdz[((zl & 1) * S + s) * 2 + 1];
#pragma unroll
                for (int r = 0; r < 4; ++r) {
                    const int w = xy[16 * b + P::of(g, r)];
                    const double dx = off_x(cand[o], w & 0xFFFF, a.hx), dy = off_y(cand[o], w >> 16, a.hy);
                    const C* c = cb + P::of(g, r) * RS + 4 * s;
                    if (w >= 0 && add_sq(sum_sq(dx, dy), dz) <= a.rcut2)
                        acc[r] += c[0] * e0 + c[1] * e1 + c[2] * e2 + c[3] * e3;
                }
            }
#pragma unroll
            for (int r = 0; r < 4; ++r)
                if (!tail || P::of(g, r) >= 16 - a.tail) yp[P::of(g, r)] = (T)acc[r];
            if (PR) {
#pragma unroll
                for (int G = 0; G < NG; ++G)
                    if ((gb >> G) & 1)
#pragma unroll
                        for (int r = 0; r < 4; ++r)
                            sum[G].p = Mfma<C>::run(cb[P::of(g, r) * RS + 16 * G + P::perm(li)], acc[r], sum[G].p);
            }
        }
        if (PR) {
#pragma unroll
            for (int G = 0; G < NG; ++G) sum[G].plane();
        }
    };
    if (mine) {
#pragma unroll
        for (int b = 0; b < WB; ++b) load(q[b], b, U.zb);
        slots(0);
    }
    zfactor(0);

    for (int z = U.zb; z < U.ze; ++z) {
        const int zl = z - U.zb;
        __syncthreads();
        build(zl);
        __syncthreads();
        if (zl + 1 < nzl) zfactor(zl + 1);
        if (!mine) continue;
        const uint64_t gv = gml[zl];
        const uint32_t glo = __builtin_amdgcn_readfirstlane((int)(uint32_t)gv);
        const uint32_t ghi = __builtin_amdgcn_readfirstlane((int)(uint32_t)(gv >> 32));
        const uint64_t gm = (uint64_t)ghi << 32 | glo;
        if (AP && __builtin_expect(odd, 0)) {
            plane_odd(z, gm);
#pragma unroll
            for (int b = 0; b < WB; ++b) load(q[b], b, min(z + 1, U.ze - 1));
            slots(zl + 1);
            continue;
        }
#pragma unroll
        for (int b = 0; b < WB; ++b) {
            const uint32_t gb = (uint32_t)(gm >> ((b0 + b) * NG)) & ((1u << NG) - 1);
            T* v = q[b];
            acc_t acc = {(C)v[0], (C)v[1], (C)v[2], (C)v[3]};
            // the block's next plane; loads and stores take no
            // branch, so that those in flight can be counted
            load(v, b, min(z + 1, U.ze - 1));
            const C* cb = chi + 16 * (b0 + b) * RS;
            // with both products the operands of the second are read along with
            // the first's, so that only one wait on LDS is left per group
            // (72^3 x 260: FP32 590 -> 550 us a degree, FP64 within 1%)
            C pr[NG][4];
            if (AP) {
                const C* A = cb + P::row(li) * RS + 4 * g;
#pragma unroll
                for (int G = 0; G < NG; ++G)
                    if ((gb >> G) & 1) {
                        C w[4];
#pragma unroll
                        for (int j = 0; j < 4; ++j) w[j] = A[16 * G + j];
                        if (PR) {
#pragma unroll
                            for (int r = 0; r < 4; ++r) pr[G][r] = cb[P::of(g, r) * RS + 16 * G + P::perm(li)];
                        }
#pragma unroll
                        for (int j = 0; j < 4; ++j) acc = Mfma<C>::run(w[j], d[G][j], acc);
                    }
                T* yp = yc + (long)z * a.nxy + pb0[b];
                const T o[4] = {(T)acc[0], (T)acc[1], (T)acc[2], (T)acc[3]};
                if (TAIL && b == WB - 1 && b0 + b == NB - 1 && part5) {
#pragma unroll
                    for (int r = 0; r < 4; ++r)
                        if (P::of(g, r) >= 16 - a.tail) yp[P::of(g, r)] = o[r];
                } else {
                    P::store(b0 + b < nb ? yp : dummy, 0, g, o);
                }
            }
            if (PR) {
#pragma unroll
                for (int G = 0; G < NG; ++G)
                    if ((gb >> G) & 1) {
#pragma unroll
                        for (int r = 0; r < 4; ++r)
                            sum[G].p = Mfma<C>::run(AP ? pr[G][r] : cb[P::of(g, r) * RS + 16 * G + P::perm(li)], acc[r],
                                                    sum[G].p);
                    }
            }
        }
        if (PR) {
#pragma unroll
            for (int G = 0; G < NG; ++G) sum[G].plane();
        }
        slots(zl + 1);
    }
}

// What the sums over entries need to form again, from the block, a projection
// that is not finite.
template <typename T>
struct NlSupport {
    const T* y;
    long ldx;
    int nx, ny, nz;
    double hx, hy, hz, inv_rc2, N0, N1, rcut, rcut2;
    const NlCand* cand;
    uint32_t* odd;
    uint32_t epoch;
    const double* alpha;    // of the filter step that will apply the projections
};

// sum of chi_lm y over the points that a pair reaches, for a projection in which
// a value that is not finite took part; ends at the first NaN.
template <typename T>
__device__ double sum_support(const NlSupport<T>& a, const NlCand& c, const T* y, int lm) {
    const int z0 = max(0, (int)ceil((c.pz - a.rcut) / a.hz) - c.bz - 1);
    const int z1 = min(a.nz - 1, (int)floor((c.pz + a.rcut) / a.hz) - c.bz + 1);
    const int y0 = max(0, (int)ceil((c.py - a.rcut) / a.hy) - c.by - 1);
    const int y1 = min(a.ny - 1, (int)floor((c.py + a.rcut) / a.hy) - c.by + 1);
    const int x0 = max(0, (int)ceil((c.px - a.rcut) / a.hx) - c.bx - 1);
    const int x1 = min(a.nx - 1, (int)floor((c.px + a.rcut) / a.hx) - c.bx + 1);
    double s = 0.0;
    for (int z = z0; z <= z1; ++z)
        for (int j = y0; j <= y1; ++j)
            for (int i = x0; i <= x1; ++i) {
                const double dx = off_x(c, i, a.hx), dy = off_y(c, j, a.hy), dz = off_z(c, z, a.hz);
                const double r2 = add_sq(sum_sq(dx, dy), dz);
                if (r2 > a.rcut2) continue;
                const double f = lm == 0 ? a.N0 : a.N1 * (lm == 1 ? dx : (lm == 2 ? dy : dz));
                s += f * exp(-r2 * a.inv_rc2) * (double)y[i + (long)a.nx * (j + (long)a.ny * z)];
                if (s != s) return s;
            }
    return s;
}

// D(4a+lm, col) = alpha gamma_lm dV sum of atom a's entries (nw partial ones each,
// 1 or kNlSplit), in `parts` runs of them side by side, each in entry order, added
// in order.
template <typename T>
__global__ __launch_bounds__(256) void k_nl_reduce(const double* __restrict__ part, int ncol, int nw, int parts,
                                                   const int* __restrict__ off, const int* __restrict__ ent,
                                                   const int* __restrict__ cand_off, NlSupport<T> sup,
                                                   const double* __restrict__ g4, double dV, T* __restrict__ D,
                                                   long ldD) {
    __shared__ double sums[256];
    const int a = blockIdx.x, per = 256 / parts, run = threadIdx.x / per;
    const long q = (long)blockIdx.y * per + threadIdx.x % per;
    const bool on = q < 4L * ncol;
    const int col = (int)(q / 4), lm = (int)(q % 4);
    // eight loads in flight, added in order
    double s = 0.0;
    const int e0 = off[a], n = (off[a + 1] - e0) * nw, len = (n + parts - 1) / parts, k1 = min(n, (run + 1) * len);
    for (int k = run * len; k < k1 && on; k += 8) {
        double v[8];
#pragma unroll
        for (int u = 0; u < 8; ++u) {
            const int i = min(k + u, k1 - 1), e = nw == 1 ? i : i / kNlSplit;
            v[u] = part[((long)ent[e0 + e] * nw + (i - e * nw)) * ncol * 4 + q];
        }
#pragma unroll
        for (int u = 0; u < 8; ++u)
            if (k + u < k1) s += v[u];
    }
    if (parts > 1) {
        sums[threadIdx.x] = s;
        __syncthreads();
        if (run == 0)
            for (int r = 1; r < parts; ++r) s += sums[r * per + threadIdx.x];
    }
    if (run || !on) return;
    if (__builtin_expect(!__builtin_isfinite(s), 0)) {
        s = 0.0;
        for (int q = cand_off[a]; q < cand_off[a + 1]; ++q)
            s += sum_support(sup, sup.cand[q], sup.y + (long)col * sup.ldx, lm);
    }
    const T v = (T)(*sup.alpha * g4[4 * a + lm] * dV * s);
    if (__builtin_expect(!__builtin_isfinite(v), 0)) sup.odd[col / 16] = sup.epoch;
    D[(long)col * ldD + 4 * a + lm] = v;
}

// cos, sin of k . sL of every (atom, image) pair
__global__ void k_nl_phase(const NlCand* __restrict__ cand, int n, int nx, int ny, int nz, double kx, double ky,
                           double kz, double* __restrict__ phase) {
    const int q = blockIdx.x * blockDim.x + threadIdx.x;
    if (q >= n) return;
    sincos(kx * (cand[q].bx / nx) + ky * (cand[q].by / ny) + kz * (cand[q].bz / nz), &phase[2 * q + 1],
           &phase[2 * q]);
}

// Bloch form, per atom and complex column c: with the real projections p_s of
// the two halves on the atom's images s,
//   D_a = alpha gamma dV sum_s exp(i k.sL) (p_s[u] + i p_s[v])   (entries as above),
// and the coefficients exp(-i k.sL) D_a of every image, real part at the
// column of u, imaginary part at that of v.
template <typename T>
__global__ __launch_bounds__(256) void k_nl_reduce_k(const double* __restrict__ part, int ncol, int nw, int parts,
                                                     const int* __restrict__ off, const int* __restrict__ ent,
                                                     const int* __restrict__ ent_cand,
                                                     const int* __restrict__ cand_off, NlSupport<T> sup, long half,
                                                     const double* __restrict__ phase, const double* __restrict__ g4,
                                                     double dV, double* __restrict__ D, long ldD) {
    __shared__ double sums[2][256];
    const int a = blockIdx.x, per = 256 / parts, run = threadIdx.x / per;
    const long q = (long)blockIdx.y * per + threadIdx.x % per;
    const bool on = q < 4L * ncol;
    const int c = (int)(q / 4), lm = (int)(q % 4);
    double zr = 0.0, zi = 0.0;
    const int e0 = off[a], n = (off[a + 1] - e0) * nw, len = (n + parts - 1) / parts, k1 = min(n, (run + 1) * len);
    for (int k = run * len; k < k1 && on; k += 4) {
        double u[4], v[4], cs[4], sn[4];
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            const int i = min(k + r, k1 - 1), e = nw == 1 ? i : i / kNlSplit, en = ent[e0 + e];
            const double* p = part + (((long)en * nw + (i - e * nw)) * 2 * ncol + 2 * c) * 4 + lm;
            u[r] = p[0];
            v[r] = p[4];
            cs[r] = phase[2 * ent_cand[en]];
            sn[r] = phase[2 * ent_cand[en] + 1];
        }
#pragma unroll
        for (int r = 0; r < 4; ++r)
            if (k + r < k1) {
                zr += cs[r] * u[r] - sn[r] * v[r];
                zi += sn[r] * u[r] + cs[r] * v[r];
            }
    }
    if (parts > 1) {
        sums[0][threadIdx.x] = zr;
        sums[1][threadIdx.x] = zi;
        __syncthreads();
        if (run == 0)
            for (int r = 1; r < parts; ++r) {
                zr += sums[0][r * per + threadIdx.x];
                zi += sums[1][r * per + threadIdx.x];
            }
    }
    if (run || !on) return;
    if (__builtin_expect(!(__builtin_isfinite(zr) && __builtin_isfinite(zi)), 0)) {
        zr = zi = 0.0;
        const T* y = sup.y + (long)c * sup.ldx;
        for (int s = cand_off[a]; s < cand_off[a + 1]; ++s) {
            const double u = sum_support(sup, sup.cand[s], y, lm), v = sum_support(sup, sup.cand[s], y + half, lm);
            zr += phase[2 * s] * u - phase[2 * s + 1] * v;
            zi += phase[2 * s + 1] * u + phase[2 * s] * v;
        }
    }
    const double g = *sup.alpha * dV * g4[4 * a + lm];
    zr *= g;
    zi *= g;
    if (__builtin_expect(!(fabs(zr) < 1e300 && fabs(zi) < 1e300), 0)) sup.odd[c / 8] = sup.epoch;
    for (int s = cand_off[a]; s < cand_off[a + 1]; ++s) {
        const double cs = phase[2 * s], sn = phase[2 * s + 1];
        D[(2L * c) * ldD + 4 * s + lm] = zr * cs + zi * sn;
        D[(2L * c + 1) * ldD + 4 * s + lm] = zi * cs - zr * sn;
    }
}

template <typename V>
sparc_status put(sparc_gpu_ctx c, V** dst, const std::vector<V>& src) {
    SG_HIP(c, hipMalloc((void**)dst, std::max<size_t>(1, src.size()) * sizeof(V)));
    if (!src.empty()) SG_HIP(c, hipMemcpy(*dst, src.data(), src.size() * sizeof(V), hipMemcpyHostToDevice));
    return SPARC_OK;
}

template <typename T>
T* D_of(sparc_gpu_ctx c);
template <>
double* D_of<double>(sparc_gpu_ctx c) {
    return c->D;
}
template <>
float* D_of<float>(sparc_gpu_ctx c) {
    return c->D32;
}

}  // namespace

void free_nl_pass(NlPass& T) {
    for (void* p : {(void*)T.blk, (void*)T.cand, (void*)T.cand_off, (void*)T.odd, (void*)T.zero, T.dummy})
        if (p) hipFree(p);
    for (NlRanges& R : T.ranges)
        for (void* p : {(void*)R.units, (void*)R.occ, (void*)R.gm, (void*)R.ent_cand, (void*)R.red_off,
                        (void*)R.red_ent})
            if (p) hipFree(p);
    T = NlPass{};
}

namespace {

// Time of a pass over `tiles` column tiles of 16 in k z ranges, `split`: one tile
// per workgroup, whose waves share the blocks.  (Time of a plane) x (planes one
// after another) on a chip that holds 512 workgroups, two per compute unit (768
// that share blocks in FP32, whose tables take half the LDS); where half of a round
// is enough, each runs alone and takes 0.65 of the time (8.3 and 13 us a plane at
// 72^3).  A range costs about 3 planes more than its own (set-up, ends of pairs).
double nl_cost(int npen, int nz, int tiles, int k, bool split, bool fp32) {
    const long slots = split && fp32 ? 768 : 512, n = (long)npen * (split ? tiles : div_up(tiles, kNlWaves)) * k;
    const long last = n % slots;
    const double rounds = n / slots + (last == 0 ? 0.0 : (2 * last <= slots ? 0.65 : 1.0));
    return rounds * (div_up(nz, k) + 3) * (split ? kNlSplitPlane : 1.0);
}

// A pair's support in a pencil's plane: the blocks it meets
struct Hit {
    int pencil, cand, z;
    uint32_t mask;
};

// The hits of a pair in a pencil
struct PairHits {
    int cand;
    size_t h0, h1;
};

}  // namespace

// The units, slots and block masks for zs ranges of z.  hits: sorted by pencil,
// pair and plane; pairs, first: where each pencil's pairs begin.
static sparc_status build_ranges(sparc_gpu_ctx c, const std::vector<NlCand>& cands, const std::vector<Hit>& hits,
                                 const std::vector<PairHits>& pairs, const std::vector<size_t>& first,
                                 const std::vector<int>& nblk, int zs, NlRanges& R) {
    const int nz = c->nz, S = c->nlp.slots, NG = S / 4, zlen = (nz + zs - 1) / zs;
    zs = (nz + zlen - 1) / zlen;
    struct Span {
        int z0, z1, cand;
        size_t h0, h1;
    };
    // slots: each pair takes, for its span of planes in the unit, a free one of the
    // group that meets the fewest further blocks for it; pairs beyond the slots or
    // the local indices go to a further layer (a further pass), which supports this
    // dense do not reach in practice
    struct Placed {
        int slot, local;
        Span s;
    };
    struct Unit {
        NlUnit u;
        std::vector<Placed> p;
    };
    std::vector<std::vector<Unit>> layers;
    std::vector<Span> sp, rest;
    std::vector<uint32_t> met;
    int ncl = 1;
    for (int pencil = 0; pencil + 1 < (int)first.size(); ++pencil)
        for (int zr = 0; zr < zs; ++zr) {
            const int zb = zr * zlen, ze = std::min(nz, zb + zlen);
            auto before = [](const Hit& h, int z) { return h.z < z; };
            sp.clear();
            for (size_t q = first[pencil]; q < first[pencil + 1]; ++q) {
                const auto b = hits.begin() + pairs[q].h0, e = hits.begin() + pairs[q].h1;
                const auto lo = std::lower_bound(b, e, zb, before), hi = std::lower_bound(lo, e, ze, before);
                if (lo != hi)
                    sp.push_back({lo->z, (hi - 1)->z, pairs[q].cand, (size_t)(lo - hits.begin()), (size_t)(hi - hits.begin())});
            }
            std::sort(sp.begin(), sp.end(),
                      [](const Span& A, const Span& B) { return A.z0 != B.z0 ? A.z0 < B.z0 : A.cand < B.cand; });
            for (int layer = 0; !sp.empty(); ++layer) {
                std::vector<int> end(S, -1);   // last plane of each slot's pair
                met.assign((size_t)NG * zlen, 0);
                rest.clear();
                Unit un;
                un.u = NlUnit{zb, ze, pencil, nblk[pencil], 0, 0};
                for (const Span& s : sp) {
                    int slot = -1, fewest = 1 << 30;
                    for (int G = 0; G < NG; ++G) {
                        int q = 4 * G;
                        while (q < 4 * G + 4 && end[q] >= s.z0) ++q;
                        if (q == 4 * G + 4) continue;
                        int n = 0;   // blocks that group G would meet for this pair alone
                        for (size_t h = s.h0; h < s.h1; ++h)
                            n += __builtin_popcount(hits[h].mask & ~met[(size_t)G * zlen + hits[h].z - zb]);
                        if (n < fewest) {
                            fewest = n;
                            slot = q;
                        }
                    }
                    if (slot < 0 || un.p.size() >= (size_t)kMaxLocal) {
                        rest.push_back(s);
                        continue;
                    }
                    end[slot] = s.z1;
                    for (size_t h = s.h0; h < s.h1; ++h) met[(size_t)(slot / 4) * zlen + hits[h].z - zb] |= hits[h].mask;
                    un.p.push_back({slot, (int)un.p.size(), s});
                }
                un.u.ncl = (int)un.p.size();
                ncl = std::max(ncl, un.u.ncl);
                if ((int)layers.size() <= layer) layers.emplace_back();
                layers[layer].push_back(std::move(un));
                sp.swap(rest);
            }
        }
    std::vector<NlUnit> units;
    std::vector<uint8_t> occ;
    std::vector<uint64_t> gm;
    std::vector<int> ent_cand;
    std::vector<std::vector<int>> per_atom(c->n_atoms);
    R.layer_off.assign(1, 0);
    for (auto& ly : layers) {
        // units of one z range and neighbouring pencils side by side
        std::stable_sort(ly.begin(), ly.end(), [](const Unit& A, const Unit& B) { return A.u.zb < B.u.zb; });
        for (Unit& un : ly) {
            un.u.ebase = (int)ent_cand.size();
            const size_t o0 = occ.size(), g0 = gm.size();
            occ.insert(occ.end(), (size_t)zlen * S, (uint8_t)kIdle);
            gm.insert(gm.end(), zlen, 0);
            for (const Placed& p : un.p) {
                per_atom[cands[p.s.cand].atom].push_back((int)ent_cand.size());
                ent_cand.push_back(p.s.cand);
                for (int z = p.s.z0; z <= p.s.z1; ++z) occ[o0 + (size_t)(z - un.u.zb) * S + p.slot] = (uint8_t)p.local;
                for (size_t h = p.s.h0; h < p.s.h1; ++h) {
                    uint64_t& w = gm[g0 + hits[h].z - un.u.zb];
                    for (int b = 0; b < kNlBlocks; ++b)
                        if ((hits[h].mask >> b) & 1) w |= 1ull << (b * NG + p.slot / 4);
                }
            }
            units.push_back(un.u);
        }
        R.layer_off.push_back((int)units.size());
    }
    std::vector<int> roff(c->n_atoms + 1, 0), rent;
    for (int a = 0; a < c->n_atoms; ++a) {
        rent.insert(rent.end(), per_atom[a].begin(), per_atom[a].end());
        roff[a + 1] = (int)rent.size();
    }
    R.zlen = zlen;
    R.ncl = ncl;
    R.whole = R.layer_off.size() == 2 && (int)units.size() == c->nlp.npen * zs;
    R.n_entries = (long)ent_cand.size();
    sparc_status st;
    if ((st = put(c, &R.units, units)) != SPARC_OK) return st;
    if ((st = put(c, &R.occ, occ)) != SPARC_OK) return st;
    if ((st = put(c, &R.gm, gm)) != SPARC_OK) return st;
    if ((st = put(c, &R.ent_cand, ent_cand)) != SPARC_OK) return st;
    if ((st = put(c, &R.red_off, roff)) != SPARC_OK) return st;
    return put(c, &R.red_ent, rent);
}

// Runs of entries that k_nl_reduce sums side by side: as many as the threads of a
// workgroup allow for ncol columns.
static int reduce_runs(int ncol) {
    int parts = 1;
    while (parts < 16 && 8 * parts * ncol <= 256) parts *= 2;
    return parts;
}

// Ranges and waves of a pass over ncol columns: the cheapest by nl_cost of the
// ranges that were built; other than those of the full block only where their
// partial sums fit the fixed scratch array, so that the allocation-free filter
// takes the same.  H X in FP64 with the full block's ranges and whole waves for
// every width, and now: 72^3 x 1 238 and 81 us, x 12 261 and 107, x 24 279 and 173;
// 120^3 x 1 1072 and 275.
struct NlShape {
    const NlRanges* R;
    int nw;   // partial entries of a unit and pair (waves that share the blocks)
};
static NlShape nl_shape(sparc_gpu_ctx c, int ncol, bool fp32) {
    const NlPass& N = c->nlp;
    NlShape best{&N.ranges[0], 1};
    double least = 0;
    for (const NlRanges& R : N.ranges)
        for (int nw : {1, kNlSplit}) {
            const bool full = &R == &N.ranges[0] && nw == 1;
            if (!full && (size_t)R.n_entries * nw * 4 * ncol > c->scratch_elems) continue;
            // the sum over an atom's entries takes 0.023 planes per entry and run
            const double cost = nl_cost(N.npen, c->nz, div_up(ncol, 16), div_up(c->nz, R.zlen), nw > 1, fp32) +
                                0.023 * R.n_entries * nw / c->n_atoms / reduce_runs(ncol);
            if (full || cost < least) {
                least = cost;
                best = NlShape{&R, nw};
            }
        }
    return best;
}

static size_t part_doubles(const NlShape& sh, int ncol) { return (size_t)sh.R->n_entries * sh.nw * 4 * ncol; }

// Partial sums of any block of up to n columns, n = 0 .. 2 n_states (halves of Bloch
// columns): with each width's own shape a narrower block can take more than a wider
// one, but a call must not allocate after one at least as wide (it may be captured,
// or a graph may hold the memory).  Within a tile, runs and the shapes allowed they
// grow with the width, so only where one of these changes is looked at.
static void plan_partials(sparc_gpu_ctx c) {
    NlPass& N = c->nlp;
    const int most = 2 * c->n_states;
    std::vector<int> at{1, 2, 4, 8};
    for (int n = 16; n < most; n += 16) at.push_back(n);
    for (const NlRanges& R : N.ranges)
        for (int nw : {1, kNlSplit})
            at.push_back((int)std::min<size_t>(most, c->scratch_elems / std::max(1L, 4 * nw * R.n_entries)));
    at.push_back(most);
    N.part_upto.assign(most + 1, 0);
    for (int n : at)
        if (n > 0 && n <= most)
            for (bool fp32 : {false, true})
                N.part_upto[n] = std::max(N.part_upto[n], part_doubles(nl_shape(c, n, fp32), n));
    for (int n = 1; n <= most; ++n) N.part_upto[n] = std::max(N.part_upto[n], N.part_upto[n - 1]);
}

// The pencils of the pass and its tables.  segs: every (atom, image)
// pair's support as line segments of the wrapped grid.
sparc_status build_nl_pass(sparc_gpu_ctx c, const std::vector<NlCand>& cands, const std::vector<NlSeg>& segs) {
    const int nx = c->nx, ny = c->ny, nz = c->nz, nxy = nx * ny;
    const int nb = (nxy + 15) / 16;
    NlPass& T = c->nlp;
    // Pencils: blocks cut into lists of kNlBlocks.  Either cells of rows x
    // x-range, a block belonging to the cell of its first point, or runs of R
    // consecutive blocks, one per row, a row taken as m whole runs (every pencil
    // but the last is full, but drifts in x where m runs are not n_x points).
    std::vector<std::vector<int>> lists, trial;
    auto cells = [&](int npx, int by) {
        trial.assign((size_t)npx * ((ny + by - 1) / by), {});
        for (int b = 0; b < nb; ++b) {
            const int x = (16 * b) % nx, y = (16 * b) / nx;
            trial[(y / by) * npx + std::min(npx - 1, (int)((long)x * npx / nx))].push_back(b);
        }
    };
    auto runs = [&](int R) {
        const int G = kNlBlocks / R, m = std::max(1, (2 * nx / (16 * R) + 1) / 2);
        trial.assign((size_t)(nb / (R * G * m) + 1) * m, {});
        for (int b = 0; b < nb; ++b) trial[b / R / (m * G) * m + b / R % m].push_back(b);
    };
    // Time of a plane of an average pencil: a block place costs one, more where
    // planes are no whole 128-byte lines and each run of blocks shares one with
    // its neighbours (97 x 98 x 81 x 504 FP64, H X without its sweep: 3420 us
    // with 5.6-block cells of single blocks, 3100 with full pencils of them, 2810
    // in runs of 2, 2840 in runs of 3); a slot in use costs 0.4 (96 x 98 x 81 x
    // 504: 2250 us with up to 9, 2421 with up to 12); past 16 slots one workgroup
    // instead of two fits a compute unit (72^3 x 260: 765 and 1250 us).
    auto plane_time = [&](int* npen) {
        double sum = 0;
        *npen = 0;
        for (const auto& l : trial) {
            if (l.empty()) continue;
            const size_t parts = (l.size() + kNlBlocks - 1) / kNlBlocks, per = (l.size() + parts - 1) / parts;
            for (size_t i = 0; i < l.size(); i += per, ++*npen) {
                const size_t e = std::min(l.size(), i + per);
                const int x0 = (16 * l[i]) % nx, y0 = (16 * l[i]) / nx;
                int lo = 0, hi = 16, y1 = y0, nrun = 0;
                for (size_t j = i; j < e; ++j) {
                    const int x = (16 * l[j]) % nx, d = (x - x0 + nx + nx / 2) % nx - nx / 2;
                    lo = std::min(lo, d);
                    hi = std::max(hi, d + 16);
                    y1 = std::min(ny - 1, (16 * l[j] + 15) / nx);
                    nrun += j == i || l[j] != l[j - 1] + 1;
                }
                const double wx = std::min(c->Lx, (hi - lo) * c->hx), wy = (y1 - y0 + 1) * c->hy, r = c->rcut_nl;
                const double area = std::min(c->Lx * c->Ly, wx * wy + 2 * r * (wx + wy) + 3.14159265358979 * r * r);
                const double slots = c->n_atoms * area / (c->Lx * c->Ly) * std::min(1.0, 2 * r / c->Lz);
                sum += (kNlBlocks + (nxy % 16 ? 0.45 * nrun : 0.0) + 0.4 * slots) * (slots > 12 ? 1.5 : 1.0);
            }
        }
        return sum / *npen;
    };
    // pencils and z ranges for the context's full block
    const int tiles = div_up(c->n_states, 16), least_zs = (nz + kMaxPlanes - 1) / kMaxPlanes;
    int zs = 0;
    double best = 0;
    auto consider = [&]() {
        int npen;
        const double plane = plane_time(&npen);
        for (int k = least_zs; k <= std::max(1, nz / 4); ++k) {
            const double cost = plane * nl_cost(npen, nz, tiles, k, false, false);
            if (zs == 0 || cost < best) {
                best = cost;
                zs = k;
                lists = trial;
            }
        }
    };
    for (int by = 1; by <= std::min(6, ny); ++by)
        for (int npx = 1; npx <= (nx + 15) / 16; ++npx) {
            cells(npx, by);
            consider();
        }
    for (int R = 1; R <= 3; ++R) {
        runs(R);
        consider();
    }
    std::vector<int> blk, nblk, pen(nb), place(nb);
    int npen = 0;
    for (auto& l : lists) {
        const int n = (int)l.size();
        if (!n) continue;
        const int parts = (n + kNlBlocks - 1) / kNlBlocks, per = (n + parts - 1) / parts;
        for (int i = 0; i < n; i += per, ++npen) {
            blk.insert(blk.end(), kNlBlocks, -1);
            nblk.push_back(std::min(per, n - i));
            for (int j = i; j < std::min(n, i + per); ++j) {
                // an incomplete last block starts 16 points before the end of
                // the plane and takes the last place
                const bool tail = nxy % 16 != 0 && l[j] == nb - 1;
                const int at = tail ? kNlBlocks - 1 : j - i;
                blk[(size_t)npen * kNlBlocks + at] = tail ? nxy - 16 : 16 * l[j];
                pen[l[j]] = npen;
                place[l[j]] = at;
            }
        }
    }
    // (pencil, pair, plane) -> blocks met
    std::vector<Hit> hits;
    hits.reserve(2 * segs.size());
    for (const NlSeg& s : segs) {
        const int p0 = s.x0 + nx * s.y, p1 = p0 + s.n - 1;
        for (int b = p0 / 16; b <= p1 / 16; ++b) {
            if (!hits.empty() && hits.back().pencil == pen[b] && hits.back().cand == s.cand && hits.back().z == s.z)
                hits.back().mask |= 1u << place[b];
            else
                hits.push_back({pen[b], s.cand, s.z, 1u << place[b]});
        }
    }
    std::sort(hits.begin(), hits.end(), [](const Hit& A, const Hit& B) {
        if (A.pencil != B.pencil) return A.pencil < B.pencil;
        if (A.cand != B.cand) return A.cand < B.cand;
        return A.z < B.z;
    });
    // per pencil the pairs' hits, and the most pairs at one plane
    std::vector<PairHits> pairs;
    std::vector<size_t> first(npen + 1, 0);
    int most = 1;
    {
        std::vector<int> live;
        for (size_t h = 0; h < hits.size();) {
            size_t k = h;
            while (k < hits.size() && hits[k].pencil == hits[h].pencil && hits[k].cand == hits[h].cand) ++k;
            if (h == 0 || hits[h].pencil != hits[h - 1].pencil) live.assign(nz, 0);
            for (int z = hits[h].z; z <= hits[k - 1].z; ++z) most = std::max(most, ++live[z]);
            pairs.push_back({hits[h].cand, h, k});
            first[hits[h].pencil + 1] = pairs.size();
            h = k;
        }
        for (int q = 0; q < npen; ++q) first[q + 1] = std::max(first[q + 1], first[q]);
    }
    T.npen = npen;
    T.slots = most <= 8 ? 8 : (most <= 16 ? 16 : kMaxSlots);
    std::vector<int> coff(c->n_atoms + 1, 0);
    for (const NlCand& q : cands) coff[q.atom + 1]++;
    for (int a = 0; a < c->n_atoms; ++a) coff[a + 1] += coff[a];
    T.n_cand = (int)cands.size();
    sparc_status st;
    SG_HIP(c, hipMalloc(&T.dummy, 256 * sizeof(double)));
    // one per column of a block at most (column groups of less than 16), two
    // blocks' worth of halves in tiles of 16 for Bloch columns
    if ((st = put(c, &T.odd, std::vector<uint32_t>(c->n_states + 1, 0))) != SPARC_OK) return st;
    if ((st = put(c, &T.zero, std::vector<double>(5, 0.0))) != SPARC_OK) return st;
    if ((st = put(c, &T.blk, blk)) != SPARC_OK) return st;
    if ((st = put(c, &T.cand, cands)) != SPARC_OK) return st;
    if ((st = put(c, &T.cand_off, coff)) != SPARC_OK) return st;
    // the ranges of the full block, then those that suit 1, 2, 4, ... column tiles
    std::vector<int> cuts{zs};
    for (int t = 1; t < tiles; t *= 2)
        for (bool fp32 : {false, true}) {
            int best_k = zs;
            double least = 0;
            for (int k = least_zs; k <= std::max(1, nz / 4); ++k) {
                const double cost = std::min(nl_cost(npen, nz, t, k, false, fp32), nl_cost(npen, nz, t, k, true, fp32));
                if (k == least_zs || cost < least) {
                    least = cost;
                    best_k = k;
                }
            }
            if (std::find(cuts.begin(), cuts.end(), best_k) == cuts.end()) cuts.push_back(best_k);
        }
    for (int k : cuts) {
        T.ranges.emplace_back();
        if ((st = build_ranges(c, cands, hits, pairs, first, nblk, k, T.ranges.back())) != SPARC_OK) return st;
        const NlRanges& R = T.ranges.back();
        if (c->debug)
            fprintf(stderr,
                    "[sparc_gpu] nonlocal pass: %d pencils, %d units of %d planes, %d slots (%d used), %zu layers, %ld "
                    "entries, at most %d pairs per unit\n",
                    npen, R.layer_off.back(), R.zlen, T.slots, most, R.layer_off.size() - 1, R.n_entries, R.ncl);
    }
    plan_partials(c);
    return SPARC_OK;
}

template <typename T, typename C, int S>
static sparc_status launch_pass(sparc_gpu_ctx c, const NlArgs<T, C>& a, int nw, NlApply ap, bool pr, size_t shmem) {
    constexpr int NB = kNlBlocks, WB = kNlBlocks / kNlSplit;
    const long nblocks = 8L * div_up(a.nunit, 8) * a.nchunk;
    if (nblocks > 0x7fffffffL) return set_err(c, SPARC_ERR_ARG, "nonlocal pass: too many blocks");
    const dim3 g((unsigned)nblocks), b(64 * kNlWaves);
    auto go = [&](auto wb, auto av, auto pv, auto tv) {
        k_nl_pass<T, C, S, wb(), av(), pv(), tv()><<<g, b, shmem, c->stream>>>(a);
    };
    auto go_form = [&](auto wb, auto tv) {
        constexpr std::integral_constant<int, 1> add;
        constexpr std::integral_constant<int, 2> write;
        if (ap == NlApply::write) go(wb, write, std::false_type(), tv);
        else if (pr) go(wb, add, std::true_type(), tv);
        else go(wb, add, std::false_type(), tv);
    };
    constexpr std::integral_constant<int, NB> whole;
    constexpr std::integral_constant<int, WB> shared;
    constexpr std::integral_constant<int, 0> none;
    if (ap == NlApply::no && nw > 1) go(shared, none, std::true_type(), std::false_type());
    else if (ap == NlApply::no) go(whole, none, std::true_type(), std::false_type());
    else if (nw > 1) go_form(shared, std::true_type());
    else if (a.tail) go_form(whole, std::true_type());
    else go_form(whole, std::false_type());
    SG_CHECK_LAUNCH(c);
    return SPARC_OK;
}

// The context's memory for the partial sums of ncol real columns (halves), and of
// fewer (see plan_partials)
static sparc_status partials(sparc_gpu_ctx c, const NlShape& sh, int ncol, double** part) {
    const std::vector<size_t>& upto = c->nlp.part_upto;
    const size_t need = std::max(part_doubles(sh, ncol), upto[std::min<size_t>(ncol, upto.size() - 1)]);
    if (c->nl_part_elems < need) {
        if (c->nl_part) {
            SG_HIP(c, hipStreamSynchronize(c->stream));
            SG_HIP(c, hipFree(c->nl_part));
            c->nl_part = nullptr;
            c->nl_part_elems = 0;
        }
        SG_HIP(c, hipMalloc((void**)&c->nl_part, need * sizeof(double)));
        c->nl_part_elems = need;
    }
    *part = c->nl_part;
    return SPARC_OK;
}

template <typename T, typename C>
static NlArgs<T, C> pass_args(sparc_gpu_ctx c, const NlRanges& R, long ldx, int mode, int step) {
    const NlPass& N = c->nlp;
    NlArgs<T, C> a;
    a.y = nullptr;
    a.ldx = ldx;
    a.halves = 0;
    a.half = c->nd;
    a.by_pair = 0;
    a.nx = c->nx;
    a.ny = c->ny;
    a.nz = c->nz;
    a.nxy = c->nx * c->ny;
    a.ncol = 0;
    a.zlen = R.zlen;
    a.ncl = R.ncl;
    a.blk = N.blk;
    a.tail = a.nxy % 16;
    a.dummy = reinterpret_cast<T*>(N.dummy);
    a.ent_cand = R.ent_cand;
    a.cand = N.cand;
    a.hx = c->hx;
    a.hy = c->hy;
    a.hz = c->hz;
    a.inv_rc2 = 1.0 / (c->rc_nl * c->rc_nl);
    a.N0 = std::pow(2.0 / (3.14159265358979323846 * c->rc_nl * c->rc_nl), 0.75);
    a.N1 = (2.0 / c->rc_nl) * a.N0;
    a.rcut2 = c->rcut_nl * c->rcut_nl;
    a.D = nullptr;
    a.ldD = 0;
    a.odd = N.odd;
    a.epoch = N.epoch;
    a.part = nullptr;
    a.zero = reinterpret_cast<const C*>(N.zero);
    a.alpha = N.zero + 4;
    a.params = c->scal + S_A;
    a.mode = mode;
    a.step = step;
    return a;
}

template <typename T, typename C>
static NlSupport<T> support(sparc_gpu_ctx c, const NlArgs<T, C>& a) {
    return NlSupport<T>{a.y,  a.ldx,      a.nx,    a.ny,   a.nz,  a.hx,        a.hy,          a.hz, a.inv_rc2, a.N0,
                        a.N1, c->rcut_nl, a.rcut2, a.cand, a.odd, a.epoch + 1, a.alpha};
}

// The pass over the columns set in a; with further layers every apply comes
// before the first projection.
template <typename T, typename C>
static sparc_status run_layers(sparc_gpu_ctx c, NlArgs<T, C> a, NlShape sh, NlApply ap, bool pr) {
    const NlRanges& R = *sh.R;
    const int S = c->nlp.slots;
    const size_t shmem = nl_lds_layout(sizeof(C), S, R.zlen, R.ncl).total;
    if (shmem > 160 * 1024) return set_err(c, SPARC_ERR_ARG, "nonlocal pass needs more than 160 KB of LDS");
    const int tiles = div_up(a.ncol, 16);
    a.nchunk = sh.nw > 1 ? tiles : div_up(tiles, kNlWaves);
    a.nwc = div_up(tiles, a.nchunk);
    const int nl = (int)R.layer_off.size() - 1;
    for (int half = 0; half < (nl > 1 ? 2 : 1); ++half) {
        const NlApply ap1 = half == 0 ? ap : NlApply::no;
        const bool pr1 = pr && (nl == 1 || half == 1);
        if (ap1 == NlApply::no && !pr1) continue;
        for (int l = 0; l < nl; ++l) {
            const long u0 = R.layer_off[l];
            a.nunit = R.layer_off[l + 1] - (int)u0;
            a.units = R.units + u0;
            a.occ = R.occ + u0 * R.zlen * S;
            a.gm = R.gm + u0 * R.zlen;
            sparc_status st = S == 8    ? launch_pass<T, C, 8>(c, a, sh.nw, ap1, pr1, shmem)
                              : S == 16 ? launch_pass<T, C, 16>(c, a, sh.nw, ap1, pr1, shmem)
                                        : launch_pass<T, C, kMaxSlots>(c, a, sh.nw, ap1, pr1, shmem);
            if (st != SPARC_OK) return st;
        }
    }
    return SPARC_OK;
}

// Writing pays where reading y would bound the pass: all four waves of its
// workgroups have columns (three where planes share 128-byte lines), and Bloch
// columns in FP32, whose products take twice their reading, are more than the
// last-level cache holds along.  H X with the pass last and first, us: 72^3 x 64
// FP64 278, 250; 120^3 x 32 728, 789; 120^3 x 130 2543, 2690; 51 x 68 x 93 x 77
// 357, 338; Bloch FP32 71 x 61 x 45 x 30 154, 176 and 72^3 x 260 1831, 1707.
bool nl_writes(sparc_gpu_ctx c, int ncol, bool fp32, bool bloch) {
    const NlPass& N = c->nlp;
    if (N.ranges.empty() || N.ranges[0].n_entries == 0) return false;
    const NlShape sh = nl_shape(c, ncol, fp32 && !bloch);
    if (!sh.R->whole || sh.nw > 1) return false;
    const int tiles = div_up(ncol, 16), waves = div_up(tiles, div_up(tiles, kNlWaves));
    if (bloch) return waves == 4 && (!fp32 || (double)c->nd * ncol * sizeof(float) > 128e6);
    return waves == 4 || (waves == 3 && (long)c->nx * c->ny % 16 != 0);
}

// One pass over a block: apply (y += chi D, or y = chi D) and / or project
// (D = alpha gamma dV chi^T y, alpha that of filter step `step` of mode `mode`,
// which will apply it).
template <typename T>
sparc_status nl_pass(sparc_gpu_ctx c, T* y, int ncol, long ldx, NlApply ap, bool pr, int mode, int step, double* part,
                     size_t part_elems) {
    const NlPass& N = c->nlp;
    if (N.ranges.empty() || N.ranges[0].n_entries == 0 || ncol == 0) return SPARC_OK;
    sparc_status st;
    const NlShape sh = nl_shape(c, ncol, sizeof(T) == 4);
    const NlRanges& R = *sh.R;
    const int runs = reduce_runs(ncol);
    const size_t per_col = part_doubles(sh, 1);
    int group = ncol;
    if (pr && part) {
        // caller memory: as many columns at a time as it holds, whole
        // 16-column tiles where it can
        if (per_col > part_elems)
            return set_err(c, SPARC_ERR_ARG, "projection partials of one column exceed the fixed scratch array");
        group = (int)std::min<size_t>((size_t)ncol, part_elems / per_col);
        if (group >= 16 && group < ncol) group -= group % 16;
    } else if (pr) {
        if ((st = partials(c, sh, ncol, &part)) != SPARC_OK) return st;
    }
    NlArgs<T, T> a = pass_args<T, T>(c, R, ldx, mode, step);
    a.ldD = 4L * c->n_atoms;
    a.part = part;
    const int slot = prof_begin(c, PK_PROJ);
    for (int c0 = 0; c0 < ncol; c0 += group) {
        a.ncol = std::min(group, ncol - c0);
        a.y = y + (long)c0 * ldx;
        a.odd = N.odd + (group < 16 ? c0 : c0 / 16);
        T* D = D_of<T>(c) + (long)c0 * a.ldD;
        a.D = D;
        if ((st = run_layers<T, T>(c, a, sh, ap, pr)) != SPARC_OK) return st;
        if (pr) {
            k_nl_reduce<T><<<dim3(c->n_atoms, div_up(4L * a.ncol, 256 / runs)), 256, 0, c->stream>>>(
                part, a.ncol, sh.nw, runs, R.red_off, R.red_ent, N.cand_off, support(c, a), c->nl.gamma4,
                c->dV, D, a.ldD);
            SG_CHECK_LAUNCH(c);
        }
    }
    if (pr) ++c->nlp.epoch;
    prof_end(c, slot);
    return SPARC_OK;
}

template sparc_status nl_pass<double>(sparc_gpu_ctx, double*, int, long, NlApply, bool, int, int, double*, size_t);
template sparc_status nl_pass<float>(sparc_gpu_ctx, float*, int, long, NlApply, bool, int, int, double*, size_t);

// The pass over Bloch columns: the halves u, v are real columns, the images'
// phases enter in the sum over an atom's entries.
template <typename T>
sparc_status nl_pass_k(sparc_gpu_ctx c, T* y, int ncol, long ldx, NlApply ap, bool pr, int mode, int step) {
    const NlPass& N = c->nlp;
    if (N.ranges.empty() || N.ranges[0].n_entries == 0 || ncol == 0) return SPARC_OK;
    sparc_status st;
    const NlShape sh = nl_shape(c, 2 * ncol, false);
    const NlRanges& R = *sh.R;
    const int runs = reduce_runs(ncol);
    double* part = nullptr;
    if (pr && (st = partials(c, sh, 2 * ncol, &part)) != SPARC_OK) return st;
    const long ldD = 4L * N.n_cand;
    if (c->kp_D_elems < (size_t)ldD * 2 * ncol) {
        if (c->kp_D) {
            SG_HIP(c, hipStreamSynchronize(c->stream));
            SG_HIP(c, hipFree(c->kp_D));
            c->kp_D = nullptr;
            c->kp_D_elems = 0;
        }
        SG_HIP(c, hipMalloc((void**)&c->kp_D, (size_t)ldD * 2 * ncol * sizeof(double)));
        c->kp_D_elems = (size_t)ldD * 2 * ncol;
    }
    if (!c->kp_phase) SG_HIP(c, hipMalloc((void**)&c->kp_phase, 2 * (size_t)N.n_cand * sizeof(double)));
    const int slot = prof_begin(c, PK_BLOCH_PROJ);
    const double* k = c->kvec;
    if (!c->kp_phase_valid || c->kp_phase_k[0] != k[0] || c->kp_phase_k[1] != k[1] || c->kp_phase_k[2] != k[2]) {
        k_nl_phase<<<div_up(N.n_cand, 256), 256, 0, c->stream>>>(N.cand, N.n_cand, c->nx, c->ny, c->nz, k[0] * c->Lx,
                                                                 k[1] * c->Ly, k[2] * c->Lz, c->kp_phase);
        SG_CHECK_LAUNCH(c);
        for (int d = 0; d < 3; ++d) c->kp_phase_k[d] = k[d];
        c->kp_phase_valid = 1;
    }
    NlArgs<T, double> a = pass_args<T, double>(c, R, ldx, mode, step);
    a.halves = 1;
    a.by_pair = 1;
    a.ldD = ldD;
    a.part = part;
    a.ncol = 2 * ncol;
    a.y = y;
    a.D = c->kp_D;
    if ((st = run_layers<T, double>(c, a, sh, ap, pr)) != SPARC_OK) return st;
    if (pr) {
        k_nl_reduce_k<T><<<dim3(c->n_atoms, div_up(4L * ncol, 256 / runs)), 256, 0, c->stream>>>(
            part, ncol, sh.nw, runs, R.red_off, R.red_ent, R.ent_cand, N.cand_off, support(c, a), a.half,
            c->kp_phase, c->nl.gamma4, c->dV, c->kp_D, ldD);
        SG_CHECK_LAUNCH(c);
        ++c->nlp.epoch;
    }
    prof_end(c, slot);
    return SPARC_OK;
}

template sparc_status nl_pass_k<double>(sparc_gpu_ctx, double*, int, long, NlApply, bool, int, int);
template sparc_status nl_pass_k<float>(sparc_gpu_ctx, float*, int, long, NlApply, bool, int, int);

}  // namespace sg
