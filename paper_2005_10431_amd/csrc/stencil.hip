// Matrix-free Hamiltonian and the Chebyshev recurrence built on it.
//
// H x = -1/2 Delta_h x + V_eff x + sum_I sum_lm gamma_Il chi_Ilm (dV chi_Ilm^T x)
// (Sec. 2 eq. (1); matrix-free stencil and outer-product nonlocal term as in
// Sec. 2.1).  The scaled three-term Chebyshev recurrence of the CheFSI filter
// (Sec. 2.1) is fused into the epilogue of the stencil sweep, so one sweep
// streams X_k (stencil operand), X_{k-1} (recurrence term) and writes X_{k+1}
// over X_{k-1}: 3 block-sized streams per filter degree.  With projectors the
// nonlocal pass (nonlocal.hip) then completes X_{k+1} and forms its
// projections for the next degree.
//
// Sweep kernel layout (one workgroup = one orbital x one y-slab x a range of z):
//  - a thread holds VX consecutive x points (16 bytes where they divide n_x), so that loads, stores
//    and the x and y reads from LDS move whole vectors and the address work is
//    shared by VX points;
//  - the slab is `ty` full x-rows; periodic x wraps inside LDS (padded rows),
//    so only y needs halo rows, read from L2 where a neighbouring slab of the
//    same orbital (mapped to the same XCD, see the block mapping below)
//    loaded them recently enough, else from the last-level cache or HBM;
//  - z is marched with a register ring of RING = 13 + PR planes per thread:
//    planes z-6 .. z+6 in use and PR planes in flight, so every point of X_k
//    is fetched once per sweep (plus the 12 planes around the range);
//  - the halo rows, X_{k-1} and V_eff of the coming planes sit in PQ-deep
//    register queues, so each load has PQ plane steps to land;
//  - two LDS plane buffers alternate so one barrier per plane suffices;
//  - a workgroup takes all of z, except those of a compute unit's last,
//    incomplete round (or of a block too small to fill the chip), which are
//    cut into equal z ranges (see sweep_rounds).
#include <cmath>
#include <map>
#include <mutex>
#include <cstdlib>
#include <utility>

#include "internal.hpp"

namespace sg {

template <typename T>
struct SweepArgs {
    const T* x;       // X_k, operand of H
    T* out;           // output block (may alias xprev, never x)
    const T* xprev;   // X_{k-1} or null
    long ldx;
    int halves;       // 0: column j at j ldx; 1: at (j / 2) ldx + (j % 2) half (Bloch columns)
    long half;
    double ph[6];     // Bloch sweeps: cos, sin of k_d L_d per axis
    int nx, ny, nz;
    int ty, ntiles_y;
    int grp;          // orbitals whose copies of a slab are dispatched side by side
    // -1/2 Delta_h: c*[q] multiplies the pair at distance q, c0 the point itself
    double c0;
    T cx[kMaxHalfOrder + 1], cy[kMaxHalfOrder + 1], cz[kMaxHalfOrder + 1];
    const T* veff;
    const double* params;  // a, b, a0 on the device
    int step;
    int ncol;
    int round, split;      // workgroups an XCD holds at once; z ranges of those past its last full round
};

constexpr int kRing = 16;            // z-ring slots: planes z-6 .. z+6 and 3 in flight
constexpr int kRingAhead = kRing - 2 * kMaxHalfOrder - 1;
constexpr int kQueue = 2;            // depth of the halo / X_{k-1} / V_eff queues
static_assert(kRing % kQueue == 0, "the unrolled step count must cycle every queue");

// Points per thread: the widest of 16, 8 and 4 bytes (FP64 16, 8) that divides
// n_x, so that a row is whole vectors, each at an aligned place in LDS.  (With
// the last vector of a row moved back instead, LDS takes unaligned accesses:
// 62 x 29 x 45 x 116 in FP32 50.7 instead of 28.7 us, 51 x 68 x 93 x 77 in FP64
// 176 instead of 123 us.)
template <typename T>
static int sweep_vx(int nx) {
    const int vx = 16 / (int)sizeof(T);
    return nx % vx == 0 ? vx : (vx == 4 && nx % 2 == 0 ? 2 : 1);
}

// columns left and right of a row in LDS, and values of a row
__host__ __device__ constexpr int sweep_pad(int vx) { return vx == 1 ? kMaxHalfOrder : 8; }
__host__ __device__ constexpr int sweep_row(int nx, int vx) { return nx + 2 * sweep_pad(vx); }

// Waves per SIMD, and with them the threads of a workgroup at most: three at 168
// VGPRs with 16 bytes per thread (FP32 with two points per thread and four waves
// per SIMD took 275 instead of 254 us at 72^3 x 260), four with less; two for the
// Bloch sweep, which keeps the other half's values too.
__host__ __device__ constexpr int sweep_simd_waves(size_t bytes, bool bloch) {
    return bloch ? 2 : (bytes == 16 ? 3 : 4);
}
// Odd rows of more than 128 points (at most 256) leave the 512 threads of a Bloch
// workgroup slabs of 2 or 3 rows, with up to 6 halo values per thread.
constexpr int kSweepMaxHalo = 6;

template <typename T, int N, int A>
struct VecOf {
    typedef T type __attribute__((ext_vector_type(N), aligned(A)));
};

// f(phase 0, z0), f(phase 1, z0 + 1), ... below ze
template <typename F, int... U>
__device__ __forceinline__ void each_phase(F& f, int z0, int ze, std::integer_sequence<int, U...>) {
    (void)((z0 + U < ze && (f(U, z0 + U), true)) && ...);
}

// The sweep.  MODE: 0 out = H_loc x; 1 first filter step; 2 filter step `step`
// (>= 2) with xprev = X_{k-1} (may alias out).  VX: points per thread, a
// divisor of n_x.  HM: halo vectors per thread and plane.  Where PQ planes of them
// would spill (PH) they are loaded one plane ahead (256 x 40 x 40 x 100 in FP64, a
// filter step: 489 us with two planes, now 383; 200 x 64 x 64 x 120: 883 and 687).
//
// One z-plane step at ring phase U (z = z0 + U).  On entry the LDS buffer of
// parity U holds plane z (own rows with x-wrap padding and halo rows), written
// during the previous step.
//  1. barrier, then the loads of the halo rows of plane z + PQ and of ring
//     plane z + 6 + PR (plane indices wrap, so the loads are unconditional);
//  2. stencil + potential + recurrence for plane z, store;
//  3. load X_{k-1} and V_eff of plane z + PQ into the queue slot plane z has
//     freed;
//  4. plane z + 1 into the other LDS buffer.
// Threads without a point of the slab (ragged slab, padding to 64) load valid
// clamped addresses and compute on them, but never store.
//
// BL: Bloch columns.  A column is one half of z = u + i v; a value past a face
// of the cell is the wrapped one times exp(+-i k_d L_d), which mixes in the
// other half: rot() wherever a wrapped value enters (x copies in LDS, halo rows,
// ring planes).  The other half's values come by loads of their own, for all
// lanes alike (where none is needed, from one place that stays in cache), so
// that the loads in flight can be counted.
template <typename T, int VX, int MODE, int HM, bool BL>
__global__ __launch_bounds__(256 * sweep_simd_waves(VX * sizeof(T), BL)) void k_hsweep(SweepArgs<T> a) {
    constexpr int NO = kMaxHalfOrder;
    constexpr int RING = kRing, PR = kRingAhead, PQ = kQueue;
    constexpr int PAD = sweep_pad(VX);
    constexpr bool tight = !BL && VX * sizeof(T) == 16 && (HM == 3 || (HM == 2 && MODE == 2 && sizeof(T) == 8));
    constexpr int PH = tight ? 1 : PQ;   // planes that halo rows are loaded ahead
    using gv = typename VecOf<T, VX, sizeof(T)>::type;        // in global memory
    using rv = typename VecOf<T, VX, VX * sizeof(T)>::type;   // in registers and LDS
    extern __shared__ __align__(16) unsigned char smem_raw[];
    const int nx = a.nx, ny = a.ny, nz = a.nz;
    const int W = sweep_row(nx, VX);
    const int R = a.ty + 2 * NO;

    // Hardware dispatches block b to XCD b % 8.  The y-slabs of one orbital (which
    // read each other's rows as halos) share an XCD, so an L2; orbital j goes to
    // XCD j % 8 (Bloch: both halves to (j / 2) % 8), so that the chip works
    // through the block from its first orbital to its last (the nonlocal pass goes
    // back from the last, so each starts on what the last-level cache still holds:
    // 72^3 x 260 FP64 1030 -> 985 us a degree, 51 x 68 x 93 x 77 300 -> 267); the
    // slabs of the last few orbitals are spread evenly over the XCDs.  Within a
    // group of grp of an XCD's orbitals the order is slab-major, so that the
    // grp copies of a slab (which read the same V_eff rows) run side by side.
    const int xcd = blockIdx.x % 8, bslot = blockIdx.x / 8;
    const int cw = BL ? 2 : 1;
    const int own = a.ncol / (8 * cw) * cw;   // orbitals of this XCD alone
    const int rest = (a.ncol - 8 * own) * a.ntiles_y;
    const int rest0 = rest * xcd / 8;
    const int mine = own * a.ntiles_y + rest * (xcd + 1) / 8 - rest0;   // tiles of this XCD
    const int full = mine / a.round * a.round;                          // of them in full rounds
    int item = bslot, zpart = 0, zparts = 1;
    if (bslot >= full) {
        zparts = a.split;
        item = full + (bslot - full) / a.split;
        zpart = (bslot - full) % a.split;
    }
    if (item >= mine) return;
    int tile, col;
    if (item < own * a.ntiles_y) {
        const int gsz = a.grp * a.ntiles_y;
        const int gi = item / gsz, gr = item - gi * gsz;
        const int gcols = min(a.grp, own - gi * a.grp);   // the last group may be short
        tile = gr / gcols;
        const int j = gi * a.grp + (gr - tile * gcols);
        col = (j / cw * 8 + xcd) * cw + j % cw;
    } else {
        const int r = rest0 + item - own * a.ntiles_y;
        col = 8 * own + r / a.ntiles_y;
        tile = r % a.ntiles_y;
    }
    const int y0 = tile * a.ty;
    const int tyn = min(a.ty, ny - y0);
    const int zlen = (nz + zparts - 1) / zparts;
    const int zb = zpart * zlen, ze = min(nz, zb + zlen);
    if (zb >= ze) return;

    const int t = threadIdx.x;
    const int nt = blockDim.x;
    const int LW = nx / VX;
    const int lx = t % LW, ly = t / LW;
    const int x0 = lx * VX;
    const bool active = ly < tyn;
    const bool wleft = x0 < NO, wright = x0 + VX > nx - NO;   // wraps into the padding
    const long plane = (long)nx * ny;

    T* const buf0 = reinterpret_cast<T*>(smem_raw);
    T* const buf1 = buf0 + R * W;

    const long co = (long)(col >> a.halves) * a.ldx + (long)(col & a.halves) * a.half;
    const T* __restrict__ xc = a.x + co;
    T* __restrict__ oc = a.out + co;
    const T* __restrict__ pc = a.xprev ? a.xprev + co : xc;
    const long pxy = x0 + (long)nx * (y0 + (active ? ly : 0));
    const int lrow = ((active ? ly : 0) + NO) * W + PAD + x0;
    auto ld = [](const T* p) -> rv { return *reinterpret_cast<const gv*>(p); };
    // the other half of a Bloch column, and a value of this half times
    // exp(i s k L) (s = +1 past the upper face, -1 past the lower one), in double; one
    // order of rounding, or it would go with the ring phase that a plane falls on
    const T* __restrict__ xo = BL ? a.x + (long)(col >> 1) * a.ldx + (long)((col & 1) ^ 1) * a.half : nullptr;
    const double sgn = (col & 1) ? 1.0 : -1.0;
    auto rot = [&](rv own, rv oth, int axis, int s) -> rv {
        const double cs = a.ph[2 * axis], sn = (s > 0 ? sgn : -sgn) * a.ph[2 * axis + 1];
        rv r;
#pragma unroll
        for (int e = 0; e < VX; ++e) r[e] = (T)fma((double)oth[e], sn, (double)own[e] * cs);
        return r;
    };
    const bool wedge = wleft || wright;
    // halo rows: 2 NO rows of LW vectors per plane, spread over the threads
    int goff[HM], loff[HM];
    int hwrap[HM];   // face that the halo row lies past: -1, 0, +1
    int hn = 0;
    const int nhalo = 2 * NO * LW;
#pragma unroll
    for (int i = 0; i < HM; ++i) {
        const int e = t + i * nt;
        goff[i] = 0;
        loff[i] = 0;
        hwrap[i] = 0;
        if (e < nhalo) {
            hn = i + 1;
            const int hr = e / LW, hl = e - hr * LW;
            const int hx = hl * VX;
            const int lr = hr < NO ? hr : tyn + hr;
            int gy = y0 - NO + lr;
            hwrap[i] = gy < 0 ? -1 : (gy >= ny ? 1 : 0);
            gy = gy < 0 ? gy + ny : (gy >= ny ? gy - ny : gy);
            goff[i] = hx + nx * gy;
            loff[i] = lr * W + PAD + hx;
        }
    }

    double alpha_d, c_d, beta_d;
    filter_coefs(a.params, MODE, a.step, alpha_d, c_d, beta_d);
    // the point's own coefficient with the shift folded in (in double): their
    // difference is small, and one rounding of it replaces two of large terms
    const T alpha = (T)alpha_d, beta = (T)beta_d, cc = (T)(a.c0 - c_d);
    auto wz = [nz](int z) { return z >= nz ? z - nz : (z < 0 ? z + nz : z); };

    rv q[RING];
    rv hq[PH][HM];
    rv xp[PQ], ve[PQ];
    // Bloch: other half of the ring plane loaded last, of the x edges and of the halo rows
    rv oz, ox[PQ], oh[PQ][HM];
    // ring: planes zb - 6 .. zb + 5 + PR (slot = plane - zb mod RING); queues: planes zb .. zb + PQ - 1
#pragma unroll
    for (int j = -NO; j <= NO - 1 + PR; ++j) q[(j + 2 * RING) % RING] = ld(xc + pxy + (long)wz(zb + j) * plane);
#pragma unroll
    for (int j = 0; j < PQ; ++j) {
        const long zo = (long)wz(zb + j) * plane;
        if (MODE == 2) xp[j] = __builtin_nontemporal_load(reinterpret_cast<const gv*>(pc + pxy + zo));
        ve[j] = ld(a.veff + pxy + zo);
    }
#pragma unroll
    for (int j = 1; j < PH; ++j)
#pragma unroll
        for (int i = 0; i < HM; ++i) hq[j][i] = ld(xc + goff[i] + (long)wz(zb + j) * plane);
    auto edge_at = [&](int z) { return wedge ? xo + pxy + (long)wz(z) * plane : xo; };
    auto halo_at = [&](int i, int z) { return hwrap[i] ? xo + goff[i] + (long)wz(z) * plane : xo; };
    if (BL) {
        rv o[2 * NO + PR];
#pragma unroll
        for (int j = -NO; j <= NO - 1 + PR; ++j) {
            const int z = zb + j;
            o[j + NO] = ld(xo + pxy + (z < 0 || z >= nz ? (long)wz(z) * plane : 0L));
        }
#pragma unroll
        for (int j = 0; j < PQ; ++j) {
            ox[j] = ld(edge_at(zb + j));
#pragma unroll
            for (int i = 0; i < HM; ++i) oh[j][i] = ld(halo_at(i, zb + j));
        }
#pragma unroll
        for (int j = -NO; j <= NO - 1 + PR; ++j) {
            const int z = zb + j;
            rv& v = q[(j + 2 * RING) % RING];
            if (z < 0) v = rot(v, o[j + NO], 2, -1);
            else if (z >= nz) v = rot(v, o[j + NO], 2, 1);
        }
    }
    // own points of one plane into a buffer, with the x-wrap copies
    auto put = [&](T* buf, rv v, rv oth) {
        if (active) {
            *reinterpret_cast<rv*>(buf + lrow) = v;
            if (wleft) *reinterpret_cast<rv*>(buf + lrow + nx) = BL ? rot(v, oth, 0, 1) : v;
            if (wright) *reinterpret_cast<rv*>(buf + lrow - nx) = BL ? rot(v, oth, 0, -1) : v;
        }
    };
    auto put_halo = [&](T* buf, int i, rv v, rv oth) {
        if (i < hn) *reinterpret_cast<rv*>(buf + loff[i]) = BL && hwrap[i] ? rot(v, oth, 1, hwrap[i]) : v;
    };
    put(buf0, q[0], ox[0]);
#pragma unroll
    for (int i = 0; i < HM; ++i) put_halo(buf0, i, ld(xc + goff[i] + (long)zb * plane), oh[0][i]);

    for (int z0 = zb; z0 < ze; z0 += RING) {
        if constexpr (BL) {
            auto step = [&](int U, int z) __attribute__((always_inline)) {
#include "sweep_step.inc"
            };
            each_phase(step, z0, ze, std::make_integer_sequence<int, RING>());
        } else {
#pragma unroll
            for (int U = 0; U < RING; ++U) {
                const int z = z0 + U;
                if (z >= ze) break;
#include "sweep_step.inc"
            }
        }
    }
}

// Rounds of a sweep: the slots an XCD has for its workgroups (`round`), and the
// z ranges of the workgroups past its last full round: the number whose rounds
// of (planes + the 8 planes' worth that filling a ring costs) are shortest.  260
// orbitals in 6 slabs leave 6 rounds and 3 workgroups per XCD, and a block of 12
// orbitals never fills one round.  Returns the planes that pass one after
// another, a resident workgroup hiding its share of the ring fills.
static long sweep_rounds(long tiles, int round, int resident, int nz, int* split) {
    const int mine = (int)((tiles + 7) / 8), full = mine / round, rest = mine - full * round;
    *split = 1;
    long least = 0;
    for (int f = 1; f <= std::max(1, nz / 3) && rest; ++f) {
        const long cost = (long)div_up((long)rest * f, round) * (div_up(nz, f) + 8);
        if (f == 1 || cost < least) {
            *split = f;
            least = cost;
        }
    }
    return full * (nz + 8L / resident) + least;
}

// Slab height of the sweep: the one with the least (planes one after another)
// x (time of a plane).  The latter goes with the points that the resident
// workgroups compute and, at a quarter (mostly L2 hits), the halo rows they read;
// from 6 waves per compute unit on the loads hide each other (72^3 x 260 FP64:
// 484 us with 7 and with 11 waves).  Slabs of less than 12 rows need two halo
// vectors per thread, which spills (72^3: 700 us with 7 rows).
static SweepPlan sweep_plan(sparc_gpu_ctx c, int vx, size_t tsize, int ncol, bool bloch) {
    const int nx = c->nx, ny = c->ny, lw = nx / vx, halo = 2 * kMaxHalfOrder;
    int forced = 0;   // tuning override: rows per y-slab
    if (const char* e = std::getenv("SPARC_GPU_SWEEP_TY")) forced = std::atoi(e);
    SweepPlan& plan = c->sweep_plans[(tsize == 8) + 2 * bloch];
    if (plan.ncol == ncol && plan.forced == forced) return plan;
    const int max_waves = 4 * sweep_simd_waves(vx * tsize, bloch), max_threads = 64 * max_waves;
    SweepPlan best;
    double least = 0;
    for (int ty = bloch ? 2 : 4; ty <= ny; ++ty) {
        SweepPlan s;
        s.ncol = ncol;
        s.forced = forced;
        s.vx = vx;
        s.ty = ty;
        s.threads = div_up((long)lw * ty, 64) * 64;
        if (s.threads > max_threads) break;
        s.lds = 2 * (size_t)(ty + halo) * sweep_row(nx, vx) * tsize;
        if (s.lds > 160 * 1024) break;
        const int waves = s.threads / 64;
        const int resident = std::max(1, std::min((int)(160 * 1024 / s.lds), max_waves / waves));
        s.round = std::max(1, c->prop.multiProcessorCount / 8) * resident;
        const double plane = resident * (ty + 0.25 * halo) * std::max(1.0, 6.0 / (resident * waves)) *
                             (halo * lw > s.threads && !bloch ? 1.5 : 1.0);
        const double cost =
            plane * sweep_rounds((long)ncol * div_up(ny, ty), s.round, resident, c->nz, &s.split);
        if (best.ty < 4 || ty == forced || (cost < least && best.ty != forced)) {
            least = cost;
            best = s;
        }
    }
    plan = best;
    return best;
}

template <typename T>
static const StencilCoef<T>& coef(sparc_gpu_ctx c);
template <>
const StencilCoef<double>& coef<double>(sparc_gpu_ctx c) {
    return c->cf64;
}
template <>
const StencilCoef<float>& coef<float>(sparc_gpu_ctx c) {
    return c->cf32;
}

template <typename T>
static const T* veff_of(sparc_gpu_ctx c);
template <>
const double* veff_of<double>(sparc_gpu_ctx c) {
    return c->veff;
}
template <>
const float* veff_of<float>(sparc_gpu_ctx c) {
    return c->veff32;
}

template <typename T>
sparc_status launch_hsweep(sparc_gpu_ctx c, const T* x, T* out, const T* xprev, int ncol, long ldx, int mode,
                           int step, bool halves) {
    hipStream_t stream = c->stream;
    SweepArgs<T> a;
    a.x = x;
    a.out = out;
    a.xprev = xprev;
    a.ldx = ldx;
    a.halves = halves ? 1 : 0;
    a.half = c->nd;
    {
        const double kl[3] = {c->kvec[0] * c->Lx, c->kvec[1] * c->Ly, c->kvec[2] * c->Lz};
        for (int d = 0; d < 3; ++d) {
            a.ph[2 * d] = std::cos(kl[d]);
            a.ph[2 * d + 1] = std::sin(kl[d]);
        }
    }
    a.nx = c->nx;
    a.ny = c->ny;
    a.nz = c->nz;
    const SweepPlan sh = sweep_plan(c, sweep_vx<T>(c->nx), sizeof(T), ncol, halves);
    if (sh.ty == 0) return set_err(c, SPARC_ERR_ARG, "grid x-extent too large for the sweep kernel");
    a.ty = sh.ty;
    a.ntiles_y = div_up(c->ny, a.ty);
    a.grp = std::max(1, std::min(c->sweep_group, ncol));
    {
        const StencilCoef<T>& cf = coef<T>(c);
        a.c0 = c->cf64.c0;
        for (int k = 0; k <= kMaxHalfOrder; ++k) {
            a.cx[k] = cf.cx[k];
            a.cy[k] = cf.cy[k];
            a.cz[k] = cf.cz[k];
        }
    }
    a.veff = veff_of<T>(c);
    a.params = c->scal + S_A;
    a.step = step;
    a.ncol = ncol;
    const int hm = div_up(2L * kMaxHalfOrder * (c->nx / sh.vx), sh.threads);   // 1 to 3; 6 with slabs of 2 rows
    const long tiles = (long)ncol * a.ntiles_y;
    if (tiles > 0x3fffffffL) return set_err(c, SPARC_ERR_ARG, "too many blocks");
    if (tiles == 0) return SPARC_OK;
    a.round = sh.round;
    a.split = sh.split;
    // per XCD: whole tiles, then the split ones (of the larger or smaller of
    // the two shares that XCDs get)
    long slots = 0;
    for (long n : {tiles / 8, (tiles + 7) / 8}) {
        const long whole = n / a.round * a.round;
        slots = std::max(slots, whole + (n - whole) * a.split);
    }
    const int slot = prof_begin(
        c, halves ? PK_BLOCH : mode == 2 && step > 0 ? PK_SWEEP : mode == 1 ? PK_SWEEP1 : PK_APPLY, stream);
    const dim3 g((unsigned)(8 * slots)), b(sh.threads);
    auto go = [&](auto vx, auto mv, auto hv, auto bl) {
        k_hsweep<T, vx(), mv(), hv(), bl()><<<g, b, sh.lds, stream>>>(a);
    };
    auto go_halo = [&](auto vx, auto mv, auto bl) {
        if (hm == 1) go(vx, mv, std::integral_constant<int, 1>(), bl);
        else if (hm == 2) go(vx, mv, std::integral_constant<int, 2>(), bl);
        else if (!(vx() == 1 && bl()) || hm == 3) go(vx, mv, std::integral_constant<int, 3>(), bl);
        else go(std::integral_constant<int, 1>(), mv, std::integral_constant<int, kSweepMaxHalo>(), std::true_type());
    };
    auto go_width = [&](auto mv, auto bl) {
        if (sh.vx == 1) return go_halo(std::integral_constant<int, 1>(), mv, bl);
        if constexpr (sizeof(T) == 4)
            if (sh.vx == 4) return go_halo(std::integral_constant<int, 4>(), mv, bl);
        go_halo(std::integral_constant<int, 2>(), mv, bl);
    };
    auto go_mode = [&](auto bl) {
        if (mode == 0) go_width(std::integral_constant<int, 0>(), bl);
        else if (mode == 1) go_width(std::integral_constant<int, 1>(), bl);
        else go_width(std::integral_constant<int, 2>(), bl);
    };
    if (halves) go_mode(std::true_type());
    else go_mode(std::false_type());
    SG_CHECK_LAUNCH(c);
    prof_end(c, slot, stream);
    return SPARC_OK;
}

template sparc_status launch_hsweep<double>(sparc_gpu_ctx, const double*, double*, const double*, int, long, int, int,
                                            bool);
template sparc_status launch_hsweep<float>(sparc_gpu_ctx, const float*, float*, const float*, int, long, int, int,
                                           bool);

// ---- allocation-free filter -----------------------------------------------
// The projection partials of sparc_gpu_chebyshev_filter_noalloc live in this
// fixed array (64 MiB; each GPU the library runs on holds its own copy until
// the process ends) instead of memory the library allocates.  Host code never
// names the array: it uses the device address looked up once per device by
// scratch_init.  Calls that overlap on one GPU share it and race.  Its size sets
// the columns of a group: 120^3 x 600 with 500 atoms, 6 degrees in FP64, 90 ms in
// groups of 112 (32 MiB, 320 workgroups of the pass on 512 places), 75 in groups of 240.
constexpr size_t kScratchDoubles = (size_t)8 << 20;
static __device__ __align__(256) double scratch[kScratchDoubles];

sparc_status scratch_init(sparc_gpu_ctx c, int dev) {
    static std::mutex mu;
    static std::map<int, double*> addr;   // device -> address of its copy of the array
    std::lock_guard<std::mutex> lock(mu);
    auto it = addr.find(dev);
    if (it == addr.end()) {
        void* ptr = nullptr;
        const hipError_t e = hipGetSymbolAddress(&ptr, HIP_SYMBOL(scratch));
        if (e != hipSuccess || !ptr) return hip_err(c, e != hipSuccess ? e : hipErrorInvalidSymbol, "scratch address");
        it = addr.emplace(dev, static_cast<double*>(ptr)).first;
    }
    c->scratch = it->second;
    c->scratch_elems = kScratchDoubles;
    return SPARC_OK;
}

template <typename T>
sparc_status apply_impl(sparc_gpu_ctx c, const T* X, T* Y, int ncol, long ldx) {
    // the projecting pass only reads X
    sparc_status st = nl_pass<T>(c, const_cast<T*>(X), ncol, ldx, NlApply::no, true, 0, 0);
    if (st != SPARC_OK) return st;
    // V_nl X first and the local part added to it, where that pays: the sweep reads
    // faster than the pass, above all where planes are no multiple of 128 bytes
    // (99 x 98 x 81 x 504 in FP64 4480 us, with the pass last 4720; 72^3 x 260 1060
    // and 1100)
    if (nl_writes(c, ncol, sizeof(T) == 4, false)) {
        if ((st = nl_pass<T>(c, Y, ncol, ldx, NlApply::write, false, 0, 0)) != SPARC_OK) return st;
        return launch_hsweep<T>(c, X, Y, Y, ncol, ldx, 2, 0);
    }
    if ((st = launch_hsweep<T>(c, X, Y, nullptr, ncol, ldx, 0, 0)) != SPARC_OK) return st;
    return nl_pass<T>(c, Y, ncol, ldx, NlApply::add, false, 0, 0);
}
template sparc_status apply_impl<double>(sparc_gpu_ctx, const double*, double*, int, long);
template sparc_status apply_impl<float>(sparc_gpu_ctx, const float*, float*, int, long);

template <typename T>
__global__ void k_copy_block(const T* __restrict__ src, T* __restrict__ dst, long nd, int ncol, long ld) {
    long i = (long)blockIdx.x * blockDim.x + threadIdx.x;
    int j = blockIdx.y;
    if (i < nd && j < ncol) dst[i + (long)j * ld] = src[i + (long)j * ld];
}

// Filter with bounds already in c->scal[S_A..S_A0].  Y_k lives in X when k is
// even and in W when k is odd; the result ends in X.  Each local sweep is
// followed by the nonlocal pass that completes Y_k with the projections of
// Y_{k-1} and forms those of Y_k.
template <typename T>
sparc_status filter_impl(sparc_gpu_ctx c, T* X, T* Wk, int ncol, long ldx, int m, double* part, size_t part_elems) {
    sparc_status st;
    if ((st = nl_pass<T>(c, X, ncol, ldx, NlApply::no, true, 1, 1, part, part_elems)) != SPARC_OK) return st;
    for (int k = 1; k <= m; ++k) {
        T* cur = (k % 2 == 0) ? Wk : X;   // Y_{k-1}
        T* dst = (k % 2 == 0) ? X : Wk;   // Y_{k-2}, overwritten with Y_k
        const int mode = k == 1 ? 1 : 2;
        if ((st = launch_hsweep<T>(c, cur, dst, k == 1 ? nullptr : dst, ncol, ldx, mode, k)) != SPARC_OK) return st;
        if ((st = nl_pass<T>(c, dst, ncol, ldx, NlApply::add, k < m, 2, k + 1, part, part_elems)) != SPARC_OK) return st;
    }
    if (m % 2 == 1) {
        dim3 grid(div_up(c->nd, 256), ncol);
        const int slot = prof_begin(c, PK_COPY);
        k_copy_block<T><<<grid, 256, 0, c->stream>>>(Wk, X, c->nd, ncol, ldx);
        SG_CHECK_LAUNCH(c);
        prof_end(c, slot);
    }
    return SPARC_OK;
}

template sparc_status filter_impl<double>(sparc_gpu_ctx, double*, double*, int, long, int, double*, size_t);
template sparc_status filter_impl<float>(sparc_gpu_ctx, float*, float*, int, long, int, double*, size_t);

__global__ void k_set3(double* dst, double a, double b, double c) {
    dst[0] = a;
    dst[1] = b;
    dst[2] = c;
}

__global__ void k_veff_convert(const double* src, double* dst, float* dst32, long n) {
    long i = (long)blockIdx.x * blockDim.x + threadIdx.x;
    if (i < n) {
        double v = src[i];
        dst[i] = v;
        dst32[i] = (float)v;
    }
}

sparc_status set_veff_impl(sparc_gpu_ctx c, const double* d_veff) {
    if (d_veff != c->veff) {
        k_veff_convert<<<div_up(c->nd, 256), 256, 0, c->stream>>>(d_veff, c->veff, c->veff32, c->nd);
    } else {
        k_veff_convert<<<div_up(c->nd, 256), 256, 0, c->stream>>>(c->veff, c->veff, c->veff32, c->nd);
    }
    SG_CHECK_LAUNCH(c);
    return SPARC_OK;
}

// lo = min V_eff + nl_lo, hi = kin + max V_eff + nl_hi
// Extrema of V_eff: per-block partials (part[2 b], part[2 b + 1]), then one
// block combines them into the spectrum bounds.
__global__ __launch_bounds__(256) void k_minmax_part(const double* v, long n, double* part) {
    __shared__ double smin[256], smax[256];
    double mn = 1e300, mx = -1e300;
    for (long i = (long)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += (long)gridDim.x * blockDim.x) {
        const double x = v[i];
        mn = fmin(mn, x);
        mx = fmax(mx, x);
    }
    smin[threadIdx.x] = mn;
    smax[threadIdx.x] = mx;
    __syncthreads();
    for (int s = blockDim.x / 2; s > 0; s >>= 1) {
        if (threadIdx.x < s) {
            smin[threadIdx.x] = fmin(smin[threadIdx.x], smin[threadIdx.x + s]);
            smax[threadIdx.x] = fmax(smax[threadIdx.x], smax[threadIdx.x + s]);
        }
        __syncthreads();
    }
    if (threadIdx.x == 0) {
        part[2 * blockIdx.x] = smin[0];
        part[2 * blockIdx.x + 1] = smax[0];
    }
}

__global__ __launch_bounds__(256) void k_bounds(const double* part, int nblk, double kin, double nl_lo,
                                                double nl_hi, double* out_lo, double* out_hi) {
    __shared__ double smin[256], smax[256];
    double mn = 1e300, mx = -1e300;
    for (int b = threadIdx.x; b < nblk; b += blockDim.x) {
        mn = fmin(mn, part[2 * b]);
        mx = fmax(mx, part[2 * b + 1]);
    }
    smin[threadIdx.x] = mn;
    smax[threadIdx.x] = mx;
    __syncthreads();
    for (int s = blockDim.x / 2; s > 0; s >>= 1) {
        if (threadIdx.x < s) {
            smin[threadIdx.x] = fmin(smin[threadIdx.x], smin[threadIdx.x + s]);
            smax[threadIdx.x] = fmax(smax[threadIdx.x], smax[threadIdx.x + s]);
        }
        __syncthreads();
    }
    if (threadIdx.x == 0) {
        *out_lo = smin[0] + nl_lo;
        *out_hi = kin + smax[0] + nl_hi;
    }
}

sparc_status bounds_impl(sparc_gpu_ctx c) {
    const int nblk = (int)std::min<long>(512, div_up(c->nd, 256));
    sparc_status st = ensure_red(c, 2 * (size_t)nblk);
    if (st != SPARC_OK) return st;
    k_minmax_part<<<nblk, 256, 0, c->stream>>>(c->veff, c->nd, c->red);
    k_bounds<<<1, 256, 0, c->stream>>>(c->red, nblk, c->kin_bound, c->nl.nl_lo, c->nl.nl_hi, c->scal + S_LO,
                                      c->scal + S_HI);
    SG_CHECK_LAUNCH(c);
    return SPARC_OK;
}

static sparc_status check_block(sparc_gpu_ctx c, int prec, const void* X, int ncol, long ldx, const char* who) {
    if (prec != SPARC_FP64 && prec != SPARC_FP32) return set_err(c, SPARC_ERR_ARG, std::string(who) + ": bad precision");
    if (!X) return set_err(c, SPARC_ERR_ARG, std::string(who) + ": null block");
    if (ncol < 1 || ncol > c->n_states) return set_err(c, SPARC_ERR_ARG, std::string(who) + ": ncol out of range");
    if (ldx < c->nd) return set_err(c, SPARC_ERR_ARG, std::string(who) + ": ldx < N_d");
    return SPARC_OK;
}

static bool overlaps(const void* a, const void* b, size_t bytes) {
    const char* pa = (const char*)a;
    const char* pb = (const char*)b;
    return pa < pb + bytes && pb < pa + bytes;
}

}  // namespace sg

using namespace sg;

extern "C" {

sparc_status sparc_gpu_apply_H(sparc_gpu_ctx c, sparc_prec prec, const void* d_X, void* d_Y, int ncol, long ldx) {
    if (!c) return SPARC_ERR_ARG;
    c->err.clear();
    sparc_status st = check_block(c, prec, d_X, ncol, ldx, "apply_H");
    if (st != SPARC_OK) return st;
    if (!d_Y) return set_err(c, SPARC_ERR_ARG, "apply_H: null output");
    size_t es = prec == SPARC_FP64 ? 8 : 4;
    size_t bytes = ((size_t)(ncol - 1) * ldx + c->nd) * es;
    if (overlaps(d_X, d_Y, bytes)) return set_err(c, SPARC_ERR_ARG, "apply_H: X and Y overlap");
    if (prec == SPARC_FP64) return apply_impl<double>(c, (const double*)d_X, (double*)d_Y, ncol, ldx);
    return apply_impl<float>(c, (const float*)d_X, (float*)d_Y, ncol, ldx);
}

sparc_status sparc_gpu_chebyshev_filter(sparc_gpu_ctx c, sparc_prec prec, void* d_X, void* d_work, int ncol,
                                        long ldx, int degree, double a, double b, double a0) {
    if (!c) return SPARC_ERR_ARG;
    c->err.clear();
    sparc_status st = check_block(c, prec, d_X, ncol, ldx, "chebyshev_filter");
    if (st != SPARC_OK) return st;
    if (!d_work) return set_err(c, SPARC_ERR_ARG, "chebyshev_filter: null work block");
    if (degree < 1 || degree > 10000) return set_err(c, SPARC_ERR_ARG, "chebyshev_filter: degree out of range");
    if (!(a0 < a && a < b) || !std::isfinite(a0) || !std::isfinite(b))
        return set_err(c, SPARC_ERR_ARG, "chebyshev_filter: need a0 < a < b");
    size_t es = prec == SPARC_FP64 ? 8 : 4;
    size_t bytes = ((size_t)(ncol - 1) * ldx + c->nd) * es;
    if (overlaps(d_X, d_work, bytes)) return set_err(c, SPARC_ERR_ARG, "chebyshev_filter: X and work overlap");
    k_set3<<<1, 1, 0, c->stream>>>(c->scal + S_A, a, b, a0);
    SG_CHECK_LAUNCH(c);
    if (prec == SPARC_FP64) return filter_impl<double>(c, (double*)d_X, (double*)d_work, ncol, ldx, degree);
    return filter_impl<float>(c, (float*)d_X, (float*)d_work, ncol, ldx, degree);
}

sparc_status sparc_gpu_chebyshev_filter_noalloc(sparc_gpu_ctx c, sparc_prec prec, void* d_X, void* d_work, int ncol,
                                                long ldx, int degree, double a, double b, double a0) {
    if (!c) return SPARC_ERR_ARG;
    c->err.clear();
    sparc_status st = check_block(c, prec, d_X, ncol, ldx, "chebyshev_filter_noalloc");
    if (st != SPARC_OK) return st;
    if (!d_work) return set_err(c, SPARC_ERR_ARG, "chebyshev_filter_noalloc: null work block");
    if (degree < 1 || degree > 10000) return set_err(c, SPARC_ERR_ARG, "chebyshev_filter_noalloc: degree out of range");
    if (!(a0 < a && a < b) || !std::isfinite(a0) || !std::isfinite(b))
        return set_err(c, SPARC_ERR_ARG, "chebyshev_filter_noalloc: need a0 < a < b");
    size_t es = prec == SPARC_FP64 ? 8 : 4;
    size_t bytes = ((size_t)(ncol - 1) * ldx + c->nd) * es;
    if (overlaps(d_X, d_work, bytes)) return set_err(c, SPARC_ERR_ARG, "chebyshev_filter_noalloc: X and work overlap");
    if (!c->scratch) return set_err(c, SPARC_ERR_ARG, "chebyshev_filter_noalloc: no scratch array on this device");
    k_set3<<<1, 1, 0, c->stream>>>(c->scal + S_A, a, b, a0);
    SG_CHECK_LAUNCH(c);
    // no timing events either (creating them could allocate)
    const bool prof = c->prof;
    c->prof = false;
    const sparc_status r =
        prec == SPARC_FP64
            ? filter_impl<double>(c, (double*)d_X, (double*)d_work, ncol, ldx, degree, c->scratch, c->scratch_elems)
            : filter_impl<float>(c, (float*)d_X, (float*)d_work, ncol, ldx, degree, c->scratch, c->scratch_elems);
    c->prof = prof;
    return r;
}

}  // extern "C"
