// Hellmann-Feynman atomic forces (Sec. 2: the forces used for structural
// relaxation and molecular dynamics).  At self-consistency only the explicit
// position dependence of the free energy contributes:
//   local     F_I = dV sum_x phi(x) grad b_I(x - R_I)
//                   - 1/2 dV sum over the atom's ball of grad(b_I V_I)
//   overlap   F_I = sum_{J,n}' Z_I Z_J u'(d) (R_J + nL - R_I) / d,  u(d) = erfc(d/s)/d
//   nonlocal  F_I = 2 sum_n w_n sum_k gamma_Ik (dV chi_Ik^T psi_n)(dV (grad chi_Ik)^T psi_n)
// Every sum runs over the same (grid point, periodic image) pairs as the
// corresponding energy: unwrapped grid indices inside the truncation sphere
// around the atom, wrapped to the periodic grid for field values.
// Reductions are in fixed order (no value atomics), so results are
// bitwise reproducible.
#include <type_traits>

#include "force_lines.hpp"
#include "internal.hpp"
#include "mfma.hpp"

namespace sg {

namespace {

constexpr double kPi = 3.14159265358979323846;

// Per-atom table: [x, y, z] * n | Z * n | rc * n | gamma (4 per atom) * n
struct ForceTab {
    const double* pos;
    const double* Z;
    const double* rc;
    const double* gamma4;
};

inline ForceTab force_tab(sparc_gpu_ctx c) {
    const int n = c->n_atoms;
    return ForceTab{c->force_tab, c->force_tab + 3 * n, c->force_tab + 4 * n, c->force_tab + 5 * n};
}

__device__ inline int wrap(int i, int n) {
    int r = i % n;
    return r < 0 ? r + n : r;
}

// Fixed-order block reduction of NV values per thread (256 threads): wave
// shuffles, then the four waves in order.  Returns the block sum of value
// q = threadIdx.x for threads below NV (0 elsewhere).
template <int NV>
__device__ inline double block_reduce(const double (&v)[NV], double (*lds)[NV]) {
    const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
#pragma unroll
    for (int q = 0; q < NV; ++q) {
        double t = v[q];
        for (int off = 32; off > 0; off >>= 1) t += __shfl_down(t, off, 64);
        if (lane == 0) lds[w][q] = t;
    }
    __syncthreads();
    const int q = threadIdx.x;
    return q < NV ? ((lds[0][q] + lds[1][q]) + lds[2][q]) + lds[3][q] : 0.0;
}

// Local part: block (atom, chunk of the z-range of its 8 rc box).
__global__ __launch_bounds__(256) void k_force_local(ForceTab tab, const double* __restrict__ phi, int nx, int ny,
                                                    int nz, double hx, double hy, double hz, double dV, int nchunk,
                                                    double* __restrict__ part) {
    const int a = blockIdx.x, ch = blockIdx.y;
    const double Z = tab.Z[a], rc = tab.rc[a];
    const double cx = tab.pos[3 * a], cy = tab.pos[3 * a + 1], cz = tab.pos[3 * a + 2];
    const double rmax = 8.0 * rc, rmax2 = rmax * rmax;
    const int lx = (int)ceil((cx - rmax) / hx), ux = (int)floor((cx + rmax) / hx);
    const int ly = (int)ceil((cy - rmax) / hy), uy = (int)floor((cy + rmax) / hy);
    const int lz = (int)ceil((cz - rmax) / hz), uz = (int)floor((cz + rmax) / hz);
    const int nxb = ux - lx + 1, nyb = uy - ly + 1, nzb = uz - lz + 1;
    const int z0 = lz + (int)((long)nzb * ch / nchunk), z1 = lz + (int)((long)nzb * (ch + 1) / nchunk);
    const long tot = (long)nxb * nyb * (z1 - z0);
    const double amp = -Z * pow(kPi * rc * rc, -1.5);
    const double inv = 1.0 / (rc * rc);
    double acc[3] = {0.0, 0.0, 0.0};
    for (long t = threadIdx.x; t < tot; t += blockDim.x) {
        const int i = lx + (int)(t % nxb);
        const int j = ly + (int)((t / nxb) % nyb);
        const int k = z0 + (int)(t / ((long)nxb * nyb));
        const double dx = i * hx - cx, dy = j * hy - cy, dz = k * hz - cz;
        const double r2 = dx * dx + dy * dy + dz * dz;
        if (r2 > rmax2) continue;
        const double ex = exp(-r2 * inv);
        const double b = amp * ex;
        const double r = sqrt(r2);
        const double V = (r < 1e-12) ? -2.0 * Z / (sqrt(kPi) * rc) : -Z * erf(r / rc) / r;
        // V'(r) / r, with its finite limit at r -> 0
        const double dVr = (r < 1e-8) ? 4.0 * Z / (3.0 * sqrt(kPi) * rc * rc * rc)
                                      : (Z * erf(r / rc) / r2 - Z * 2.0 / (sqrt(kPi) * rc) * ex / r) / r;
        const double ph = phi[wrap(i, nx) + (long)nx * (wrap(j, ny) + (long)ny * wrap(k, nz))];
        const double g = -2.0 * inv * b;    // grad b = g d
        const double s = ph * g - 0.5 * (V * g + b * dVr);
        acc[0] += s * dx;
        acc[1] += s * dy;
        acc[2] += s * dz;
    }
    __shared__ double lds[4][3];
    const double sum = block_reduce<3>(acc, lds);
    if (threadIdx.x < 3) part[((long)a * nchunk + ch) * 3 + threadIdx.x] = dV * sum;
}

// out[3 a + d] = sum over chunks (in order) of the local partials
__global__ void k_force_local_reduce(const double* __restrict__ part, int n_atoms, int nchunk,
                                     double* __restrict__ out) {
    const long t = (long)blockIdx.x * blockDim.x + threadIdx.x;
    if (t >= 3L * n_atoms) return;
    const long a = t / 3, d = t % 3;
    double s = 0.0;
    for (int ch = 0; ch < nchunk; ++ch) s += part[(a * nchunk + ch) * 3 + d];
    out[t] = s;
}

// Overlap part, added to out: one block per atom I, threads over J.
__global__ __launch_bounds__(256) void k_force_overlap(ForceTab tab, int n_atoms, double Lx, double Ly, double Lz,
                                                      double rmax, int nimx, int nimy, int nimz,
                                                      double* __restrict__ out) {
    const int I = blockIdx.x;
    double acc[3] = {0.0, 0.0, 0.0};
    const double xI = tab.pos[3 * I], yI = tab.pos[3 * I + 1], zI = tab.pos[3 * I + 2];
    for (int J = threadIdx.x; J < n_atoms; J += blockDim.x) {
        const double s = sqrt(tab.rc[I] * tab.rc[I] + tab.rc[J] * tab.rc[J]);
        const double zz = tab.Z[I] * tab.Z[J];
        for (int a = -nimx; a <= nimx; ++a)
            for (int b = -nimy; b <= nimy; ++b)
                for (int c = -nimz; c <= nimz; ++c) {
                    if (I == J && a == 0 && b == 0 && c == 0) continue;
                    const double vx = tab.pos[3 * J] + a * Lx - xI;
                    const double vy = tab.pos[3 * J + 1] + b * Ly - yI;
                    const double vz = tab.pos[3 * J + 2] + c * Lz - zI;
                    const double d = sqrt(vx * vx + vy * vy + vz * vz);
                    if (!(d < rmax)) continue;
                    const double du = -erfc(d / s) / (d * d) - 2.0 / (sqrt(kPi) * s) * exp(-(d / s) * (d / s)) / d;
                    const double f = zz * du / d;
                    acc[0] += f * vx;
                    acc[1] += f * vy;
                    acc[2] += f * vz;
                }
    }
    __shared__ double lds[4][3];
    const double sum = block_reduce<3>(acc, lds);
    if (threadIdx.x < 3) out[3 * I + threadIdx.x] += sum;
}

constexpr int kForceTiles = 5;   // 16-column tiles of a workgroup at most

// Projections of the columns on the atom's projectors and their gradients:
// pd[((part n_atoms + a) ncol + col) 16 + q] with q = k (chi_k^T psi, k = s, px,
// py, pz) and q = 4 + 3 k + d ((d/dx_d chi_k)^T psi), each times dV; parts are
// added later.
//
// The 16 functions of an atom are the rows of one FP64 MFMA tile.  A workgroup
// takes an atom, up to 80 columns (TL tiles of 16) and one of `parts` shares of the
// x-lines of the atom's sphere, its waves every (4 parts)-th of them, 24 points at
// a time with the next ones' loads in flight, and for each point every lane forms
// the one function of its row,
//   f_q = exp(-r^2 / rc^2) (c0 + c1 u v),   u, v each 1, dx, dy or dz,
// which all columns then share.  Reading is what bounds it: the lanes of a wave
// hold 16 different columns, so that a load of 8 bytes per lane costs the L1 57
// accesses, and the overlapping spheres read the block 5 times (4 GB at 72^3, 108
// atoms, 260 columns).  There 1.95 ms as vector code with the 16 sums of four
// columns per thread; 1.27 on the matrix cores with loads of single points, 1.06
// with pairs, 0.86 in three parts whose lines outside the sphere are skipped (the
// products alone would take 0.13).  Neighbouring atoms on one XCD made no
// difference.
template <typename T, int TL>
__global__ __launch_bounds__(256, 2) void k_force_nl_proj(const T* __restrict__ X, long ldx, int ncol, ForceTab tab,
                                                          int nx, int ny, int nz, double hx, double hy, double hz,
                                                          double rc, double rcut, double N0, double N1, double dV,
                                                          double* __restrict__ pd) {
    constexpr int CH = kForcePoints / 8;   // 8-point chunks of a step
    __shared__ double ex[3][256];   // Gaussian factors along the box's axes (at most 255 points)
    __shared__ double red[4][16][16 * TL];
    const int a = blockIdx.x, col0 = 16 * TL * blockIdx.y, parts = gridDim.z, part = blockIdx.z;
    const double cx = tab.pos[3 * a], cy = tab.pos[3 * a + 1], cz = tab.pos[3 * a + 2];
    const ForceBox B = force_box(cx, cy, cz, hx, hy, hz, rcut);
    const int lx = B.lx, ly = B.ly, lz = B.lz;
    const int t = threadIdx.x, lane = t & 63, li = lane & 15, g = lane >> 4;
    for (int i = t; i < 256; i += blockDim.x) {
        const double dx = (lx + i) * hx - cx, dy = (ly + i) * hy - cy, dz = (lz + i) * hz - cz;
        ex[0][i] = exp(-dx * dx / (rc * rc));
        ex[1][i] = exp(-dy * dy / (rc * rc));
        ex[2][i] = exp(-dz * dz / (rc * rc));
    }
    __syncthreads();
    // the lane's function: c0 + c1 u v
    const double gr = -2.0 / (rc * rc);
    const int ku = li < 4 ? li - 1 : (li < 7 ? li - 4 : (li - 7) / 3);   // axis of u, -1: one
    const int kv = li < 7 ? -1 : (li - 7) % 3;
    const double c0 = li == 0 ? N0 : (li >= 7 && ku == kv ? N1 : 0.0);
    const double c1 = li == 0 ? 0.0 : (li < 4 ? N1 : (li < 7 ? N0 * gr : N1 * gr));
    const double u1 = ku < 0 ? 1.0 : 0.0, uX = ku == 0 ? 1.0 : 0.0, uY = ku == 1 ? 1.0 : 0.0, uZ = ku == 2 ? 1.0 : 0.0;
    const double v1 = kv < 0 ? 1.0 : 0.0, vX = kv == 0 ? 1.0 : 0.0, vY = kv == 1 ? 1.0 : 0.0, vZ = kv == 2 ? 1.0 : 0.0;
    // columns past the last repeat it and are not stored
    const int nt = min(TL, (ncol - col0 + 15) / 16);
    const T* xc[TL];
#pragma unroll
    for (int k = 0; k < TL; ++k) xc[k] = X + (long)min(ncol - 1, col0 + 16 * min(k, nt - 1) + li) * ldx;
    using acc_t = Mfma<double>::acc_t;
    typedef T vec __attribute__((ext_vector_type(2), aligned(sizeof(T))));
    acc_t acc[TL];
#pragma unroll
    for (int k = 0; k < TL; ++k) acc[k] = acc_t{0, 0, 0, 0};

    // a step of the walk over the sphere's lines; x0: its first point on the grid
    struct Step : ForceStep {
        int x0;
    };
    auto advance = [&](Step& s) -> bool {
        if (!force_advance(B, s, 4 * parts, [](int v) { return __builtin_amdgcn_readfirstlane(v); })) return false;
        s.x0 = wrap(lx + s.i0, nx);
        return true;
    };
    // pairs of points by one load, which never passes a row's end (the pair of a
    // row's last point starts one earlier); a step that wraps by single points
    auto load = [&](const Step& s, vec (&x)[CH][TL]) {
        const long row = (long)nx * (wrap(ly + s.j, ny) + (long)ny * wrap(lz + s.k, nz));
        if (s.x0 + s.n <= nx) {
#pragma unroll
            for (int c = 0; c < CH; ++c) {
                const long o = row + min(s.x0 + min(8 * c + 2 * g, s.n - 1), nx - 2);
#pragma unroll
                for (int k = 0; k < TL; ++k) x[c][k] = *reinterpret_cast<const vec*>(xc[k] + o);
            }
        } else {
#pragma unroll
            for (int c = 0; c < CH; ++c)
#pragma unroll
                for (int u = 0; u < 2; ++u) {
                    const long o = row + wrap(s.x0 + min(8 * c + 2 * g + u, s.n - 1), nx);
#pragma unroll
                    for (int k = 0; k < TL; ++k) x[c][k][u] = xc[k][o];
                }
        }
    };
    auto compute = [&](const Step& s, const vec (&x)[CH][TL]) {
        const double dy = (ly + s.j) * hy - cy, dz = (lz + s.k) * hz - cz;
        const double eyz = ex[1][s.j] * ex[2][s.k];
        const double ub = u1 + uY * dy + uZ * dz, vb = v1 + vY * dy + vZ * dz;
#pragma unroll
        for (int c = 0; c < CH; ++c) {
            if (8 * c >= s.n) break;
            const bool late = s.x0 + 8 * c + 2 * g == nx - 1 && s.x0 + s.n <= nx;
#pragma unroll
            for (int u = 0; u < 2; ++u) {
                const int e = 8 * c + 2 * g + u, i = s.i0 + min(e, s.n - 1);
                const double dx = (lx + i) * hx - cx;
                const bool in = e < s.n && dx * dx + dy * dy + dz * dz <= B.rcut2;
                const double f = in ? ex[0][i] * eyz * (c0 + c1 * (ub + uX * dx) * (vb + vX * dx)) : 0.0;
#pragma unroll
                for (int k = 0; k < TL; ++k)
                    if (k < nt)
                        acc[k] = Mfma<double>::run(f, in ? (double)(late ? x[c][k][1] : x[c][k][u]) : 0.0, acc[k]);
            }
        }
    };
    Step s{{__builtin_amdgcn_readfirstlane(4 * part + (t >> 6) - 4 * parts), 0, 0, 0, 1, 0}, 0};
    vec xa[CH][TL], xb[CH][TL];
    bool more = advance(s);
    if (more) load(s, xa);
    while (more) {
        Step s2 = s;
        const bool m2 = advance(s2);
        if (m2) load(s2, xb);
        compute(s, xa);
        if (!m2) break;
        s = s2;
        more = advance(s);
        if (more) load(s, xa);
        compute(s2, xb);
    }
#pragma unroll
    for (int k = 0; k < TL; ++k)
#pragma unroll
        for (int r = 0; r < 4; ++r) red[t >> 6][Mfma<double>::row(lane, r)][16 * k + li] = acc[k][r];
    __syncthreads();
    for (int e = t; e < 256 * nt; e += blockDim.x) {
        const int q = e & 15, c = e >> 4;
        if (col0 + c < ncol)
            pd[(((long)part * gridDim.x + a) * ncol + col0 + c) * 16 + q] =
                dV * (red[0][q][c] + red[1][q][c] + red[2][q][c] + red[3][q][c]);
    }
}

// out[3 a + d] += 2 sum_n w_n sum_k gamma_k P_k D_kd (one block per atom; the parts
// of P and D in order, columns in fixed order per thread, then the fixed-order
// block reduction)
__global__ __launch_bounds__(256) void k_force_nl_reduce(const double* __restrict__ pd, int ncol, int parts,
                                                        const double* __restrict__ w, ForceTab tab,
                                                        double* __restrict__ out) {
    const int a = blockIdx.x;
    double acc[3] = {0.0, 0.0, 0.0};
    for (int n = threadIdx.x; n < ncol; n += blockDim.x) {
        double v[16];
#pragma unroll
        for (int q = 0; q < 16; ++q) v[q] = pd[((long)a * ncol + n) * 16 + q];
        for (int p = 1; p < parts; ++p)
#pragma unroll
            for (int q = 0; q < 16; ++q) v[q] += pd[(((long)p * gridDim.x + a) * ncol + n) * 16 + q];
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            const double cpk = 2.0 * tab.gamma4[4 * a + k] * w[n] * v[k];
#pragma unroll
            for (int d = 0; d < 3; ++d) acc[d] += cpk * v[4 + 3 * k + d];
        }
    }
    __shared__ double lds[4][3];
    const double sum = block_reduce<3>(acc, lds);
    if (threadIdx.x < 3) out[3 * a + threadIdx.x] += sum;
}

constexpr int kLocalChunks = 8;

}  // namespace

sparc_status ensure_force_tables(sparc_gpu_ctx c) {
    if (c->force_tab) return SPARC_OK;
    const int n = c->n_atoms;
    std::vector<double> h(9 * (size_t)n, 0.0);
    for (int a = 0; a < n; ++a) {
        for (int d = 0; d < 3; ++d) h[3 * a + d] = c->pos[3 * a + d];
        h[3 * n + a] = c->Z[a];
        h[4 * n + a] = c->rc_loc[a];
        if (c->nl_lmax >= 1) {
            h[5 * n + 4 * a] = c->gamma[2 * a];
            h[5 * n + 4 * a + 1] = h[5 * n + 4 * a + 2] = h[5 * n + 4 * a + 3] = c->gamma[2 * a + 1];
        }
    }
    SG_HIP(c, hipMalloc((void**)&c->force_tab, h.size() * sizeof(double)));
    SG_HIP(c, hipMemcpyAsync(c->force_tab, h.data(), h.size() * sizeof(double), hipMemcpyHostToDevice, c->stream));
    SG_HIP(c, hipStreamSynchronize(c->stream));
    return SPARC_OK;
}

namespace {

// Tiles of a workgroup, chunks of columns and parts of a sphere.  A chip holds 512
// workgroups, and the last ones run on after the others for about 0.6 of their
// time; a part costs 0.03 spheres more than its lines (set-up, the sum over the
// waves).  In one part few atoms or columns leave the chip idle: 4 atoms x 12
// columns 521 and now 209 us with the local part, 46 x 77 600 and 293, 108 x 16 724
// and 328; 108 x 260 fills it unevenly (1302 us in one part, 1124 in 3, 1146 in 4).
struct ForceGrid {
    int tiles, chunks, parts;
};
ForceGrid force_grid(int n_atoms, int ncol) {
    const int tiles = div_up(ncol, 16);
    ForceGrid g;
    g.chunks = div_up(tiles, kForceTiles);
    g.tiles = div_up(tiles, g.chunks);
    g.parts = 1;
    double least = 0;
    for (int p = 1; p <= 16; ++p) {
        const double rounds = (double)n_atoms * g.chunks * p / 512, cost = (rounds + 0.6) / p + 0.03 * rounds;
        if (p == 1 || cost < least) {
            least = cost;
            g.parts = p;
        }
    }
    return g;
}

// Doubles of projections that blocks of up to ncol columns take: fewer columns in
// more parts can take more, and a call must not allocate after a wider one.
size_t force_doubles(int n_atoms, int ncol) {
    size_t most = 0;
    for (int n = std::min(16, ncol);; n = std::min(n + 16, ncol)) {
        most = std::max(most, (size_t)n_atoms * n * 16 * force_grid(n_atoms, n).parts);
        if (n == ncol) return most;
    }
}

template <typename T>
sparc_status nl_force(sparc_gpu_ctx c, const T* X, int ncol, long ldx, const double* w, double* pd, double* out) {
    const ForceTab tab = force_tab(c);
    const double rc = c->rc_nl;
    const double N0 = std::pow(2.0 / (kPi * rc * rc), 0.75);
    const double N1 = (2.0 / rc) * N0;
    const ForceGrid G = force_grid(c->n_atoms, ncol);
    auto go = [&](auto tl) {
        k_force_nl_proj<T, tl()><<<dim3(c->n_atoms, G.chunks, G.parts), 256, 0, c->stream>>>(
            X, ldx, ncol, tab, c->nx, c->ny, c->nz, c->hx, c->hy, c->hz, rc, c->rcut_nl, N0, N1, c->dV, pd);
    };
    switch (G.tiles) {
        case 1: go(std::integral_constant<int, 1>()); break;
        case 2: go(std::integral_constant<int, 2>()); break;
        case 3: go(std::integral_constant<int, 3>()); break;
        case 4: go(std::integral_constant<int, 4>()); break;
        default: go(std::integral_constant<int, kForceTiles>()); break;
    }
    k_force_nl_reduce<<<c->n_atoms, 256, 0, c->stream>>>(pd, ncol, G.parts, w, tab, out);
    SG_CHECK_LAUNCH(c);
    return SPARC_OK;
}

}  // namespace

}  // namespace sg

using namespace sg;

extern "C" {

sparc_status sparc_gpu_forces(sparc_gpu_ctx c, const double* d_phi, sparc_prec prec, const void* const* d_X,
                              int n_blocks, int ncol, long ldx, const double* d_occ, double* d_forces) {
    if (!c) return SPARC_ERR_ARG;
    c->err.clear();
    if (!d_phi || !d_forces) return set_err(c, SPARC_ERR_ARG, "forces: null potential or output");
    if (prec != SPARC_FP64 && prec != SPARC_FP32) return set_err(c, SPARC_ERR_ARG, "forces: bad precision");
    if (n_blocks < 0 || n_blocks > 2) return set_err(c, SPARC_ERR_ARG, "forces: n_blocks must be 0, 1 or 2");
    const bool nl = c->nl_lmax >= 1 && n_blocks > 0;
    if (nl) {
        if (!d_X || !d_occ) return set_err(c, SPARC_ERR_ARG, "forces: null orbital blocks or occupations");
        for (int b = 0; b < n_blocks; ++b)
            if (!d_X[b]) return set_err(c, SPARC_ERR_ARG, "forces: null orbital block");
        if (ncol < 1 || ncol > c->n_states) return set_err(c, SPARC_ERR_ARG, "forces: ncol out of range");
        if (ldx < c->nd) return set_err(c, SPARC_ERR_ARG, "forces: ldx < N_d");
    }
    sparc_status st;
    if ((st = ensure_force_tables(c)) != SPARC_OK) return st;
    const int na = c->n_atoms;
    const size_t need = std::max((size_t)na * kLocalChunks * 3, nl ? force_doubles(na, ncol) : 0);
    if ((st = ensure_red(c, need)) != SPARC_OK) return st;
    const ForceTab tab = force_tab(c);
    int slot = prof_begin(c, PK_FORCE_LOCAL);
    k_force_local<<<dim3(na, kLocalChunks), 256, 0, c->stream>>>(tab, d_phi, c->nx, c->ny, c->nz, c->hx, c->hy,
                                                                  c->hz, c->dV, kLocalChunks, c->red);
    k_force_local_reduce<<<div_up(3 * na, 256), 256, 0, c->stream>>>(c->red, na, kLocalChunks, d_forces);
    const double rmax = 10.0;
    k_force_overlap<<<na, 256, 0, c->stream>>>(tab, na, c->Lx, c->Ly, c->Lz, rmax, (int)std::ceil(rmax / c->Lx) + 1,
                                               (int)std::ceil(rmax / c->Ly) + 1, (int)std::ceil(rmax / c->Lz) + 1,
                                               d_forces);
    SG_CHECK_LAUNCH(c);
    prof_end(c, slot);
    if (nl) {
        slot = prof_begin(c, PK_FORCE_NL);
        for (int b = 0; b < n_blocks; ++b) {
            const double* w = d_occ + (long)b * ncol;
            if (prec == SPARC_FP64)
                st = nl_force<double>(c, (const double*)d_X[b], ncol, ldx, w, c->red, d_forces);
            else
                st = nl_force<float>(c, (const float*)d_X[b], ncol, ldx, w, c->red, d_forces);
            if (st != SPARC_OK) return st;
        }
        prof_end(c, slot);
    }
    return SPARC_OK;
}

}  // extern "C"
