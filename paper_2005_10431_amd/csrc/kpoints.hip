// Bloch-periodic k-points (Sec. 2.1: Bloch-periodic boundary conditions on
// the orbitals along extended directions, Brillouin-zone integration over
// k-points).
//
// Representation: a complex orbital z = u + i v on the home cell is stored as
// one real column [u ; v] of 2 N_d values.  The complex-linear Hermitian H_k
// acts on such columns as the real symmetric operator [[Re H, -Im H],
// [Im H, Re H]]; a block whose span is closed under z -> i z (the columns
// come in pairs [u; v], [-v; u]) is filtered and Rayleigh-Ritz-rotated by the
// real machinery of the Gamma point with every Bloch eigenvalue appearing
// twice.
//
// H_k z = -1/2 Lap_h^k z + V_eff z + sum_I sum_lm gamma_Il chi~_Ilm <chi~_Ilm, z>,
//   Lap_h^k: the stencil with exp(+-i k_d L_d) on neighbours past the faces;
//   chi~_Ilm(x) = sum_s chi_lm(x + sL - R_I) exp(-i k . sL), over the images s.
#include "internal.hpp"

#include <algorithm>
#include <array>

namespace sg {

namespace {

constexpr double kPi = 3.14159265358979323846;

template <typename T>
__global__ void k_copy_block_k(const T* __restrict__ src, T* __restrict__ dst, long rows, int ncol, long ld) {
    const long i = (long)blockIdx.x * blockDim.x + threadIdx.x;
    const int j = blockIdx.y;
    if (i < rows && j < ncol) dst[i + (long)j * ld] = src[i + (long)j * ld];
}

}  // namespace

// Signed nonlocal bounds at k: sum over atoms and lm of min/max(gamma, 0)
// dV ||chi~_lm||^2 (the k-dependent projector norms), cached per k.
sparc_status kp_nl_bounds(sparc_gpu_ctx c, const double* k, double* nl_lo, double* nl_hi) {
    *nl_lo = *nl_hi = 0.0;
    if (c->nl_lmax < 1) return SPARC_OK;
    for (auto& e : c->kp_bound_cache)
        if (e[0] == k[0] && e[1] == k[1] && e[2] == k[2]) {
            *nl_lo = e[3];
            *nl_hi = e[4];
            return SPARC_OK;
        }
    const double h[3] = {c->hx, c->hy, c->hz}, L[3] = {c->Lx, c->Ly, c->Lz};
    const int N[3] = {c->nx, c->ny, c->nz};
    const double rc = c->rc_nl, rcut = c->rcut_nl;
    const double N0 = std::pow(2.0 / (kPi * rc * rc), 0.75), N1 = (2.0 / rc) * N0;
    double lo = 0.0, hi = 0.0;
    for (int a = 0; a < c->n_atoms; ++a) {
        std::vector<std::pair<long, std::array<double, 8>>> pts;
        int l0[3], h0[3];
        for (int d = 0; d < 3; ++d) {
            l0[d] = (int)std::ceil((c->pos[3 * a + d] - rcut) / h[d]);
            h0[d] = (int)std::floor((c->pos[3 * a + d] + rcut) / h[d]);
        }
        for (int kk = l0[2]; kk <= h0[2]; ++kk)
            for (int j = l0[1]; j <= h0[1]; ++j)
                for (int i = l0[0]; i <= h0[0]; ++i) {
                    const int ii[3] = {i, j, kk};
                    double dd[3], r2 = 0.0;
                    for (int d = 0; d < 3; ++d) {
                        dd[d] = ii[d] * h[d] - c->pos[3 * a + d];
                        r2 += dd[d] * dd[d];
                    }
                    if (r2 > rcut * rcut) continue;
                    int s[3], w[3];
                    double th = 0.0;
                    for (int d = 0; d < 3; ++d) {
                        s[d] = ii[d] >= 0 ? ii[d] / N[d] : -((-ii[d] + N[d] - 1) / N[d]);
                        w[d] = ii[d] - s[d] * N[d];
                        th += k[d] * s[d] * L[d];
                    }
                    const double ex = std::exp(-r2 / (rc * rc));
                    const double chi[4] = {N0 * ex, N1 * dd[0] * ex, N1 * dd[1] * ex, N1 * dd[2] * ex};
                    std::array<double, 8> v;
                    for (int l = 0; l < 4; ++l) {
                        v[l] = chi[l] * std::cos(th);
                        v[4 + l] = -chi[l] * std::sin(th);
                    }
                    pts.push_back({w[0] + (long)N[0] * (w[1] + (long)N[1] * w[2]), v});
                }
        std::sort(pts.begin(), pts.end(), [](const auto& x, const auto& y) { return x.first < y.first; });
        double nrm[4] = {0, 0, 0, 0};
        for (size_t b = 0; b < pts.size();) {
            std::array<double, 8> s{};
            size_t e = b;
            for (; e < pts.size() && pts[e].first == pts[b].first; ++e)
                for (int r = 0; r < 8; ++r) s[r] += pts[e].second[r];
            for (int l = 0; l < 4; ++l) nrm[l] += s[l] * s[l] + s[4 + l] * s[4 + l];
            b = e;
        }
        const double g[4] = {c->gamma[2 * a], c->gamma[2 * a + 1], c->gamma[2 * a + 1], c->gamma[2 * a + 1]};
        for (int l = 0; l < 4; ++l) {
            lo += std::min(g[l], 0.0) * c->dV * nrm[l];
            hi += std::max(g[l], 0.0) * c->dV * nrm[l];
        }
    }
    c->kp_bound_cache.push_back({k[0], k[1], k[2], lo, hi});
    *nl_lo = lo;
    *nl_hi = hi;
    return SPARC_OK;
}

template <typename T>
sparc_status bloch_apply_impl(sparc_gpu_ctx c, const T* X, T* Y, int ncol, long ldx) {
    // the projecting pass only reads X; then as at the Gamma point
    sparc_status st = nl_pass_k<T>(c, const_cast<T*>(X), ncol, ldx, NlApply::no, true, 0, 0);
    if (st != SPARC_OK) return st;
    if (nl_writes(c, 2 * ncol, sizeof(T) == 4, true)) {
        if ((st = nl_pass_k<T>(c, Y, ncol, ldx, NlApply::write, false, 0, 0)) != SPARC_OK) return st;
        return launch_hsweep<T>(c, X, Y, Y, 2 * ncol, ldx, 2, 0, true);
    }
    if ((st = launch_hsweep<T>(c, X, Y, nullptr, 2 * ncol, ldx, 0, 0, true)) != SPARC_OK) return st;
    return nl_pass_k<T>(c, Y, ncol, ldx, NlApply::add, false, 0, 0);
}
template sparc_status bloch_apply_impl<double>(sparc_gpu_ctx, const double*, double*, int, long);
template sparc_status bloch_apply_impl<float>(sparc_gpu_ctx, const float*, float*, int, long);

// Filter with bounds in c->scal[S_A..S_A0]: Y_k in X for even k, in W for
// odd k; the result ends in X (the Gamma filter's schedule).
template <typename T>
sparc_status bloch_filter_impl(sparc_gpu_ctx c, T* X, T* W, int ncol, long ldx, int m) {
    sparc_status st;
    if ((st = nl_pass_k<T>(c, X, ncol, ldx, NlApply::no, true, 1, 1)) != SPARC_OK) return st;
    for (int k = 1; k <= m; ++k) {
        T* cur = (k % 2 == 0) ? W : X;
        T* dst = (k % 2 == 0) ? X : W;
        const int mode = k == 1 ? 1 : 2;
        if ((st = launch_hsweep<T>(c, cur, dst, k == 1 ? nullptr : dst, 2 * ncol, ldx, mode, k, true)) != SPARC_OK)
            return st;
        if ((st = nl_pass_k<T>(c, dst, ncol, ldx, NlApply::add, k < m, 2, k + 1)) != SPARC_OK) return st;
    }
    if (m % 2 == 1) {
        k_copy_block_k<T><<<dim3(div_up(2 * c->nd, 256), ncol), 256, 0, c->stream>>>(W, X, 2 * c->nd, ncol, ldx);
        SG_CHECK_LAUNCH(c);
    }
    return SPARC_OK;
}
template sparc_status bloch_filter_impl<double>(sparc_gpu_ctx, double*, double*, int, long, int);
template sparc_status bloch_filter_impl<float>(sparc_gpu_ctx, float*, float*, int, long, int);

// Spectrum bounds of H_k into S_LO / S_HI (V_eff extrema plus the
// k-dependent nonlocal bounds).
sparc_status bloch_bounds_impl(sparc_gpu_ctx c) {
    double lo, hi;
    sparc_status st = kp_nl_bounds(c, c->kvec, &lo, &hi);
    if (st != SPARC_OK) return st;
    // the Gamma routine with the k-dependent nonlocal terms (its kernels take
    // them as launch arguments)
    const double glo = c->nl.nl_lo, ghi = c->nl.nl_hi;
    c->nl.nl_lo = lo;
    c->nl.nl_hi = hi;
    st = bounds_impl(c);
    c->nl.nl_lo = glo;
    c->nl.nl_hi = ghi;
    return st;
}

}  // namespace sg

using namespace sg;

namespace {

__global__ void k_set_params3(double* dst, double a, double b, double c) {
    dst[0] = a;
    dst[1] = b;
    dst[2] = c;
}

sparc_status check_k_block(sparc_gpu_ctx c, const double* k, int prec, const void* X, int ncol, long ldx,
                           const char* who) {
    if (!k || !std::isfinite(k[0]) || !std::isfinite(k[1]) || !std::isfinite(k[2]))
        return set_err(c, SPARC_ERR_ARG, std::string(who) + ": bad k");
    if (prec != SPARC_FP64 && prec != SPARC_FP32) return set_err(c, SPARC_ERR_ARG, std::string(who) + ": bad precision");
    if (!X) return set_err(c, SPARC_ERR_ARG, std::string(who) + ": null block");
    if (ncol < 1 || ncol > 2 * c->n_states)
        return set_err(c, SPARC_ERR_ARG, std::string(who) + ": ncol outside [1, 2 n_states]");
    if (ldx < 2 * c->nd) return set_err(c, SPARC_ERR_ARG, std::string(who) + ": ldx < 2 N_d");
    return SPARC_OK;
}

bool blocks_overlap(const void* a, const void* b, size_t bytes) {
    const char* pa = (const char*)a;
    const char* pb = (const char*)b;
    return pa < pb + bytes && pb < pa + bytes;
}

void set_k(sparc_gpu_ctx c, const double* k) {
    for (int d = 0; d < 3; ++d) c->kvec[d] = k[d];
}

}  // namespace

extern "C" {

sparc_status sparc_gpu_apply_H_k(sparc_gpu_ctx c, const double* k, sparc_prec prec, const void* d_X, void* d_Y,
                                 int ncol, long ldx) {
    if (!c) return SPARC_ERR_ARG;
    c->err.clear();
    sparc_status st = check_k_block(c, k, prec, d_X, ncol, ldx, "apply_H_k");
    if (st != SPARC_OK) return st;
    if (!d_Y) return set_err(c, SPARC_ERR_ARG, "apply_H_k: null output");
    const size_t es = prec == SPARC_FP64 ? 8 : 4;
    if (blocks_overlap(d_X, d_Y, ((size_t)(ncol - 1) * ldx + 2 * c->nd) * es))
        return set_err(c, SPARC_ERR_ARG, "apply_H_k: X and Y overlap");
    set_k(c, k);
    if (prec == SPARC_FP64) return bloch_apply_impl<double>(c, (const double*)d_X, (double*)d_Y, ncol, ldx);
    return bloch_apply_impl<float>(c, (const float*)d_X, (float*)d_Y, ncol, ldx);
}

sparc_status sparc_gpu_chebyshev_filter_k(sparc_gpu_ctx c, const double* k, sparc_prec prec, void* d_X, void* d_work,
                                          int ncol, long ldx, int degree, double a, double b, double a0) {
    if (!c) return SPARC_ERR_ARG;
    c->err.clear();
    sparc_status st = check_k_block(c, k, prec, d_X, ncol, ldx, "chebyshev_filter_k");
    if (st != SPARC_OK) return st;
    if (!d_work) return set_err(c, SPARC_ERR_ARG, "chebyshev_filter_k: null work block");
    if (degree < 1 || degree > 10000) return set_err(c, SPARC_ERR_ARG, "chebyshev_filter_k: degree out of range");
    if (!(a0 < a && a < b) || !std::isfinite(a0) || !std::isfinite(b))
        return set_err(c, SPARC_ERR_ARG, "chebyshev_filter_k: need a0 < a < b");
    const size_t es = prec == SPARC_FP64 ? 8 : 4;
    if (blocks_overlap(d_X, d_work, ((size_t)(ncol - 1) * ldx + 2 * c->nd) * es))
        return set_err(c, SPARC_ERR_ARG, "chebyshev_filter_k: X and work overlap");
    set_k(c, k);
    k_set_params3<<<1, 1, 0, c->stream>>>(c->scal + S_A, a, b, a0);
    SG_CHECK_LAUNCH(c);
    if (prec == SPARC_FP64) return bloch_filter_impl<double>(c, (double*)d_X, (double*)d_work, ncol, ldx, degree);
    return bloch_filter_impl<float>(c, (float*)d_X, (float*)d_work, ncol, ldx, degree);
}

sparc_status sparc_gpu_rayleigh_ritz_k(sparc_gpu_ctx c, const double* k, sparc_prec prec, void* d_X, int ncol,
                                       long ldx, double* d_eig) {
    if (!c) return SPARC_ERR_ARG;
    c->err.clear();
    sparc_status st = check_k_block(c, k, prec, d_X, ncol, ldx, "rayleigh_ritz_k");
    if (st != SPARC_OK) return st;
    if (!d_eig) return set_err(c, SPARC_ERR_ARG, "rayleigh_ritz_k: null eigenvalue output");
    if (ncol > kEighMaxN) return set_err(c, SPARC_ERR_ARG, "rayleigh_ritz_k: ncol above the eigensolver limit");
    set_k(c, k);
    if (prec == SPARC_FP64) return rayleigh_ritz_k_impl<double>(c, (double*)d_X, ncol, ldx, d_eig, true);
    return rayleigh_ritz_k_impl<float>(c, (float*)d_X, ncol, ldx, d_eig, true);
}

sparc_status sparc_gpu_spectrum_bounds_k(sparc_gpu_ctx c, const double* k, double* lo, double* hi) {
    if (!c) return SPARC_ERR_ARG;
    c->err.clear();
    if (!k || !std::isfinite(k[0]) || !std::isfinite(k[1]) || !std::isfinite(k[2]))
        return set_err(c, SPARC_ERR_ARG, "spectrum_bounds_k: bad k");
    set_k(c, k);
    sparc_status st = bloch_bounds_impl(c);
    if (st != SPARC_OK) return st;
    double h2[2];
    SG_HIP(c, hipMemcpyAsync(h2, c->scal + S_LO, 2 * sizeof(double), hipMemcpyDeviceToHost, c->stream));
    SG_HIP(c, hipStreamSynchronize(c->stream));
    if (lo) *lo = h2[0];
    if (hi) *hi = h2[1];
    return SPARC_OK;
}

}  // extern "C"
