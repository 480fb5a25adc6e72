// Internal declarations of the MI355X CheFSI library (not part of the ABI).
#pragma once

#include <hip/hip_runtime.h>

#include <array>
#include <cstdint>
#include <string>
#include <vector>

#include "sparc_gpu.h"

namespace sg {

constexpr int kMaxHalfOrder = 6;  // stencil half-width instantiated in the kernels

// Finite-difference coefficients of H's kinetic part -1/2 Delta_h along each
// axis: c*[q] multiplies f(p + q e_d) + f(p - q e_d); c0 multiplies f(p).
template <typename T>
struct StencilCoef {
    T cx[kMaxHalfOrder + 1];
    T cy[kMaxHalfOrder + 1];
    T cz[kMaxHalfOrder + 1];
    T c0;
};

// An (atom, periodic image) pair of the projector supports: grid point
// (x, y, z) of the home cell lies at ((x + bx) hx - px, ...) from the image's
// centre; id: its place in the pair table, where an atom's pairs are consecutive.
struct NlCand {
    double px, py, pz;
    int bx, by, bz;
    int atom, id;
};

// One line of a pair's support: n points from (x0, y, z) along x.
struct NlSeg {
    int cand, x0, y, z, n;
};

constexpr int kNlBlocks = 6;   // 16-point blocks of a pencil of the nonlocal pass

// A pencil of nb blocks over planes [zb, ze); its pairs are entries ebase .. ebase + ncl - 1
struct NlUnit {
    int zb, ze, pencil, nb, ebase, ncl;
};

// Tables of the nonlocal pass (nonlocal.hip).  NlRanges: the units and slots for
// one cut of z into ranges.
struct NlRanges {
    NlUnit* units = nullptr;
    uint8_t* occ = nullptr;      // per unit zlen x slots: the unit's pair in each slot (255: none)
    uint64_t* gm = nullptr;      // per unit zlen: slot groups that meet each block
    int* ent_cand = nullptr;     // pair of every entry
    int* red_off = nullptr;      // entries of each atom
    int* red_ent = nullptr;
    int zlen = 1, ncl = 1;
    long n_entries = 0;
    bool whole = false;          // one layer, whose units hold every point of the grid
    std::vector<int> layer_off;  // unit ranges of the layers
};
struct NlPass {
    int* blk = nullptr;          // first points of the kNlBlocks blocks of each pencil, -1 pads
    void* dummy = nullptr;       // 256 doubles: target of the stores of pads
    double* zero = nullptr;      // 4 coefficients of a slot without a pair; alpha of the step that will apply D
    NlCand* cand = nullptr;
    uint32_t* odd = nullptr;     // per 16 columns: epoch of the last projection that was not finite
    uint32_t epoch = 0;          // projections formed so far (the one that an apply takes is the last)
    int* cand_off = nullptr;     // pairs of each atom
    int n_cand = 0, npen = 0, slots = 8;
    std::vector<NlRanges> ranges;   // the first is made for the context's full block
    std::vector<size_t> part_upto;  // doubles of partial sums that blocks of up to n columns take
};

// Shape of a sweep over ncol columns (see sweep_plan)
struct SweepPlan {
    int ncol = 0, forced = 0;        // what it was made for
    int vx = 0, ty = 0;              // points per thread, rows of a slab
    int threads = 0;                 // of a workgroup
    size_t lds = 0;
    int round = 1, split = 1;        // workgroups an XCD holds, z ranges past its last full round
};

// Nonlocal projector tables on the device.
//  - spectral bound: projector values per unique support point (sup_*).
struct NonlocalTables {
    int n_atoms = 0;
    long n_sup = 0;
    long* sup_off = nullptr;   // n_atoms + 1: each atom's unique support points
    double* sup_chi = nullptr; // 4 n_sup projector values (summed over images; for the spectral bound)
    double* gamma4 = nullptr;  // 4 n_atoms: (g_s, g_p, g_p, g_p)
    double nl_hi = 0.0, nl_lo = 0.0;  // signed spectral bound contributions
    int max_per_atom = 0;
};

}  // namespace sg

struct sparc_gpu_ctx_s {
    // geometry
    int nx = 0, ny = 0, nz = 0;
    long nd = 0;
    double hx = 0, hy = 0, hz = 0, dV = 0;
    double Lx = 0, Ly = 0, Lz = 0;
    int n_o = 6;
    double w[sg::kMaxHalfOrder + 1] = {0};
    sg::StencilCoef<double> cf64;
    sg::StencilCoef<float> cf32;
    double kin_bound = 0;    // upper bound of -1/2 Delta_h

    // atoms
    int n_atoms = 0;
    std::vector<double> pos, Z, rc_loc, gamma;
    int nl_lmax = -1;
    double rc_nl = 0, rcut_nl = 0;
    int n_states = 0;
    double n_electrons = 0, kT = 0, rho_floor = 1e-14, sad_width = 1.0;

    hipStream_t stream = nullptr;
    hipDeviceProp_t prop;

    // device fields
    double* veff = nullptr;     // N_d
    float* veff32 = nullptr;    // N_d
    double* veff_spin = nullptr;  // 2 N_d: V_eff of both spins (spin-polarised SCF, allocated on use)
    double* force_tab = nullptr;  // per-atom force table: pos (3n), Z (n), rc (n), gamma (4n); on use
    // Bloch k-points (allocated on use)
    double kvec[3] = {0, 0, 0};   // current k (1/Bohr)
    double* kp_phase = nullptr;   // per (atom, image) pair: cos, sin of k . sL at kp_phase_k
    double kp_phase_k[3] = {0, 0, 0};
    int kp_phase_valid = 0;
    double* kp_D = nullptr;       // per half column and (atom, image) pair: 4 coefficients
    size_t kp_D_elems = 0;
    double* kp_bounds = nullptr;  // 3 per k-point: filter bounds of the k-point SCF
    int kp_bounds_n = 0;
    double* kp_wts = nullptr;     // per-state k weights of the k-point SCF
    int kp_wts_n = 0;
    std::vector<std::array<double, 5>> kp_bound_cache;  // (k, nonlocal lo, hi)
    double* b = nullptr;        // pseudocharge, N_d
    double e_self = 0, e_c = 0;
    sg::NonlocalTables nl;
    sg::NlPass nlp;
    sg::SweepPlan sweep_plans[4];   // FP32, FP64, their Bloch forms: of the last block width

    // Poisson: real orthonormal Fourier bases per axis and the operator's
    // eigenvalues on the product basis
    double* pois_ux = nullptr;  // nx*nx
    double* pois_uy = nullptr;
    double* pois_uz = nullptr;
    double* pois_inv = nullptr; // N_d: 4 pi / eigenvalue of -Delta_h (0 for k = 0)

    // workspace (lazily sized)
    void* work = nullptr;       // one block of n_states columns (bytes below)
    size_t work_bytes = 0;
    double* D = nullptr;        // projector coefficients: 4 n_atoms x n_states
    double* nl_part = nullptr;  // projection partials per (entry, column)
    double* scratch = nullptr;  // this device's fixed scratch array (allocation-free filter)
    size_t scratch_elems = 0;
    size_t nl_part_elems = 0;
    float* D32 = nullptr;
    double* gemm_part = nullptr; // split-K partials
    size_t gemm_part_elems = 0;
    double* small = nullptr;    // dense subspace matrices
    size_t small_elems = 0;
    double* red = nullptr;      // reduction partials
    size_t red_elems = 0;
    double* scal = nullptr;     // device scalars (filter params, mu, ...)
    int* flags = nullptr;       // device status flags
    double* field = nullptr;    // grid scratch fields (several N_d)
    int n_field = 0;

    hipEvent_t ev[8];
    std::vector<hipEvent_t> step_ev;  // events of one SCF call, read after its single synchronisation
    double* h_scal = nullptr;   // pinned host mirror of scal (S_COUNT), filled by the SCF calls
    int* h_flags = nullptr;     // pinned host mirror of flags (F_COUNT)
    std::string err;

    // captured Jacobi sweep (see dense.hip)
    hipStream_t cap_stream = nullptr;
    int sweep_group = 4;        // SPARC_GPU_SWEEP_GROUP: orbitals whose copies of a slab run side by side
    int gemm_tile = 0;          // SPARC_GPU_GEMM_TILE: FP64 Gram tiles above 64 columns (128, 160; 0: by size)
    int cnn_tz = 8;             // SPARC_GPU_CNN_TZ: depth of the matrix-core 16 -> 16 convolution tile (4, 8; 0: vector kernel)
    int cnn_per_cu[2][2] = {};  // resident convolution workgroups per CU, by (tile depth 8, MODE)
    hipGraphExec_t jac_exec = nullptr;
    int jac_N = 0;
    double *jac_A = nullptr, *jac_A2 = nullptr, *jac_V = nullptr, *jac_V2 = nullptr;
    int debug = 0;              // SPARC_GPU_DEBUG: diagnostics on stderr
    int eig_jacobi = 0;         // SPARC_GPU_EIG=jacobi: parallel Jacobi instead of tridiagonal
    int trd_multi_min = 320;    // SPARC_GPU_TRD_MULTI_MIN: N from which the reduction uses many workgroups
    int trd_tail = 256;         // SPARC_GPU_TRD_TAIL: trailing size below which one workgroup finishes it
    int stein_lds_min_tpw = 3;  // SPARC_GPU_STEIN_LDS_MIN_TPW: fewest solves per workgroup for the LDS inverse iteration
    int chol_multi_min = 384;   // SPARC_GPU_CHOL_MULTI_MIN: N from which Cholesky updates over many workgroups
    double* chol_dorig = nullptr;  // original diagonal for the many-workgroup Cholesky (kEighMaxN)
    double* atom_pos = nullptr;    // 3 n_atoms

    // kernel timing (sparc_gpu_profile)
    bool prof = false;
    std::vector<hipEvent_t> prof_pool;        // 2 events per recorded launch
    std::vector<int> prof_kernel;             // kernel id per recorded launch
    int prof_used = 0;
    double prof_ms[32] = {0};   // indexed by sg::ProfKernel
    long prof_n[32] = {0};
};

namespace sg {

// ---- error handling -----------------------------------------------------
sparc_status set_err(sparc_gpu_ctx c, sparc_status s, const std::string& msg);
sparc_status hip_err(sparc_gpu_ctx c, hipError_t e, const char* what);

#define SG_HIP(ctx, call)                                             \
    do {                                                              \
        hipError_t _e = (call);                                       \
        if (_e != hipSuccess) return ::sg::hip_err((ctx), _e, #call); \
    } while (0)

#define SG_CHECK_LAUNCH(ctx) SG_HIP(ctx, hipGetLastError())

// ---- workspace ----------------------------------------------------------
sparc_status ensure_work(sparc_gpu_ctx c, size_t bytes);
sparc_status ensure_gemm_part(sparc_gpu_ctx c, size_t elems);
sparc_status ensure_small(sparc_gpu_ctx c, size_t elems);
sparc_status ensure_red(sparc_gpu_ctx c, size_t elems);
sparc_status ensure_fields(sparc_gpu_ctx c, int n);

// Device scalar slots in ctx->scal
enum Scalar {
    S_A = 0, S_B = 1, S_A0 = 2,      // filter bounds
    S_LO = 4, S_HI = 5,              // spectrum bounds of the current H
    S_RED0 = 8,                      // grid reductions (6 slots)
    S_OCC = 16,                      // mu, entropy term, band energy
    S_EIG = 22,                      // eigensolver norms (2 slots)
    S_CNN = 32,                      // warm-start network head sums (6 slots)
    S_PULAY = 40,                    // Pulay weights gamma (SPARC_PULAY_MAX slots)
    S_SPINB = 50,                    // filter bounds a, b, a0 of both spins (6 slots)
    S_COUNT = 64
};
enum Flag {
    F_NOT_SPD = 0, F_EIG_NOCONV = 1, F_FERMI = 2, F_NONFINITE = 3, F_JACOBI_DONE = 4, F_PULAY_SINGULAR = 5,
    F_INPUT_NONFINITE = 6,   // a non-finite value in an SCF call's input density
    F_COUNT = 16
};

// ---- kernels (launchers) -------------------------------------------------
// Local part of H / Chebyshev sweeps. mode: 0 out = H_loc x; 1 first filter
// step; 2 filter step `step` (>= 2) with xprev = X_{k-1} (may alias out), and with
// step 0 out = H_loc x + xprev.
// halves: column j is half j % 2 (N_d rows) of Bloch column j / 2, at the
// context's k.
template <typename T>
sparc_status launch_hsweep(sparc_gpu_ctx c, const T* x, T* out, const T* xprev, int ncol, long ldx,
                           int mode, int step, bool halves = false);
// The nonlocal term of a block in one pass: apply (add: y += chi D; write: y = chi D,
// only where nl_writes says so) and / or project (D = alpha gamma dV chi^T y of the
// completed y, alpha that of the filter step (mode, step) that will apply it, 1
// for mode 0).  The partial sums go to `part` (part_elems doubles, as many columns
// at a time as fit) when given, else to context memory sized for the whole block.
// Does nothing without projectors.
enum class NlApply { no, add, write };
template <typename T>
sparc_status nl_pass(sparc_gpu_ctx c, T* y, int ncol, long ldx, NlApply apply, bool project, int mode, int step,
                     double* part = nullptr, size_t part_elems = 0);
// Whether H X had better let the pass over ncol real columns (halves of Bloch
// columns) write y before the sweep adds to it: it has projectors, whose units
// hold every point, and the shape is right.
bool nl_writes(sparc_gpu_ctx c, int ncol, bool fp32, bool bloch);
// The pass for ncol Bloch columns [u; v] at the context's k, in FP64 arithmetic
// for both block precisions.
template <typename T>
sparc_status nl_pass_k(sparc_gpu_ctx c, T* y, int ncol, long ldx, NlApply apply, bool project, int mode, int step);
// Y = H X
template <typename T>
sparc_status apply_impl(sparc_gpu_ctx c, const T* X, T* Y, int ncol, long ldx);
// Chebyshev filter of degree m on X (Wk: scratch block); projection partials
// as in nl_pass.
template <typename T>
sparc_status filter_impl(sparc_gpu_ctx c, T* X, T* Wk, int ncol, long ldx, int m, double* part = nullptr,
                         size_t part_elems = 0);
// Filter coefficients of step k of the scaled recurrence:
//   e = (b-a)/2, c = (b+a)/2, sigma_1 = e/(a0-c), tau = 2/sigma_1,
//   sigma_k = 1/(tau - sigma_{k-1});
//   step 1: out = (sigma_1/e)(Hx - c x)
//   step k: out = (2 sigma_k/e)(Hx - c x) - sigma_{k-1} sigma_k xprev
// and of mode 2, step 0: out = Hx + xprev.
__device__ inline void filter_coefs(const double* params, int mode, int step, double& alpha, double& cshift,
                                    double& beta) {
    alpha = 1.0;
    cshift = 0.0;
    beta = 0.0;
    if (mode == 2 && step == 0) beta = 1.0;
    if (mode == 0 || step == 0) return;
    double A = params[0], B = params[1], A0 = params[2];
    double e = 0.5 * (B - A), c = 0.5 * (B + A);
    double s1 = e / (A0 - c);
    cshift = c;
    if (mode == 1) {
        alpha = s1 / e;
        return;
    }
    double tau = 2.0 / s1;
    double sp = s1, s = s1;
    for (int k = 2; k <= step; ++k) {
        sp = s;
        s = 1.0 / (tau - s);
    }
    alpha = 2.0 * s / e;
    beta = -sp * s;
}

// C(MxN, col-major, ldc) = alpha * A^T B, A: K x M (lda), B: K x N (ldb),
// T inputs, double output, deterministic split-K.
template <typename T>
sparc_status gemm_tn(sparc_gpu_ctx c, int M, int N, long K, const T* A, long lda, const T* B, long ldb,
                     double alpha, double* C, int ldc, bool symmetric);
// Out(K x N, ldo) = A (K x M, lda) * Bm (M x N, ldb; double, converted to T)
template <typename T>
sparc_status gemm_nn(sparc_gpu_ctx c, long K, int N, int M, const T* A, long lda, const double* Bm, int ldb,
                     T* Out, long ldo);

// Dense subspace algebra (FP64, N x N col-major)
sparc_status dense_cholesky(sparc_gpu_ctx c, double* M, int N, int* flag);
sparc_status dense_tri_inverse_lower(sparc_gpu_ctx c, const double* L, double* Linv, int N);
sparc_status dense_gemm(sparc_gpu_ctx c, char ta, char tb, int N, const double* A, const double* B, double* C);
sparc_status dense_symmetrize(sparc_gpu_ctx c, double* A, int N);
sparc_status dense_eigh(sparc_gpu_ctx c, double* A, int N, double* V, double* eig, double* work);
sparc_status dense_eigh_tridiag(sparc_gpu_ctx c, double* A, int N, double* V, double* eig, double* work);
constexpr int kEighMaxN = 4096;
inline size_t eigh_work_doubles(int N) { return 6 * (size_t)N * N + 320 * (size_t)N + 64; }

// RR core shared by the public entry point and the SCF step; eig on device.
// check: synchronise after the Cholesky factor and return SPARC_ERR_NOT_SPD
// with X unchanged on a non-SPD Gram matrix (the public call); without it the
// flag F_NOT_SPD stays set on the device for the caller's one final read and
// the rest of the step runs on (bounded loops only).
template <typename T>
sparc_status rayleigh_ritz_impl(sparc_gpu_ctx c, T* X, int ncol, long ldx, double* d_eig, bool check);

// Grid-field kernels
sparc_status potential_impl(sparc_gpu_ctx c, const double* rho, double* phi, double* exc, double* vxc,
                            double* veff);
// deg: electrons per state (2 spin-unpolarised, 1 per spin state); wts:
// optional per-state weights (k-point weights), null for 1
sparc_status occupations_impl(sparc_gpu_ctx c, const double* eig, int ncol, double* occ, double* mu,
                              double deg = 2.0, const double* wts = nullptr);
template <typename T>
sparc_status density_impl(sparc_gpu_ctx c, const T* X, int ncol, long ldx, const double* occ, double* rho);
sparc_status set_veff_impl(sparc_gpu_ctx c, const double* d_veff);
sparc_status bounds_impl(sparc_gpu_ctx c);  // writes S_LO / S_HI on device
sparc_status ensure_force_tables(sparc_gpu_ctx c);
// Bloch k-points at c->kvec; blocks hold columns [Re z; Im z] of 2 N_d rows
sparc_status kp_nl_bounds(sparc_gpu_ctx c, const double* k, double* nl_lo, double* nl_hi);
sparc_status bloch_bounds_impl(sparc_gpu_ctx c);
template <typename T>
sparc_status bloch_apply_impl(sparc_gpu_ctx c, const T* X, T* Y, int ncol, long ldx);
template <typename T>
sparc_status bloch_filter_impl(sparc_gpu_ctx c, T* X, T* W, int ncol, long ldx, int m);
template <typename T>
sparc_status rayleigh_ritz_k_impl(sparc_gpu_ctx c, T* X, int ncol, long ldx, double* d_eig, bool check);

// Kernel timing: prof_begin returns a slot (or -1 when disabled), prof_end
// records its closing event.
enum ProfKernel {
    PK_SWEEP = 0,    // filter step k >= 2 (reads X_k, X_{k-1}; writes X_{k+1})
    PK_PROJ = 1,     // projections (streaming pass and per-atom sum)
    PK_GEMM_TN = 2,
    PK_GEMM_NN = 3,
    PK_DENSITY = 4,
    PK_SWEEP1 = 5,   // first filter step
    PK_APPLY = 6,    // plain H application
    PK_CHOL = 7,     // Cholesky of the Gram matrix
    PK_TRINV = 8,    // inverse of the Cholesky factor
    PK_EIG = 9,      // subspace eigensolver (all its launches)
    PK_SMALL = 10,   // N_s x N_s products
    PK_COPY = 11,    // block copies
    PK_EIG_TRD = 12, // eigensolver: tridiagonalisation
    PK_EIG_BIS = 13, // eigensolver: eigenvalues of the tridiagonal matrix
    PK_EIG_VEC = 14, // eigensolver: inverse iteration
    PK_EIG_BACK = 15,// eigensolver: back-transformation
    PK_CNN_FWD = 16, // warm-start network forward (all launches)
    PK_CNN_CONV2 = 17,  // its 16 -> 16 convolution
    PK_CNN_BWD = 18, // network gradient (all launches)
    PK_MIX = 19,     // density mixing step (all launches of one step)
    PK_FORCE_LOCAL = 20,  // local and overlap forces
    PK_FORCE_NL = 21,     // nonlocal forces (all orbital blocks)
    PK_BLOCH = 22,        // Bloch H_k application / filter step
    PK_BLOCH_PROJ = 23,   // Bloch projections
    PK_COUNT = 32    // size of the per-context timing tables
};
static_assert(PK_COUNT == sizeof(sparc_gpu_ctx_s::prof_n) / sizeof(long), "timing table size");
int prof_begin(sparc_gpu_ctx c, int kernel, hipStream_t s = nullptr);  // s = null: the context stream
void prof_end(sparc_gpu_ctx c, int slot, hipStream_t s = nullptr);

// Build geometry tables (ctx.hip)
sparc_status build_tables(sparc_gpu_ctx c);
sparc_status build_nl_pass(sparc_gpu_ctx c, const std::vector<NlCand>& cands, const std::vector<NlSeg>& segs);
void free_nl_pass(NlPass& T);
// Device address of the fixed scratch array on device `dev` (current),
// looked up once per device and kept in the context.
sparc_status scratch_init(sparc_gpu_ctx c, int dev);

inline int div_up(long a, long b) { return (int)((a + b - 1) / b); }

}  // namespace sg
