// Dense subspace products of Rayleigh-Ritz on MFMA (the Gram matrix
// dV Y^T Y, the projected Hamiltonian dV Y^T (H Y) and the rotation Y T).
//
// gemm_tn: C = alpha A^T B for tall-skinny A (K x M), B (K x N), K = N_d.
//   Deterministic split-K: each wave reduces one K-chunk of one tile (FP64
//   MFMA for double; FP32 MFMA with FP32 accumulation inside the chunk for
//   float) and writes a double partial; a second kernel sums the partials in
//   a fixed order in double.
// gemm_nn: Out = A Bm with A tall (K x M), Bm small (M x N, double, rounded
//   to the block precision).
//
// gemm_nn and the FP32 and narrow forms of gemm_tn take their operands from L2
// straight into registers, without LDS and without barriers: a 16x16x4 MFMA lasts 64 cycles in FP64 (32 in FP32), so a
// tile of 4 x 4 of them asks for 16 bytes per cycle and compute unit, a quarter
// of what the L1 delivers, and a wave that waits for nobody keeps its matrix
// core busy through the loads two steps ahead.  (Staged through LDS, with a
// barrier per 16 rows, the cores were busy for 76% of the time.)
//
// Of 4 V contraction rows a lane holds the V consecutive ones of its group
// lane / 16 (16 bytes), and the MFMAs take one of them each.  Which rows one MFMA
// sums does not matter as long as both operands agree.
#include "internal.hpp"
#include "mfma.hpp"

namespace sg {

template <typename T, int N>
struct GemmVec {
    typedef T type __attribute__((ext_vector_type(N), aligned(sizeof(T))));
};

// Partial[split][n][m] = sum_{k in chunk} A[k, m] B[k, n] for one tile of
// MT x NT strips of 16 columns.  A, B are K x M / K x N column-major.
//
// A step takes whole 128-byte lines of every column (of half lines the other half
// was often gone from the L1 at the next step: 40.0 instead of 38.3 ms at 1.73M x
// 1200 x 1200 FP32; through LDS 45.8).  One wave per (active tile, split); only
// tiles with a strip pair sn >= sm are active when `symmetric`, and such a tile
// skips its other pairs.  Hardware dispatches block b to XCD b % 8.  When nsplit
// is a multiple of 8, every tile of one split runs on one XCD, and its tiles are
// dispatched together, so that they can share the panels of that K-chunk in the
// XCD's L2.
template <typename T, int MT, int NT, int RING>
__global__ __launch_bounds__(64, 2) void k_gemm_tn_split(int M, int N, long K, long kchunk, const T* __restrict__ A,
                                                         long lda, const T* __restrict__ B, long ldb,
                                                         double* __restrict__ part, int tiles_m, bool symmetric,
                                                         int active, int nsplit) {
    using acc_t = typename Mfma<T>::acc_t;
    constexpr int V = 16 / sizeof(T), H = 2, KS = 4 * V * H;   // rows of a vector; vectors and rows of a step
    using vec = typename GemmVec<T, V>::type;
    const int bid = blockIdx.x;
    int split, tidx;
    if (nsplit % 8 == 0) {
        const int slot = bid / 8;
        split = bid % 8 + 8 * (slot / active);
        tidx = slot % active;
    } else {
        split = bid / active;
        tidx = bid % active;
    }
    int tm = tidx % tiles_m, tn = tidx / tiles_m;
    if (symmetric) {
        // column by column the tiles down to the diagonal
        tm = tidx;
        for (tn = 0;; ++tn) {
            const int col = min(tiles_m, (tn * NT + NT - 1) / MT + 1);
            if (tm < col) break;
            tm -= col;
        }
    }
    const int sm = tm * MT, sn = tn * NT;   // first strips
    const int mi = min(MT, (M + 15) / 16 - sm), nj = min(NT, (N + 15) / 16 - sn);
    const long k0 = (long)split * kchunk;
    const long k1 = min(K, k0 + kchunk);
    const long nst = k1 > k0 ? (k1 - k0) / KS : 0;   // whole steps
    const int lane = threadIdx.x, li = lane & 15, g = lane >> 4;
    // columns past the last repeat it; their sums are not stored
    const T* pa[MT];
    const T* pb[NT];
#pragma unroll
    for (int i = 0; i < MT; ++i) pa[i] = A + (long)min(M - 1, 16 * (sm + min(i, mi - 1)) + li) * lda + k0 + V * g;
#pragma unroll
    for (int j = 0; j < NT; ++j) pb[j] = B + (long)min(N - 1, 16 * (sn + min(j, nj - 1)) + li) * ldb + k0 + V * g;
    acc_t acc[MT][NT];
#pragma unroll
    for (int i = 0; i < MT; ++i)
#pragma unroll
        for (int j = 0; j < NT; ++j) acc[i][j] = acc_t{0, 0, 0, 0};
    auto products = [&](const vec (&va)[H][MT], const vec (&vb)[H][NT], bool all) __attribute__((always_inline)) {
#pragma unroll
        for (int u = 0; u < H * V; ++u)
#pragma unroll
            for (int i = 0; i < MT; ++i)
#pragma unroll
                for (int j = 0; j < NT; ++j)
                    if (all || (i < mi && j < nj && !(symmetric && sm + i > sn + j)))
                        acc[i][j] = Mfma<T>::run(va[u / V][i][u % V], vb[u / V][j][u % V], acc[i][j]);
    };
    if (nst > 0) {
        vec qa[RING][H][MT], qb[RING][H][NT];
        auto load = [&](int r, long s) __attribute__((always_inline)) {
            const long o = min(s, nst - 1) * KS;
#pragma unroll
            for (int i = 0; i < MT; ++i)
#pragma unroll
                for (int h = 0; h < H; ++h) qa[r][h][i] = *reinterpret_cast<const vec*>(pa[i] + o + 4 * V * h);
#pragma unroll
            for (int j = 0; j < NT; ++j)
#pragma unroll
                for (int h = 0; h < H; ++h) qb[r][h][j] = *reinterpret_cast<const vec*>(pb[j] + o + 4 * V * h);
        };
#pragma unroll
        for (int r = 0; r < RING - 1; ++r) load(r, r);
        auto run = [&](bool all) __attribute__((always_inline)) {
            for (long s = 0; s < nst; s += RING) {
#pragma unroll
                for (int r = 0; r < RING; ++r) {
                    if (s + r >= nst) break;
                    load((r + RING - 1) % RING, s + r + RING - 1);
                    products(qa[r], qb[r], all);
                }
            }
        };
        if (mi == MT && nj == NT && !(symmetric && sm + MT - 1 > sn)) run(true);
        else run(false);
    }
    if (k1 - k0 > nst * KS) {
        // the rows past the last whole step, zero past the end
        vec va[H][MT], vb[H][NT];
#pragma unroll
        for (int h = 0; h < H; ++h)
#pragma unroll
            for (int u = 0; u < V; ++u) {
                const long o = nst * KS + 4 * V * h + u;
                const bool in = k0 + o + V * g < k1;
#pragma unroll
                for (int i = 0; i < MT; ++i) va[h][i][u] = in ? pa[i][o] : (T)0;
#pragma unroll
                for (int j = 0; j < NT; ++j) vb[h][j][u] = in ? pb[j][o] : (T)0;
            }
        products(va, vb, false);
    }
    double* P = part + (long)split * M * N;
#pragma unroll
    for (int i = 0; i < MT; ++i)
#pragma unroll
        for (int j = 0; j < NT; ++j)
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                const int m = 16 * (sm + i) + Mfma<T>::row(lane, r);
                const int n = 16 * (sn + j) + li;
                if (m < M && n < N && !(symmetric && sm + i > sn + j)) P[m + (long)n * M] = (double)acc[i][j][r];
            }
}

// The same for FP64 blocks of more than 32 columns: a workgroup of 2 x 2 waves
// takes 2 MT x 2 MT strips and stages their rows through LDS, 16 at a time in two
// buffers (the next rows' loads are issued before this stage's MFMAs and written
// to the other buffer after them: one barrier per stage).  Straight from L2 as
// above, 64 x 64 tiles drift apart and read the block from memory over and over
// (1.73M x 1200 x 1200: 450 GB of L2 misses, 68 ms).  A wave skips the strips past
// the last column and, `symmetric`, those below the diagonal: 47 ms; without that,
// and with 8 splits, which left 14% of the workgroup slots empty, 67.
constexpr int kTnRows = 16;
template <int MT>
__global__ __launch_bounds__(256) void k_gemm_tn_lds(int M, int N, long K, long kchunk, const double* __restrict__ A,
                                                     long lda, const double* __restrict__ B, long ldb,
                                                     double* __restrict__ part, int tiles_m, bool symmetric,
                                                     int active, int nsplit) {
    using acc_t = typename Mfma<double>::acc_t;
    using vec = typename GemmVec<double, 2>::type;
    constexpr int BK = kTnRows, LD = 32 * MT + 2;
    __shared__ double sA[2][BK * LD];
    __shared__ double sB[2][BK * LD];
    const int bid = blockIdx.x;
    int split, tidx;
    if (nsplit % 8 == 0) {
        const int slot = bid / 8;
        split = bid % 8 + 8 * (slot / active);
        tidx = slot % active;
    } else {
        split = bid / active;
        tidx = bid % active;
    }
    int tm = tidx % tiles_m, tn = tidx / tiles_m;
    if (symmetric) {
        // tidx-th upper tile, column by column: (0,0), (0,1), (1,1), (0,2), ...
        tn = 0;
        while ((tn + 1) * (tn + 2) / 2 <= tidx) ++tn;
        tm = tidx - tn * (tn + 1) / 2;
    }
    const long k0 = (long)split * kchunk, k1 = min(K, k0 + kchunk);
    const int t = threadIdx.x, lane = t & 63, wv = t >> 6, li = lane & 15, g = lane >> 4;
    const int wr = (wv & 1) * MT, wc = (wv >> 1) * MT;      // first strips of the wave in the tile
    const int sm = tm * 2 * MT + wr, sn = tn * 2 * MT + wc;
    const int mi = min(MT, (M + 15) / 16 - sm), nj = min(MT, (N + 15) / 16 - sn);
    const bool all = mi == MT && nj == MT && !(symmetric && sm + MT - 1 > sn);
    acc_t acc[MT][MT];
#pragma unroll
    for (int i = 0; i < MT; ++i)
#pragma unroll
        for (int j = 0; j < MT; ++j) acc[i][j] = acc_t{0, 0, 0, 0};
    // loader: thread t reads rows 2 (t % 8) + {0, 1} of columns t / 8 + 32 p, the
    // last column again past it (its sums are not stored)
    const int lk = 2 * (t & 7), lc = t >> 3;
    const double* pa[MT];
    const double* pb[MT];
#pragma unroll
    for (int p = 0; p < MT; ++p) {
        pa[p] = A + (long)min(M - 1, 32 * MT * tm + lc + 32 * p) * lda + k0 + lk;
        pb[p] = B + (long)min(N - 1, 32 * MT * tn + lc + 32 * p) * ldb + k0 + lk;
    }
    vec ra[MT], rb[MT];
    auto load = [&](long o) __attribute__((always_inline)) {
        if (k0 + o + BK <= k1) {
#pragma unroll
            for (int p = 0; p < MT; ++p) ra[p] = *reinterpret_cast<const vec*>(pa[p] + o);
#pragma unroll
            for (int p = 0; p < MT; ++p) rb[p] = *reinterpret_cast<const vec*>(pb[p] + o);
        } else {
            // the last rows, zero past the end
#pragma unroll
            for (int u = 0; u < 2; ++u) {
                const bool in = k0 + o + lk + u < k1;
#pragma unroll
                for (int p = 0; p < MT; ++p) ra[p][u] = in ? pa[p][o + u] : 0.0;
#pragma unroll
                for (int p = 0; p < MT; ++p) rb[p][u] = in ? pb[p][o + u] : 0.0;
            }
        }
    };
    auto store = [&](int buf) __attribute__((always_inline)) {
#pragma unroll
        for (int p = 0; p < MT; ++p)
#pragma unroll
            for (int u = 0; u < 2; ++u) {
                sA[buf][(lk + u) * LD + lc + 32 * p] = ra[p][u];
                sB[buf][(lk + u) * LD + lc + 32 * p] = rb[p][u];
            }
    };
    auto products = [&](int buf, bool whole) __attribute__((always_inline)) {
#pragma unroll
        for (int kk = 0; kk < BK; kk += 4) {
            double av[MT], bv[MT];
#pragma unroll
            for (int i = 0; i < MT; ++i) av[i] = sA[buf][(kk + g) * LD + 16 * (wr + i) + li];
#pragma unroll
            for (int j = 0; j < MT; ++j) bv[j] = sB[buf][(kk + g) * LD + 16 * (wc + j) + li];
#pragma unroll
            for (int i = 0; i < MT; ++i)
#pragma unroll
                for (int j = 0; j < MT; ++j)
                    if (whole || (i < mi && j < nj && !(symmetric && sm + i > sn + j)))
                        acc[i][j] = Mfma<double>::run(av[i], bv[j], acc[i][j]);
        }
    };
    const long nst = k1 > k0 ? (k1 - k0 + BK - 1) / BK : 0;
    if (nst > 0) {
        load(0);
        store(0);
    }
    __syncthreads();
    for (long s = 0; s < nst; ++s) {
        const int buf = (int)(s & 1);
        if (s + 1 < nst) load((s + 1) * BK);
        if (all) products(buf, true);
        else if (mi > 0 && nj > 0) products(buf, false);
        if (s + 1 < nst) store(buf ^ 1);
        __syncthreads();
    }
    // the tile's partial: TT x TT, of active tiles only
    constexpr int TT = 32 * MT;
    double* P = part + ((long)split * active + tidx) * TT * TT;
#pragma unroll
    for (int i = 0; i < MT; ++i)
#pragma unroll
        for (int j = 0; j < MT; ++j)
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                const int m = 16 * (sm + i) + Mfma<double>::row(lane, r);
                const int n = 16 * (sn + j) + li;
                if (m < M && n < N && !(symmetric && sm + i > sn + j))
                    P[m - TT * tm + (n - TT * tn) * TT] = acc[i][j][r];
            }
}

// C = alpha * sum over splits, eighths of them by a thread each and in order;
// with `symmetric` only strip pairs sn >= sm were computed and the lower ones are
// mirrored.  tile: edge of the active tiles that a split's partial holds one after
// another, 0 where it holds an M x N matrix.
__global__ __launch_bounds__(256) void k_gemm_reduce(int M, int N, int nsplit, const double* __restrict__ part,
                                                     double alpha, double* __restrict__ C, int ldc, bool symmetric,
                                                     int tile, int tiles_m, int active) {
    __shared__ double eighth[8][33];
    const int el = threadIdx.x & 31, q = threadIdx.x >> 5;
    const long ms = (long)M * N, e = (long)blockIdx.x * 32 + el;
    const int m = (int)(min(e, ms - 1) % M), n = (int)(min(e, ms - 1) / M);
    int sm = m, sn = n;
    if (symmetric && n / 16 < m / 16) {
        sm = n;
        sn = m;
    }
    const double* p = part + sm + (long)sn * M;
    long step = ms;
    if (tile) {
        const int tm = sm / tile, tn = sn / tile, tidx = symmetric ? tn * (tn + 1) / 2 + tm : tn * tiles_m + tm;
        p = part + (long)tidx * tile * tile + (sm - tm * tile) + (long)(sn - tn * tile) * tile;
        step = (long)active * tile * tile;
    }
    const int len = (nsplit + 7) / 8, end = min(nsplit, (q + 1) * len);
    double s = 0.0;
    for (int k = q * len; k < end; k += 4) {
        double v[4];
#pragma unroll
        for (int u = 0; u < 4; ++u) v[u] = p[min(k + u, end - 1) * step];
#pragma unroll
        for (int u = 0; u < 4; ++u)
            if (k + u < end) s += v[u];
    }
    eighth[q][el] = s;
    __syncthreads();
    if (q || e >= ms) return;
    s = 0.0;
    for (int k = 0; k < 8; ++k) s += eighth[k][el];
    C[m + (long)n * ldc] = alpha * s;
}

// Splits of K in FP64: the fewest that fill whole rounds of the workgroups that
// the chip holds to within 3%, in multiples of 8 (see the kernels), at least 128
// rows each, and no more than 512 MB of partial sums (`bytes` each) unless 8 take
// more.  1.73M x 1200 x 1200: 64, 461 MB (737 as full matrices), 48.8 ms; 9, the fewest
// of any count that fill a round, 104 MB and 50.7 ms.
static int tn_splits(int active, long K, int waves, size_t bytes) {
    const long most = std::min(std::max<long>(1, K / 128), std::max<long>(8, ((long)512 << 20) / (long)bytes));
    if (most < 8) return (int)most;
    int best = 8;
    double full = 0;
    for (long f = 8; f <= most && (f == 8 || f * active <= 8L * waves); f += 8) {
        const long n = f * active;
        const double use = (double)n / (double)((n + waves - 1) / waves * waves);
        if (use > full + 0.03) {
            full = use;
            best = (int)f;
        }
    }
    return best;
}

// Splits of K in FP32, whose sums run in FP32 inside a split: their number sets
// the rounding, so it goes with the sizes alone (about 512 tiles of 32, 64, 160
// or 128 columns, in a multiple of 8, at least 1024 rows each).
static int tn_splits_f32(int M, int N, long K, bool symmetric) {
    const int mx = std::max(M, N), tile = mx <= 32 ? 32 : (mx <= 64 ? 64 : (mx <= 320 ? 160 : 128));
    const int tm = div_up(M, tile), tn = div_up(N, tile), tiles = symmetric ? tm * (tm + 1) / 2 : tm * tn;
    const long want = std::max<long>(1, 512 / tiles);
    const int n = 8 * (int)std::max<long>(1, (want + 4) / 8);
    return (long)n * 1024 > K ? (int)std::max<long>(1, K / 1024) : n;
}

// Where the K rows go: MT x NT strips per workgroup.
struct TnGrid {
    int tiles_m = 0, active = 0, nsplit = 0;
    long kchunk = 0;
    size_t part = 0;   // values of a split's partial
};
static TnGrid tn_grid(int M, int N, long K, bool symmetric, int MT, int NT, int f32_splits, int slots, bool tiles) {
    TnGrid G;
    G.tiles_m = div_up(M, 16 * MT);
    const int tiles_n = div_up(N, 16 * NT);
    G.active = G.tiles_m * tiles_n;
    if (symmetric) {
        G.active = 0;
        for (int tn = 0; tn < tiles_n; ++tn) G.active += std::min(G.tiles_m, (tn * NT + NT - 1) / MT + 1);
    }
    G.part = tiles ? (size_t)G.active * 256 * MT * NT : (size_t)M * N;
    G.nsplit = f32_splits ? f32_splits : tn_splits(G.active, K, slots, G.part * sizeof(double));
    G.kchunk = ((K + G.nsplit - 1) / G.nsplit + 15) / 16 * 16;
    return G;
}

// Up to 32 columns (in FP32 64 of at most half a million rows) a step holds few
// products and its loads dominate: small tiles straight from L2, two steps of loads
// in flight, a wave per workgroup (24^3 rows x 24: 8 us, through LDS 35; FP32 24^3 x
// 33 26, in 4 x 3 strips 55; 72^3 x 48 51 and 56, 100^3 x 48 103 and 97).
// FP32 above that 4 x 3 strips (its splits are few: 8 of 1200 columns in 4 x 4
// strips fill three quarters of the chip's wave slots).  FP64 through LDS: up to 64
// columns in one tile of that width (24^3 rows x 33 columns 14 us, in a 128-wide
// tile 21; 72^3 x 64 62 and 100, 100^3 x 33 98 and 199; from L2 11, 87, 133), above it 128
// columns per tile (two workgroups per compute unit), or 160 (one) where up to
// 320 columns need fewer tiles that way: 72^3 rows x 128 columns 190 and 281 us,
// x 160 436 and 337, x 200 590 and 979, x 320 1282 and 1137.
template <typename T>
sparc_status gemm_tn(sparc_gpu_ctx c, int M, int N, long K, const T* A, long lda, const T* B, long ldb,
                     double alpha, double* C, int ldc, bool symmetric) {
    if (symmetric && M != N) return set_err(c, SPARC_ERR_ARG, "gemm_tn: symmetric needs M == N");
    const int mx = std::max(M, N), cus = c->prop.multiProcessorCount;
    const int f32 = sizeof(T) == 4 ? tn_splits_f32(M, N, K, symmetric) : 0;
    // strips of a tile's edge
    int strips = sizeof(T) == 4 ? (mx <= 32 || (mx <= 64 && K < 1L << 19) ? 2 : 4)
                 : mx <= 32     ? 2
                 : mx <= 64     ? 4
                                : (mx <= 320 && div_up(mx, 160) < div_up(mx, 128) ? 10 : 8);
    if (sizeof(T) == 8 && mx > 64 && c->gemm_tile) strips = c->gemm_tile / 16;
    const bool lds = sizeof(T) == 8 && strips > 2;
    const TnGrid G = tn_grid(M, N, K, symmetric, strips, strips == 4 && !lds ? 3 : strips, f32,
                             strips == 10 ? cus : (lds ? (strips == 8 ? 2 : 4) * cus : 8 * cus), lds);
    sparc_status st = ensure_gemm_part(c, G.nsplit * G.part);
    if (st != SPARC_OK) return st;
    const long nblocks = (long)G.active * G.nsplit;
    if (nblocks > 0x7fffffffL) return set_err(c, SPARC_ERR_ARG, "gemm_tn: too many blocks");
    const int slot = prof_begin(c, PK_GEMM_TN);
    const dim3 g((unsigned)nblocks);
    double* part = c->gemm_part;
    if (strips == 2) {
        k_gemm_tn_split<T, 2, 2, 3><<<g, 64, 0, c->stream>>>(M, N, K, G.kchunk, A, lda, B, ldb, part, G.tiles_m,
                                                             symmetric, G.active, G.nsplit);
    } else if constexpr (sizeof(T) == 4) {
        k_gemm_tn_split<T, 4, 3, 2><<<g, 64, 0, c->stream>>>(M, N, K, G.kchunk, A, lda, B, ldb, part, G.tiles_m,
                                                             symmetric, G.active, G.nsplit);
    } else if (strips == 4) {
        k_gemm_tn_lds<2><<<g, 256, 0, c->stream>>>(M, N, K, G.kchunk, A, lda, B, ldb, part, G.tiles_m, symmetric,
                                                   G.active, G.nsplit);
    } else if (strips == 10) {
        k_gemm_tn_lds<5><<<g, 256, 0, c->stream>>>(M, N, K, G.kchunk, A, lda, B, ldb, part, G.tiles_m, symmetric,
                                                   G.active, G.nsplit);
    } else {
        k_gemm_tn_lds<4><<<g, 256, 0, c->stream>>>(M, N, K, G.kchunk, A, lda, B, ldb, part, G.tiles_m, symmetric,
                                                   G.active, G.nsplit);
    }
    SG_CHECK_LAUNCH(c);
    prof_end(c, slot);
    k_gemm_reduce<<<div_up((long)M * N, 32), 256, 0, c->stream>>>(M, N, G.nsplit, part, alpha, C, ldc, symmetric,
                                                                 lds ? 16 * strips : 0, G.tiles_m, G.active);
    SG_CHECK_LAUNCH(c);
    return SPARC_OK;
}

// Out (K x N) = A (K x M) Bm (M x N).  A wave owns 64 rows and NT strips of 16
// columns, a workgroup 4 / WN x WN waves, whose shared operands meet in the L1.  The
// products run transposed (Bm's columns are MFMA rows), so that the 16 lanes of a
// group hold neighbouring rows of A and of Out: V per lane, whole 256-byte runs
// in FP64.  Row blocks go round the XCDs, all columns of one on the same.
// Bm is double, rounded to T.
constexpr int kNnRows = 64;

template <typename T, int NT, int WN>
__global__ __launch_bounds__(256, 2) void k_gemm_nn(long K, int N, int M, const T* __restrict__ A, long lda,
                                                    const double* __restrict__ Bm, int ldb, T* __restrict__ Out,
                                                    long ldo, int tiles_n, long tiles_r) {
    using acc_t = typename Mfma<T>::acc_t;
    constexpr int V = 16 / sizeof(T), KS = 4 * V;   // rows and contraction columns of a lane; columns of a step
    constexpr int MT = 4, MG = MT / V;              // strips of rows, in groups of V
    constexpr int WR = 4 / WN;                      // waves along the rows
    constexpr int RING = 3;                         // steps in registers, one of them in use
    using vec = typename GemmVec<T, V>::type;
    using bvec = typename GemmVec<double, V>::type;
    const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6, li = lane & 15, g = lane >> 4;
    const long slot = blockIdx.x / 8, rb = slot / tiles_n * 8 + blockIdx.x % 8;
    if (rb >= tiles_r) return;
    // the last rows' block is moved back to a whole one (the same results twice)
    const long r0 = min(K - kNnRows, (WR * rb + wv % WR) * kNnRows);
    const int sn = ((int)(slot % tiles_n) * WN + wv / WR) * NT;
    const int nj = min(NT, (N + 15) / 16 - sn);
    if (nj <= 0) return;
    const int nst = M / KS;
    const T* pa[MG];
#pragma unroll
    for (int i = 0; i < MG; ++i) pa[i] = A + r0 + 16 * V * i + V * li + (long)(V * g) * lda;
    const double* pb[NT];
#pragma unroll
    for (int j = 0; j < NT; ++j) pb[j] = Bm + (long)min(N - 1, 16 * (sn + min(j, nj - 1)) + li) * ldb + V * g;
    acc_t acc[MT][NT];
#pragma unroll
    for (int i = 0; i < MT; ++i)
#pragma unroll
        for (int j = 0; j < NT; ++j) acc[i][j] = acc_t{0, 0, 0, 0};
    auto products = [&](const vec (&va)[V][MG], const bvec (&vb)[NT], bool all) __attribute__((always_inline)) {
#pragma unroll
        for (int u = 0; u < V; ++u)
#pragma unroll
            for (int j = 0; j < NT; ++j)
                if (all || j < nj) {
                    const T b = (T)vb[j][u];
#pragma unroll
                    for (int i = 0; i < MT; ++i) acc[i][j] = Mfma<T>::run(b, va[u][i / V][i % V], acc[i][j]);
                }
    };
    if (nst > 0) {
        vec qa[RING][V][MG];
        bvec qb[RING][NT];
        auto load = [&](int r, int s) __attribute__((always_inline)) {
            const int k = min(s, nst - 1) * KS;
#pragma unroll
            for (int u = 0; u < V; ++u)
#pragma unroll
                for (int i = 0; i < MG; ++i) qa[r][u][i] = *reinterpret_cast<const vec*>(pa[i] + (long)(k + u) * lda);
#pragma unroll
            for (int j = 0; j < NT; ++j) qb[r][j] = *reinterpret_cast<const bvec*>(pb[j] + k);
        };
#pragma unroll
        for (int r = 0; r < RING - 1; ++r) load(r, r);
        auto run = [&](bool all) __attribute__((always_inline)) {
            for (int s = 0; s < nst; s += RING) {
#pragma unroll
                for (int r = 0; r < RING; ++r) {
                    if (s + r >= nst) break;
                    load((r + RING - 1) % RING, s + r + RING - 1);
                    products(qa[r], qb[r], all);
                }
            }
        };
        if (nj == NT) run(true);
        else run(false);
    }
    if (M % KS) {
        // the columns past the last whole step, zero past the end
        vec va[V][MG];
        bvec vb[NT];
#pragma unroll
        for (int u = 0; u < V; ++u) {
            const int k = nst * KS + u;
            const bool in = k + V * g < M;
#pragma unroll
            for (int i = 0; i < MG; ++i) va[u][i] = in ? *reinterpret_cast<const vec*>(pa[i] + (long)k * lda) : vec(0);
#pragma unroll
            for (int j = 0; j < NT; ++j) vb[j][u] = in ? pb[j][k] : 0.0;
        }
        products(va, vb, false);
    }
#pragma unroll
    for (int i = 0; i < MG; ++i)
#pragma unroll
        for (int j = 0; j < NT; ++j)
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                const int n = 16 * (sn + j) + Mfma<T>::row(lane, r);
                vec o;
#pragma unroll
                for (int v = 0; v < V; ++v) o[v] = acc[V * i + v][j][r];
                if (n < N) *reinterpret_cast<vec*>(Out + r0 + 16 * V * i + V * li + (long)n * ldo) = o;
            }
}

template <typename T, int NT, int WN>
static sparc_status gemm_nn_launch(sparc_gpu_ctx c, long K, int N, int M, const T* A, long lda, const double* Bm,
                                   int ldb, T* Out, long ldo) {
    if (K < kNnRows) return set_err(c, SPARC_ERR_ARG, "gemm_nn: fewer than 64 rows");
    constexpr long rows = kNnRows * 4 / WN;
    const int tiles_n = div_up(N, 16 * NT * WN);
    const long tiles_r = (K + rows - 1) / rows, nblocks = (tiles_r + 7) / 8 * 8 * tiles_n;
    if (nblocks > 0x7fffffffL) return set_err(c, SPARC_ERR_ARG, "gemm_nn: too many blocks");
    const int slot = prof_begin(c, PK_GEMM_NN);
    k_gemm_nn<T, NT, WN><<<dim3((unsigned)nblocks), 256, 0, c->stream>>>(K, N, M, A, lda, Bm, ldb, Out, ldo, tiles_n,
                                                                         tiles_r);
    SG_CHECK_LAUNCH(c);
    prof_end(c, slot);
    return SPARC_OK;
}

// Tiles of 64 columns, two side by side above 64 (64^3 rows x 64: 57 us, 84 with
// two), and of 32 up to 32 columns (60^3 rows x 30: 23 us, 31).  At 1.73M x 1200 x
// 1200 78 ms in FP64 and 53 in FP32, through LDS 92 and 71.
template <typename T>
sparc_status gemm_nn(sparc_gpu_ctx c, long K, int N, int M, const T* A, long lda, const double* Bm, int ldb, T* Out,
                     long ldo) {
    if (N <= 32) return gemm_nn_launch<T, 2, 1>(c, K, N, M, A, lda, Bm, ldb, Out, ldo);
    if (N <= 64) return gemm_nn_launch<T, 4, 1>(c, K, N, M, A, lda, Bm, ldb, Out, ldo);
    return gemm_nn_launch<T, 4, 2>(c, K, N, M, A, lda, Bm, ldb, Out, ldo);
}

template sparc_status gemm_tn<double>(sparc_gpu_ctx, int, int, long, const double*, long, const double*, long, double,
                                      double*, int, bool);
template sparc_status gemm_tn<float>(sparc_gpu_ctx, int, int, long, const float*, long, const float*, long, double,
                                     double*, int, bool);
template sparc_status gemm_nn<double>(sparc_gpu_ctx, long, int, int, const double*, long, const double*, int, double*,
                                      long);
template sparc_status gemm_nn<float>(sparc_gpu_ctx, long, int, int, const float*, long, const double*, int, float*,
                                     long);

}  // namespace sg
