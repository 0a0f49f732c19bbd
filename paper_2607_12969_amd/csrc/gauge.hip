// Left-orthogonal gauge of an FP64 Tensor Train (Sec. 6.1; Algorithm
// alg:tt_compensation, gauge step): for l = 1..d-1 the left unfolding of
// core l, A = G_l as (r_{l-1} n_l) x r_l, is factored A = Q R with
// Q^T Q = I and diag(R) > 0; core l becomes Q and R is multiplied into the
// left unfolding of core l+1 (r_l x n_{l+1} r_{l+1}).
//
// The QR of each unfolding is CholeskyQR2: with the Gram matrix A^T A = R_1^T
// R_1 (Cholesky), Q_1 = A R_1^{-1}; then Q_1^T Q_1 = R_2^T R_2, Q = Q_1
// R_2^{-1} and R = R_2 R_1.  The first pass leaves an orthogonality error of
// order cond(A)^2 u, the second removes it while cond(A)^2 u stays well
// below one; the Cholesky stops with an error when a pivot falls below 2^-46
// of its column's squared norm (cond(A) above about 10^7), where the
// factorization would no longer be accurate.  With positive diagonals both
// R and Q are the unique thin QR factors of a full-rank A, so the result
// agrees to rounding with a Householder QR of the same convention.
//
// Work per unfolding (m rows, r columns): two Gram products on the FP64
// matrix cores (launch_gram: 2 m r^2 flop each, half of it computed), two
// triangular solves x R = a per row (blocked forward substitution on the
// matrix cores, m r^2 flop each; only diagonal blocks are inverted, with a
// correction), and R G_{l+1} applied as R_2 (R_1 G_{l+1})
// (two triangular products, r^2 n_{l+1} r_{l+1} flop each).  All of it is
// small next to the reconstruction.
#include <hip/hip_runtime.h>

#include <algorithm>

#include "../../include/lrc.h"
#include "lrc_device.h"
#include "lrc_internal.h"

namespace lrc {

// dst[i][j] = src[i][j] for j < r, 0 for r <= j < ldd (rows x ldd)
__global__ __launch_bounds__(256) void k_gauge_pad(const double* __restrict__ src, int64_t rows, int r,
                                                   double* __restrict__ dst, int ldd) {
    const int64_t total = rows * ldd;
    for (int64_t idx = (int64_t)blockIdx.x * 256 + threadIdx.x; idx < total; idx += (int64_t)gridDim.x * 256) {
        const int64_t i = idx / ldd;
        const int j = (int)(idx - i * ldd);
        dst[idx] = j < r ? src[i * r + j] : 0.0;
    }
}

// One workgroup.  G (r x r inside pitch ld, symmetric, upper triangle used)
// = R^T R with R upper triangular, diag(R) > 0: right-looking Cholesky, the
// trailing update with the unscaled pivot row, S[i][j] -= S[k][i] S[k][j] /
// S[k][k], rows scaled at the end.  R is written with pitch ld, zero below
// the diagonal and in the pad rows and columns.  flag: set to 1 + (pivot
// index) when a pivot is not above 2^-46 of the column's original diagonal
// (or not a number); R is then unspecified.  shift_rel > 0 factors G + s I
// instead, s = shift_rel trace(G) (the shifted first pass of shifted
// CholeskyQR3).
//
// Bound by the chain of pivots (row to LDS, barrier, division, update): the
// matrix stays in the registers of a 16 x 16 thread grid (thread (ty, tx)
// holds rows ty + 16 a and columns tx + 16 b, b >= a), only the pivot row
// passes through LDS (two buffers, one barrier per pivot), and NB = ceil(r /
// 16) is a template argument so that one wave per SIMD issues no more than
// the live blocks.  r = 74: 23 us (47 with the matrix in LDS, 1024 threads).
constexpr int kGaugeMaxRank = LRC_GAUGE_MAX_RANK;
constexpr int kGaugeMaxBlocks = (kGaugeMaxRank + 15) / 16;

template <int NB, int KB>
__device__ __forceinline__ void chol_block(double (&S)[NB][NB], double (*buf)[16 * NB], double* piv,
                                           const double* diag0, int r, int tx, int ty, int* bad) {
    if constexpr (KB < NB) {
        const int kend = r - 16 * KB < 16 ? r - 16 * KB : 16;
        for (int kk = 0; kk < kend; ++kk) {
            const int k = 16 * KB + kk;
            double* row = buf[kk & 1];
            if (ty == kk) {
#pragma unroll
                for (int b = KB; b < NB; ++b) row[16 * b + tx] = S[KB][b];
            }
            __syncthreads();
            const double d = row[k];
            const double inv = 1.0 / (d > 0.0 ? d : 0.0);
            double rj[NB], ri[NB];
#pragma unroll
            for (int b = KB; b < NB; ++b) {
                rj[b] = row[16 * b + tx];
                ri[b] = row[16 * b + ty];
            }
            if (tx == 0 && ty == 0) {
                piv[k] = d;
                if (!(d > 0x1p-46 * diag0[k]) && *bad == 0) *bad = 1 + k;
            }
#pragma unroll
            for (int a = KB; a < NB; ++a) {
                // finished rows (only in block KB) keep their values; entries
                // below the diagonal are never used
                const double ski = (a > KB || ty > kk) ? ri[a] * inv : 0.0;
#pragma unroll
                for (int b = a; b < NB; ++b) S[a][b] = S[a][b] - ski * rj[b];
            }
        }
        // a block with an odd number of pivots is the last one, so the next
        // block's first pivot always uses the other buffer than the one read last
        chol_block<NB, KB + 1>(S, buf, piv, diag0, r, tx, ty, bad);
    }
}

template <int NB>
__global__ __launch_bounds__(256) void k_gauge_chol(const double* __restrict__ G, int r, int ld,
                                                    double* __restrict__ R, int* __restrict__ flag,
                                                    double shift_rel) {
    __shared__ double buf[2][16 * NB];
    __shared__ double diag0[16 * NB], piv[16 * NB];
    __shared__ int bad;
    const int tid = threadIdx.x, tx = tid & 15, ty = tid >> 4;
    double S[NB][NB];
#pragma unroll
    for (int a = 0; a < NB; ++a)
#pragma unroll
        for (int b = a; b < NB; ++b) {
            const int i = 16 * a + ty, j = 16 * b + tx;
            S[a][b] = (j >= i && j < r) ? G[(int64_t)i * ld + j] : 0.0;
        }
    if (tid == 0) bad = 0;
    if (tx == ty) {
#pragma unroll
        for (int a = 0; a < NB; ++a) diag0[16 * a + tx] = S[a][a];
    }
    __syncthreads();
    if (shift_rel > 0.0) {
        // trace summed by every thread in index order (deterministic)
        double tr = 0.0;
        for (int i = 0; i < r; ++i) tr += diag0[i];
        const double sh = shift_rel * tr;
        __syncthreads();
        if (tx == ty) {
#pragma unroll
            for (int a = 0; a < NB; ++a) {
                S[a][a] += sh;
                diag0[16 * a + tx] = S[a][a];
            }
        }
        __syncthreads();
    }
    chol_block<NB, 0>(S, buf, piv, diag0, r, tx, ty, &bad);
    __syncthreads();
    if (tid == 0 && bad) *flag = bad;
#pragma unroll
    for (int a = 0; a < NB; ++a) {
        const int i = 16 * a + ty;
        const double d = i < r ? piv[i] : 0.0;
        const double sq = __builtin_sqrt(d > 0.0 ? d : 0.0);
#pragma unroll
        for (int b = 0; b < NB; ++b) {
            const int j = 16 * b + tx;
            if (i >= ld || j >= ld) continue;
            double v = 0.0;
            if (b >= a && i < r && j < r && j >= i) v = j == i ? sq : S[a][b >= a ? b : a] / sq;
            R[(int64_t)i * ld + j] = v;
        }
    }
}

static void launch_chol(const double* G, int r, int ld, double* R, int* flag, double shift_rel, hipStream_t st) {
    switch ((r + 15) / 16) {
        case 1: hipLaunchKernelGGL(k_gauge_chol<1>, dim3(1), dim3(256), 0, st, G, r, ld, R, flag, shift_rel); break;
        case 2: hipLaunchKernelGGL(k_gauge_chol<2>, dim3(1), dim3(256), 0, st, G, r, ld, R, flag, shift_rel); break;
        case 3: hipLaunchKernelGGL(k_gauge_chol<3>, dim3(1), dim3(256), 0, st, G, r, ld, R, flag, shift_rel); break;
        case 4: hipLaunchKernelGGL(k_gauge_chol<4>, dim3(1), dim3(256), 0, st, G, r, ld, R, flag, shift_rel); break;
        case 5: hipLaunchKernelGGL(k_gauge_chol<5>, dim3(1), dim3(256), 0, st, G, r, ld, R, flag, shift_rel); break;
        default: hipLaunchKernelGGL(k_gauge_chol<6>, dim3(1), dim3(256), 0, st, G, r, ld, R, flag, shift_rel);
    }
}
static_assert(kGaugeMaxBlocks == 6, "launch_chol and launch_trsm name every block count");

// C = A R^{-1} row by row (R upper triangular r x r with pitch ldr, A with
// pitch lda, C with pitch ldc whose pad columns r <= j < ldc are zeroed):
// blocked forward substitution on the FP64 matrix cores.  With L = R^T and
// X = C^T in blocks of 16, X_i = L_ii^{-1} (A^T_i - sum_{j < i} L_ij X_j).
// A wave holds NT tiles of 16 rows of A as columns of X: lane (g = lane >> 4,
// c = lane & 15) keeps X[16 i + 4 g + v][row c] in element v of block i.
// That is 32 consecutive bytes of a row, and, with the rows of a block
// numbered 4 (n & 3) + (n >> 2) for the instruction's index n, at once the
// result and the right operand of the instruction, so X never leaves the
// registers.  The blocks of -L sit in LDS in the order the lanes read them;
// each workgroup inverts the diagonal blocks itself (one thread per column).
// A diagonal block is solved as x = D b, x += D (b - L_ii x), D = L_ii^{-1}:
// the correction leaves a residual of order u |L_ii| |x|, as substitution
// does.  114688 x 74: 66 us (substitution by lane broadcasts took 204; memory
// takes 23); 32768 x 74: 24 us (67).  lda even, A 16-byte aligned; C any
// alignment.
__device__ __forceinline__ int trsm_perm(int n) { return 4 * (n & 3) + (n >> 2); }   // its own inverse

template <int NB, int NT>
__global__ __launch_bounds__(256) void k_gauge_trsm(const double* __restrict__ A, int64_t rows, int r, int lda,
                                                    const double* __restrict__ R, int ldr,
                                                    double* __restrict__ C, int ldc) {
    constexpr int kPairs = NB * (NB + 1) / 2;
    __shared__ double F[kPairs][4][64];   // -L_ij, i >= j, pair i (i + 1) / 2 + j
    __shared__ double D[NB][4][64];       // L_ii^{-1}
    const int tid = threadIdx.x, lane = tid & 63, c = lane & 15, g = lane >> 4;
    {
        double v[kPairs];
        const int s = tid >> 6, t = trsm_perm(c);
#pragma unroll
        for (int i = 0, p = 0; i < NB; ++i)
#pragma unroll
            for (int j = 0; j <= i; ++j, ++p) {
                const int row = 16 * j + 4 * g + s, col = 16 * i + t;
                v[p] = (row <= col && col < r) ? -R[(int64_t)row * ldr + col] : row == col ? -1.0 : 0.0;
            }
#pragma unroll
        for (int p = 0; p < kPairs; ++p) F[p][s][lane] = v[p];
    }
    __syncthreads();
    if (tid < 16 * NB) {
        const int i = tid >> 4, col = tid & 15;
        const double(*Fi)[64] = F[i * (i + 1) / 2 + i];
        double y[16];
#pragma unroll
        for (int t = 0; t < 16; ++t) {
            double sum = t == col ? 1.0 : 0.0;
#pragma unroll
            for (int k = 0; k < t; ++k) sum += Fi[k & 3][(k >> 2) * 16 + trsm_perm(t)] * y[k];
            y[t] = sum / -Fi[t & 3][(t >> 2) * 16 + trsm_perm(t)];
        }
#pragma unroll
        for (int t = 0; t < 16; ++t) D[i][col & 3][(col >> 2) * 16 + trsm_perm(t)] = y[t];
    }
    __syncthreads();
    const bool wide = ldc % 2 == 0 && reinterpret_cast<uintptr_t>(C) % 16 == 0;
    const int64_t step = (int64_t)gridDim.x * 4 * NT * 16;
    for (int64_t i0 = ((int64_t)blockIdx.x * 4 + (tid >> 6)) * NT * 16; i0 < rows; i0 += step) {
        double4_t x[NT][NB];
#pragma unroll
        for (int q = 0; q < NT; ++q) {
            const int64_t i = i0 + 16 * q + c;
            const double* a = A + (i < rows ? i : rows - 1) * lda;
#pragma unroll
            for (int b = 0; b < NB; ++b)
#pragma unroll
                for (int h = 0; h < 2; ++h) {
                    const int t = 16 * b + 4 * g + 2 * h;
                    double2 w = make_double2(0.0, 0.0);
                    if (t < r) w = *reinterpret_cast<const double2*>(a + t);   // t even, so t + 1 < lda
                    x[q][b][2 * h] = w.x;
                    x[q][b][2 * h + 1] = t + 1 < r ? w.y : 0.0;
                }
        }
#pragma unroll
        for (int i = 0; i < NB; ++i) {
            const int p0 = i * (i + 1) / 2;
#pragma unroll
            for (int j = 0; j < i; ++j)
#pragma unroll
                for (int s = 0; s < 4; ++s) {
                    const double f = F[p0 + j][s][lane];
#pragma unroll
                    for (int q = 0; q < NT; ++q) x[q][i] = mfma(f, x[q][j][s], x[q][i]);
                }
            double d[4], f[4];
#pragma unroll
            for (int s = 0; s < 4; ++s) {
                d[s] = D[i][s][lane];
                f[s] = F[p0 + i][s][lane];
            }
            double4_t x0[NT];
#pragma unroll
            for (int q = 0; q < NT; ++q) x0[q] = zero_accv<double4_t>();
#pragma unroll
            for (int s = 0; s < 4; ++s)
#pragma unroll
                for (int q = 0; q < NT; ++q) x0[q] = mfma(d[s], x[q][i][s], x0[q]);
#pragma unroll
            for (int s = 0; s < 4; ++s)
#pragma unroll
                for (int q = 0; q < NT; ++q) x[q][i] = mfma(f[s], x0[q][s], x[q][i]);
#pragma unroll
            for (int s = 0; s < 4; ++s)
#pragma unroll
                for (int q = 0; q < NT; ++q) x0[q] = mfma(d[s], x[q][i][s], x0[q]);
#pragma unroll
            for (int q = 0; q < NT; ++q) x[q][i] = x0[q];
        }
#pragma unroll
        for (int q = 0; q < NT; ++q) {
            const int64_t i = i0 + 16 * q + c;
            if (i >= rows) continue;
            double* o = C + i * ldc;
#pragma unroll
            for (int b = 0; b < NB; ++b) {
                const int t = 16 * b + 4 * g;
                if (wide) {
#pragma unroll
                    for (int h = 0; h < 2; ++h)
                        if (t + 2 * h < ldc)
                            *reinterpret_cast<double2*>(o + t + 2 * h) = make_double2(x[q][b][2 * h], x[q][b][2 * h + 1]);
                } else {
#pragma unroll
                    for (int v = 0; v < 4; ++v)
                        if (t + v < ldc) o[t + v] = x[q][b][v];
                }
            }
        }
    }
}

// C[i][c] = sum_{t >= i} R[i][t] X[t][c] for i < r, c < ncols (R upper
// triangular with pitch ldr, X and C r x ncols dense).  Workgroup (x, y)
// takes columns 256 x .. 256 x + 255 (one per thread, read coalesced) and
// output rows ROWS y .. ROWS y + ROWS - 1, whose rows of R it keeps in LDS
// (zero below the diagonal, so the loop has no masks).  32 rows share a read
// of a wide X; a product of two triangles (a single column of workgroups) is
// bound by the latency of its reads, which 8 rows and batches of 32 reads
// spread over more units and hide (r = 74: 22 -> 9 us).
template <int ROWS, int BATCH>
__global__ __launch_bounds__(256) void k_gauge_lmul(const double* __restrict__ R, int r, int ldr,
                                                    const double* __restrict__ X, int64_t ncols,
                                                    double* __restrict__ C) {
    __shared__ double Rs[LRC_GAUGE_MAX_RANK][ROWS];   // Rs[t][u] = R[i0 + u][t]
    const int i0 = blockIdx.y * ROWS;
    // all loads first, then the LDS writes (their latencies overlap)
    constexpr int kPer = LRC_GAUGE_MAX_RANK * ROWS / 256;
    double v[kPer];
#pragma unroll
    for (int q = 0; q < kPer; ++q) {
        const int idx = threadIdx.x + q * 256;
        const int t = idx / ROWS, i = i0 + idx % ROWS;
        v[q] = (t < r && i < r && t >= i) ? R[(int64_t)i * ldr + t] : 0.0;
    }
#pragma unroll
    for (int q = 0; q < kPer; ++q) {
        const int idx = threadIdx.x + q * 256;
        Rs[idx / ROWS][idx % ROWS] = v[q];
    }
    __syncthreads();
    const int64_t c = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (c >= ncols) return;
    double acc[ROWS];
#pragma unroll
    for (int u = 0; u < ROWS; ++u) acc[u] = 0.0;
    // columns of X in batches of rows: the loads of a batch overlap
    for (int t0 = i0; t0 < r; t0 += BATCH) {
        double xv[BATCH];
#pragma unroll
        for (int q = 0; q < BATCH; ++q) xv[q] = t0 + q < r ? X[(int64_t)(t0 + q) * ncols + c] : 0.0;
#pragma unroll
        for (int q = 0; q < BATCH; ++q) {
            if (t0 + q < r) {
#pragma unroll
                for (int u = 0; u < ROWS; ++u) acc[u] += Rs[t0 + q][u] * xv[q];
            }
        }
    }
#pragma unroll
    for (int u = 0; u < ROWS; ++u)
        if (i0 + u < r) C[(int64_t)(i0 + u) * ncols + c] = acc[u];
}

static unsigned gauge_grid(int64_t items, int per_block) {
    int64_t g = (items + per_block - 1) / per_block;
    if (g > 8192) g = 8192;
    return (unsigned)(g < 1 ? 1 : g);
}

size_t gauge_workspace_bytes(const int64_t* dims, const int64_t* ranks, int d) {
    size_t need = 0;
    for (int l = 0; l + 1 < d; ++l) {
        const int64_t rows = ranks[l] * dims[l], r = ranks[l + 1];
        const int64_t rp = round_up(r, 2);
        const int64_t ncols = dims[l + 1] * ranks[l + 2];
        size_t b = 0;
        b += round_up((int64_t)(rows * rp * 8), 256) * 2;                   // W1, W2
        b += round_up((int64_t)(rp * rp * 8), 256) * 3;                     // G, R1, R2
        b += round_up((int64_t)gram_workspace_bytes(rows, rp), 256);        // Gram partials
        b += round_up((int64_t)(r * ncols * 8), 256);                       // R1 G_{l+1}
        need = b > need ? b : need;
    }
    return need + 256 + (size_t)round_up(4 * (int64_t)d, 256);
}

__global__ void k_gauge_zero(int* p, int n) {
    for (int i = threadIdx.x; i < n; i += blockDim.x) p[i] = 0;
}

// Two row tiles per wave share each fragment of R where that still leaves a
// wave for every SIMD (1024 waves of 32 rows); the grid is bounded so that a
// workgroup's set-up (R to LDS, diagonal blocks inverted, most of the 13 us
// that 512 rows take) is spread over several tiles.
template <int NB>
static void launch_trsm_nb(const double* A, int64_t rows, int r, int lda, const double* R, int ldr, double* C,
                           int ldc, hipStream_t st) {
    const int nt = rows >= 32768 ? 2 : 1;
    const int64_t g = std::min<int64_t>((rows + 64 * nt - 1) / (64 * nt), 512);
    if (nt == 2)
        hipLaunchKernelGGL((k_gauge_trsm<NB, 2>), dim3((unsigned)g), dim3(256), 0, st, A, rows, r, lda, R, ldr, C, ldc);
    else
        hipLaunchKernelGGL((k_gauge_trsm<NB, 1>), dim3((unsigned)g), dim3(256), 0, st, A, rows, r, lda, R, ldr, C, ldc);
}

static void launch_trsm(const double* A, int64_t rows, int r, int lda, const double* R, int ldr, double* C,
                        int ldc, hipStream_t st) {
    switch ((r + 15) / 16) {
        case 1: launch_trsm_nb<1>(A, rows, r, lda, R, ldr, C, ldc, st); break;
        case 2: launch_trsm_nb<2>(A, rows, r, lda, R, ldr, C, ldc, st); break;
        case 3: launch_trsm_nb<3>(A, rows, r, lda, R, ldr, C, ldc, st); break;
        case 4: launch_trsm_nb<4>(A, rows, r, lda, R, ldr, C, ldc, st); break;
        case 5: launch_trsm_nb<5>(A, rows, r, lda, R, ldr, C, ldc, st); break;
        default: launch_trsm_nb<6>(A, rows, r, lda, R, ldr, C, ldc, st);
    }
}

size_t cholqr2_workspace_bytes(int64_t rows, int r) {
    const int64_t rp = round_up(r, 2);
    return (size_t)round_up(rows * rp * 8, 256) + 5 * (size_t)round_up(rp * rp * 8, 256) +
           (size_t)round_up((int64_t)gram_workspace_bytes(rows, rp), 256);
}

hipError_t launch_cholqr2(const double* A, int64_t rows, int r, double* Q, double* R, int* flag, Workspace& ws,
                          hipStream_t stream, const char* label, bool shifted) {
    const int rp = (int)round_up(r, 2);
    double* W2 = static_cast<double*>(ws.take((size_t)rows * rp * 8));
    double* G = static_cast<double*>(ws.take((size_t)rp * rp * 8));
    double* R1 = static_cast<double*>(ws.take((size_t)rp * rp * 8));
    double* R2 = static_cast<double*>(ws.take((size_t)rp * rp * 8));
    double* R3 = static_cast<double*>(ws.take((size_t)rp * rp * 8));
    double* RX = static_cast<double*>(ws.take((size_t)rp * rp * 8));
    if (ws.overrun) return hipErrorOutOfMemory;
    KernelTimer tm(label, stream);
    const size_t gmark = ws.used;
    // one pass: Gram of `in`, its Cholesky factor `Rk`, out = in Rk^{-1}
    auto pass = [&](const double* in, double* Rk, double* out, double shift_rel) {
        hipError_t e = launch_gram(in, rows, rp, G, ws, stream);
        ws.used = gmark;
        if (e != hipSuccess) return e;
        launch_chol(G, r, rp, Rk, flag, shift_rel, stream);
        launch_trsm(in, rows, r, rp, Rk, rp, out, rp, stream);
        return hipGetLastError();
    };
    // rows 0..r-1 of the triangular product dst = Ra Rb (Rb taken as an r x rp block)
    auto tri = [&](const double* Ra, const double* Rb, double* dst) {
        const dim3 gl((unsigned)((rp + 255) / 256), (unsigned)((r + 7) / 8));
        hipLaunchKernelGGL((k_gauge_lmul<8, 32>), gl, dim3(256), 0, stream, Ra, r, rp, Rb, (int64_t)rp, dst);
    };
    hipError_t e;
    if (!shifted) {
        if ((e = pass(A, R1, W2, 0.0)) != hipSuccess || (e = pass(W2, R2, Q, 0.0)) != hipSuccess) return e;
        if (R) tri(R2, R1, R);
    } else {
        // shifted CholeskyQR3 (Fukaya, Kannan, Nakatsukasa, Yamamoto, Yanagisawa 2020): the shift
        // s = 11 (m r + r (r + 1)) u ||A||_F^2 keeps the first factorization away from breakdown for
        // condition numbers up to about u^-1; two plain passes restore orthogonality
        const double shift_rel = 11.0 * ((double)rows * r + (double)r * (r + 1)) * 0x1p-53;
        if ((e = pass(A, R1, Q, shift_rel)) != hipSuccess || (e = pass(Q, R2, W2, 0.0)) != hipSuccess ||
            (e = pass(W2, R3, Q, 0.0)) != hipSuccess)
            return e;
        if (R) {
            tri(R2, R1, RX);
            tri(R3, RX, R);
        }
    }
    return hipGetLastError();
}

hipError_t launch_gauge(double* const* cores, const int64_t* dims, const int64_t* ranks, int d, int* flags,
                        Workspace& ws, hipStream_t stream) {
    hipLaunchKernelGGL(k_gauge_zero, dim3(1), dim3(64), 0, stream, flags, d);
    for (int l = 0; l + 1 < d; ++l) {
        const int64_t rows = ranks[l] * dims[l];
        const int r = (int)ranks[l + 1];
        const int rp = (int)round_up(r, 2);
        const int64_t ncols = dims[l + 1] * ranks[l + 2];
        const size_t mark = ws.used;
        double* W1 = static_cast<double*>(ws.take((size_t)rows * rp * 8));
        double* W2 = static_cast<double*>(ws.take((size_t)rows * rp * 8));
        double* G = static_cast<double*>(ws.take((size_t)rp * rp * 8));
        double* R1 = static_cast<double*>(ws.take((size_t)rp * rp * 8));
        double* R2 = static_cast<double*>(ws.take((size_t)rp * rp * 8));
        double* NX = static_cast<double*>(ws.take((size_t)r * ncols * 8));
        if (ws.overrun) return hipErrorOutOfMemory;
        KernelTimer tm("gauge_qr_f64", stream);
        hipLaunchKernelGGL(k_gauge_pad, dim3(gauge_grid(rows * rp, 256)), dim3(256), 0, stream, cores[l], rows, r,
                           W1, rp);
        // first pass: A^T A = R1^T R1, W2 = A R1^{-1}
        const size_t gmark = ws.used;
        hipError_t e = launch_gram(W1, rows, rp, G, ws, stream);
        if (e != hipSuccess) return e;
        ws.used = gmark;
        launch_chol(G, r, rp, R1, flags + l, 0.0, stream);
        launch_trsm(W1, rows, r, rp, R1, rp, W2, rp, stream);
        // second pass on W2: core l = W2 R2^{-1}; R = R2 R1
        e = launch_gram(W2, rows, rp, G, ws, stream);
        if (e != hipSuccess) return e;
        ws.used = gmark;
        launch_chol(G, r, rp, R2, flags + l, 0.0, stream);
        launch_trsm(W2, rows, r, rp, R2, rp, cores[l], r, stream);
        // core l+1 <- R2 (R1 core l+1) on its left unfolding (r x ncols)
        const dim3 gl((unsigned)((ncols + 255) / 256), (unsigned)((r + 31) / 32));
        hipLaunchKernelGGL((k_gauge_lmul<32, 8>), gl, dim3(256), 0, stream, R1, r, rp, cores[l + 1], ncols, NX);
        hipLaunchKernelGGL((k_gauge_lmul<32, 8>), gl, dim3(256), 0, stream, R2, r, rp, NX, ncols, cores[l + 1]);
        e = hipGetLastError();
        if (e != hipSuccess) return e;
        ws.used = mark;
    }
    return hipSuccess;
}

}  // namespace lrc
