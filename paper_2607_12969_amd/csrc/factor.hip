// Randomized FP64 factorizations on the device: the end-to-end decomposition
// that Sec. sec:conclusion leaves to future work, so that a dense matrix or
// tensor can be factored where the rank-compensated factors are then
// stored, applied and certified.  The method is the randomized range finder
// of Halko, Martinsson and Tropp (SIAM Review 2011) with the exact SVD of the
// small projected matrix, and TT-SVD (Sec. 5.1) with every truncated SVD
// replaced by it.  The Gaussian test vectors are inputs.
//
// Matrix A (m x n), l test vectors as the rows of Omega (l x n):
//   Y = A Omega^T                 split-K MFMA GEMM (m x l)
//   Y = Q R_Y                     CholeskyQR2 (Q^T Q = I)
//   q times: Z = orth(A^T Q), Q = orth(A Z)
//   B^T = A^T Q = Q_2 R           MFMA GEMM (n x l), CholeskyQR2
//   R^T = W diag(sigma) Z^T       one-sided Jacobi in one workgroup (l x l)
//   U = Q W,  V = Q_2 Z           (A ~= Q B = Q R^T Q_2^T = U diag(sigma) V^T)
// Only the GEMMs over A touch more than O((m + n) l) data; they run on the
// FP64 matrix cores and bound the whole (2 m n l flop each).
#include <hip/hip_runtime.h>

#include <algorithm>

#include "../../include/lrc.h"
#include "jac_rotation.h"
#include "lrc_device.h"
#include "lrc_internal.h"

namespace lrc {

constexpr int kFactMaxL = LRC_RSVD_MAX_SAMPLES;
constexpr int kJacSweeps = 40;

// dst (drows x ldd) = src (rows x cols, pitch lds) with zeros past rows / cols
__global__ __launch_bounds__(256) void k_fact_pad(const double* __restrict__ src, int64_t rows, int64_t cols,
                                                  int64_t lds, double* __restrict__ dst, int64_t drows, int64_t ldd) {
    const int64_t total = drows * ldd;
    for (int64_t idx = (int64_t)blockIdx.x * 256 + threadIdx.x; idx < total; idx += (int64_t)gridDim.x * 256) {
        const int64_t i = idx / ldd, j = idx - i * ldd;
        dst[idx] = (i < rows && j < cols) ? src[i * lds + j] : 0.0;
    }
}

// dst[j][i] = src[i][j] (src rows x cols with pitch lds; dst cols x ldd),
// zero for rows <= i < ldd; 32 x 32 tiles through LDS.
__global__ __launch_bounds__(256) void k_fact_transpose(const double* __restrict__ src, int64_t rows, int64_t cols,
                                                        int64_t lds, double* __restrict__ dst, int64_t ldd) {
    __shared__ double tile[32][33];
    const int64_t i0 = (int64_t)blockIdx.x * 32, j0 = (int64_t)blockIdx.y * 32;
    const int tx = threadIdx.x & 31, ty = threadIdx.x >> 5;
    for (int u = ty; u < 32; u += 8) {
        const int64_t i = i0 + u, j = j0 + tx;
        tile[u][tx] = (i < rows && j < cols) ? src[i * lds + j] : 0.0;
    }
    __syncthreads();
    for (int u = ty; u < 32; u += 8) {
        const int64_t j = j0 + u, i = i0 + tx;
        if (j < cols && i < ldd) dst[j * ldd + i] = tile[tx][u];
    }
}

__global__ void k_fact_zero(int* p, int n) {
    for (int i = threadIdx.x; i < n; i += blockDim.x) p[i] = 0;
}

// Value of lane `ctl` (a DPP row permutation) for a double: its two halves
// moved by the same data-parallel-primitive move.
template <int CTL>
__device__ __forceinline__ double dpp_f64(double v) {
    const long long b = __builtin_bit_cast(long long, v);
    // every lane receives a value, so there is no old one to keep
    const int lo = __builtin_amdgcn_mov_dpp((int)(b & 0xFFFFFFFFll), CTL, 0xF, 0xF, false);
    const int hi = __builtin_amdgcn_mov_dpp((int)(b >> 32), CTL, 0xF, 0xF, false);
    return __builtin_bit_cast(double, ((long long)hi << 32) | (unsigned int)lo);
}

// Sums of three values over each group of 16 lanes: butterfly by lane
// swaps within quads (xor 1, xor 2), then the mirror within each half row
// (lane i with 7 - i) and within the row (i with 15 - i).  Each step adds
// two equal-ordered partial sums, so all 16 lanes end with identical
// totals (branches on them stay uniform within the group).
__device__ __forceinline__ void group16_sum3(double& a, double& b, double& c) {
    constexpr int kXor1 = 0xB1, kXor2 = 0x4E, kHalfMirror = 0x141, kMirror = 0x140;
    a += dpp_f64<kXor1>(a); b += dpp_f64<kXor1>(b); c += dpp_f64<kXor1>(c);
    a += dpp_f64<kXor2>(a); b += dpp_f64<kXor2>(b); c += dpp_f64<kXor2>(c);
    a += dpp_f64<kHalfMirror>(a); b += dpp_f64<kHalfMirror>(b); c += dpp_f64<kHalfMirror>(c);
    a += dpp_f64<kMirror>(a); b += dpp_f64<kMirror>(b); c += dpp_f64<kMirror>(c);
}

// Move within quads of lanes: lane i receives the value of lane i ^ X.
template <int X>
__device__ __forceinline__ double quad_xor(double v) {
    return dpp_f64<X == 1 ? 0xB1 : X == 2 ? 0x4E : 0x1B>(v);
}

// Sum over the 16 lanes with equal lane & 3: rotations by 8 and 4 within
// rows of 16 lanes, then swaps of neighbouring rows and of the wave's halves.
// Every step adds two equal-ordered partial sums, so that the 16 lanes end
// with identical totals.
__device__ __forceinline__ double stride4_sum(double x) {
    x += dpp_f64<0x128>(x);
    x += dpp_f64<0x124>(x);
    {
        const long long b = __builtin_bit_cast(long long, x);
        const auto lo = __builtin_amdgcn_permlane16_swap((unsigned)b, (unsigned)b, false, false);
        const auto hi = __builtin_amdgcn_permlane16_swap((unsigned)(b >> 32), (unsigned)(b >> 32), false, false);
        x = __builtin_bit_cast(double, ((unsigned long long)hi[0] << 32) | lo[0]) +
            __builtin_bit_cast(double, ((unsigned long long)hi[1] << 32) | lo[1]);
    }
    const long long b = __builtin_bit_cast(long long, x);
    const auto lo = __builtin_amdgcn_permlane32_swap((unsigned)b, (unsigned)b, false, false);
    const auto hi = __builtin_amdgcn_permlane32_swap((unsigned)(b >> 32), (unsigned)(b >> 32), false, false);
    return __builtin_bit_cast(double, ((unsigned long long)hi[0] << 32) | lo[0]) +
           __builtin_bit_cast(double, ((unsigned long long)hi[1] << 32) | lo[1]);
}

// A column's share of a lane: entries e0 + 16 u of m_j and of z_j, and |m_j|^2.
template <int PER>
struct JacCol {
    double m[PER], z[PER], nn;
    __device__ __forceinline__ void load(const double* mc, const double* jc) {
#pragma unroll
        for (int u = 0; u < PER; ++u) {
            m[u] = mc[16 * u];
            z[u] = jc[16 * u];
        }
        nn = stride4_sum(dot(*this));
    }
    __device__ __forceinline__ void store(double* mc, double* jc) const {
#pragma unroll
        for (int u = 0; u < PER; ++u) {
            mc[16 * u] = m[u];
            jc[16 * u] = z[u];
        }
    }
    __device__ __forceinline__ double dot(const JacCol& o) const {
        double x = 0.0;
#pragma unroll
        for (int u = 0; u < PER; ++u) x = __builtin_fma(m[u], o.m[u], x);
        return x;
    }
    template <int X>
    __device__ __forceinline__ JacCol moved() const {
        JacCol r;
#pragma unroll
        for (int u = 0; u < PER; ++u) {
            r.m[u] = quad_xor<X>(m[u]);
            r.z[u] = quad_xor<X>(z[u]);
        }
        r.nn = quad_xor<X>(nn);
        return r;
    }
    // this = c this + s o
    __device__ __forceinline__ void combine(double c, double s, const JacCol& o) {
#pragma unroll
        for (int u = 0; u < PER; ++u) {
            m[u] = c * m[u] + s * o.m[u];
            z[u] = c * z[u] + s * o.z[u];
        }
    }
};

// Pair (a, b) of a lane's quarter of the wave, a before b.
template <int PER>
__device__ __forceinline__ bool jac_cross(JacCol<PER>& a, JacCol<PER>& b, double tol) {
    double t, c, s;
    const double ga = stride4_sum(a.dot(b));
    const bool rot = jac_rotation(a.nn, b.nn, ga, tol, false, t, c, s);
    const JacCol<PER> a0 = a;   // applied without a branch: one would cost copies of all columns
    a.combine(c, -s, b);
    b.combine(c, s, a0);
    a.nn = __builtin_fma(-t, ga, a.nn);
    b.nn = __builtin_fma(t, ga, b.nn);
    return __builtin_amdgcn_ballot_w64(rot) != 0;
}

// Pairs of the columns of one block, (q, q ^ X) for q = lane & 3: both lanes
// of a pair form the same rotation and update their own column.
template <int PER, int X>
__device__ __forceinline__ bool jac_inside(JacCol<PER>& a, bool second, double tol) {
    double t, c, s;
    const JacCol<PER> o = a.template moved<X>();
    const double ga = stride4_sum(a.dot(o));
    const bool rot = jac_rotation(a.nn, o.nn, ga, tol, second, t, c, s);
    a.combine(c, -s, o);
    a.nn = __builtin_fma(-t, ga, a.nn);
    return __builtin_amdgcn_ballot_w64(rot) != 0;
}

// One workgroup: SVD of M = R^T (R upper triangular, l x l inside pitch ldr)
// by one-sided (Hestenes) Jacobi.  The columns of M (rows of R) and of the
// accumulated rotation Z sit in LDS, the columns first put in non-increasing
// order of their norms (de Rijk's ordering).  A pair (p, q) is rotated when
// |m_p . m_q| > tol ||m_p|| ||m_q||, tol = max(l, 8) 2^-53, by the rotation
// that makes the two columns orthogonal.  A sweep visits every pair once,
// by blocks of four columns: in each of nb - 1 rounds of the round-robin
// (circle) ordering of the nb blocks (rounded up to even; columns past l are
// zero) a wave takes two blocks into registers, four columns of each on the
// four residues of lane & 3, rotates the 16 pairs across them in four steps
// (the second block moves one residue on within quads), and puts them back;
// one barrier per round.  Round 0 begins with the pairs inside the blocks.
// Norms are summed when a block is loaded and updated by its rotations.  The
// sweeps stop when one rotates nothing (all its norms are then the summed
// ones); *flag = 1 if 40 sweeps do not get there.  Then sigma_j = ||m_j||,
// and the columns are written in non-increasing order of sigma (ties by
// index): sv[pos] = sigma, Wt[pos][:] = m_j / sigma_j (zero when sigma_j =
// 0), Zt[pos][:] = z_j, and, when Zts is not null, Zts[pos][:] = sigma_j z_j;
// rows of pitch ldw with zeros in columns l..ldw-1; s_out[pos] = sigma for
// pos < k when not null.
// Bound by the issue of one compute unit and the chain dot - rotation -
// update of a step: a sweep is 8 ceil(l / 8) + 2 steps, and sketches with decaying
// spectra take 7 (l = 16) to 9 sweeps.  A round per column pair, with IEEE
// divisions and a trip through LDS each, took 1006 us at l = 74 (8 sweeps), this
// takes 601.
constexpr int kJacPitch = 104;   // doubles: four neighbouring columns fall on distinct banks
constexpr int kJacThreads = 64 * (kFactMaxL / 8);
static_assert(kFactMaxL % 16 == 0 && kFactMaxL <= kJacPitch, "blocks of the largest sketch");
template <int PER>
__global__ __launch_bounds__(kJacThreads) void k_fact_jacobi(const double* __restrict__ R, int l, int ldr, int k,
                                                             double* __restrict__ sv, double* __restrict__ s_out,
                                                             double* __restrict__ Wt, double* __restrict__ Zt,
                                                             double* __restrict__ Zts, int ldw, int* __restrict__ flag) {
    __shared__ double Mc[16 * PER][kJacPitch];
    __shared__ double Jc[16 * PER][kJacPitch];
    __shared__ double sig[16 * PER];
    __shared__ int pos[16 * PER];
    __shared__ int rotated[kJacSweeps];
    const int tid = threadIdx.x, nth = blockDim.x;
    const int grp = tid >> 4, gl = tid & 15;
    // columns of M = R^T (rows of R) placed in non-increasing order of their
    // norms (ties by index), which shortens the sweeps; the rotation
    // accumulator starts as that permutation
    for (int j = grp; j < l; j += nth / 16) {
        double x = 0.0, y = 0.0, z = 0.0;
#pragma unroll
        for (int u = 0; u < PER; ++u) {
            const int e = gl + 16 * u;
            const double v = (e < l && e >= j) ? R[(int64_t)j * ldr + e] : 0.0;
            x += v * v;
        }
        group16_sum3(x, y, z);
        if (gl == 0) sig[j] = x;
    }
    for (int i = tid; i < kJacSweeps; i += nth) rotated[i] = 0;
    __syncthreads();
    for (int j = tid; j < l; j += nth) {
        const double sj = sig[j];
        int c = 0;
        for (int i = 0; i < l; ++i) c += (sig[i] > sj || (sig[i] == sj && i < j)) ? 1 : 0;
        pos[j] = c;
    }
    __syncthreads();
    for (int idx = tid; idx < 256 * PER * PER; idx += nth) {
        const int j = idx / (16 * PER), i = idx - j * (16 * PER);
        const int pj = j < l ? pos[j] : j;
        Mc[pj][i] = (j < l && i < l && i >= j) ? R[(int64_t)j * ldr + i] : 0.0;
        Jc[pj][i] = (j < l && i == j) ? 1.0 : 0.0;
    }
    __syncthreads();
    const int nb = nth / 32;   // blocks of four columns, two per wave
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6), q = tid & 3, e0 = (tid & 63) >> 2;
    const double tol = (double)(l > 8 ? l : 8) * 0x1p-53;
    bool converged = false;
    for (int sweep = 0; sweep < kJacSweeps; ++sweep) {
        bool any = false;
        for (int t = 0; t + 1 < nb; ++t) {
            int x = t, y = nb - 1;
            if (wave > 0) {
                x = t + wave;
                x = x >= nb - 1 ? x - (nb - 1) : x;
                y = t - wave;
                y = y < 0 ? y + (nb - 1) : y;
            }
            const int pa = 4 * (x < y ? x : y), pb = 4 * (x < y ? y : x);
            JacCol<PER> a, b;
            a.load(&Mc[pa + q][e0], &Jc[pa + q][e0]);
            b.load(&Mc[pb + q][e0], &Jc[pb + q][e0]);
            if (t == 0) {
                any |= jac_inside<PER, 1>(a, (q & 1) != 0, tol);
                any |= jac_inside<PER, 1>(b, (q & 1) != 0, tol);
                any |= jac_inside<PER, 2>(a, (q & 2) != 0, tol);
                any |= jac_inside<PER, 2>(b, (q & 2) != 0, tol);
                any |= jac_inside<PER, 3>(a, (q & 2) != 0, tol);
                any |= jac_inside<PER, 3>(b, (q & 2) != 0, tol);
            }
            any |= jac_cross(a, b, tol);
            b = b.template moved<1>();
            any |= jac_cross(a, b, tol);
            b = b.template moved<3>();
            any |= jac_cross(a, b, tol);
            b = b.template moved<1>();
            any |= jac_cross(a, b, tol);
            a.store(&Mc[pa + q][e0], &Jc[pa + q][e0]);
            b.store(&Mc[pb + (q ^ 3)][e0], &Jc[pb + (q ^ 3)][e0]);
            if (t + 2 == nb && any && (tid & 63) == 0) rotated[sweep] = 1;
            __syncthreads();
        }
        if (!rotated[sweep]) {
            converged = true;
            break;
        }
    }
    if (tid == 0 && !converged) *flag = 1;
    // singular values: one group of 16 lanes per column
    for (int j = grp; j < l; j += nth / 16) {
        double x = 0.0, y = 0.0, z = 0.0;
#pragma unroll
        for (int u = 0; u < PER; ++u) {
            const double v = Mc[j][gl + 16 * u];
            x += v * v;
        }
        group16_sum3(x, y, z);
        if (gl == 0) sig[j] = __builtin_sqrt(x);
    }
    __syncthreads();
    for (int j = tid; j < l; j += nth) {
        const double sj = sig[j];
        int c = 0;
        for (int i = 0; i < l; ++i) c += (sig[i] > sj || (sig[i] == sj && i < j)) ? 1 : 0;
        pos[j] = c;
        sv[c] = sj;
        if (s_out && c < k) s_out[c] = sj;
    }
    __syncthreads();
    for (int idx = tid; idx < l * ldw; idx += nth) {
        const int j = idx / ldw, e = idx - j * ldw;
        const double sj = sig[j];
        const int64_t o = (int64_t)pos[j] * ldw + e;
        const double m = e < l ? Mc[j][e] : 0.0, z = e < l ? Jc[j][e] : 0.0;
        Wt[o] = sj > 0.0 ? m / sj : 0.0;
        Zt[o] = z;
        if (Zts) Zts[o] = sj * z;
    }
}

template <int PER>
static void launch_jacobi(const double* R, int l, int ldr, int k, double* sv, double* s_out, double* Wt, double* Zt,
                          double* Zts, int* flag, hipStream_t st) {
    if constexpr (PER < kFactMaxL / 16) {
        if (l > 16 * PER)
            return launch_jacobi<PER + 1>(R, l, ldr, k, sv, s_out, Wt, Zt, Zts, flag, st);
    }
    hipLaunchKernelGGL(k_fact_jacobi<PER>, dim3(1), dim3(64 * ((l + 7) / 8)), 0, st, R, l, ldr, k, sv, s_out, Wt, Zt,
                       Zts, ldr, flag);
}

static unsigned fact_grid(int64_t items) {
    int64_t g = (items + 255) / 256;
    if (g > 8192) g = 8192;
    return (unsigned)(g < 1 ? 1 : g);
}

static size_t r256(int64_t bytes) { return (size_t)round_up(bytes, 256); }

size_t rsvd_workspace_bytes(int64_t m, int64_t n, int l, int k, int q, bool vts) {
    const int64_t rp = round_up(l, 2), ldn = round_up(n, 2);
    size_t keep = 2 * r256(m * rp * 8) + 2 * r256(n * rp * 8) + 4 * r256(rp * rp * 8) + r256(rp * 8);
    if (q > 0) keep += r256(rp * ldn * 8);
    size_t tmp = gemm_nt_workspace_bytes(l, m, n);
    tmp = std::max(tmp, gemm_tn_workspace_bytes(l, n, m));
    tmp = std::max(tmp, cholqr2_workspace_bytes(m, l));
    tmp = std::max(tmp, cholqr2_workspace_bytes(n, l));
    tmp = std::max(tmp, gemm_nt_workspace_bytes(k, m, l));
    tmp = std::max(tmp, gemm_nt_workspace_bytes(k, n, l));
    if (vts) tmp = std::max(tmp, gemm_nt_workspace_bytes(n, k, l));
    return keep + tmp + 4096;
}

// A (m x n, pitch lda) and Omega (l x n, pitch ldo): 16-byte aligned, even
// pitches.  Outputs (any that are null are skipped): U (m x k, pitch ldu),
// s_out (k), V (n x k, pitch ldv), Vts = diag(s) V^T (k x n, pitch ldvt).
// flags[0]: range finder QR, flags[1]: QR of B^T, flags[2]: Jacobi.
// shifted: every orthonormalization by shifted CholeskyQR3 instead of
// CholeskyQR2 (for sketches with condition numbers between about 1e7 and
// 1e15; half as much QR work again).
hipError_t launch_rsvd(const double* A, int64_t m, int64_t n, int64_t lda, const double* Om, int64_t ldo, int l,
                       int q, int k, double* U, int64_t ldu, double* s_out, double* V, int64_t ldv, double* Vts,
                       int64_t ldvt, int* flags, Workspace& ws, hipStream_t st, bool shifted) {
    const int rp = (int)round_up(l, 2);
    const int64_t ldn = round_up(n, 2);
    double* Y = static_cast<double*>(ws.take((size_t)m * rp * 8));
    double* Q = static_cast<double*>(ws.take((size_t)m * rp * 8));
    double* Bt = static_cast<double*>(ws.take((size_t)n * rp * 8));
    double* Q2 = static_cast<double*>(ws.take((size_t)n * rp * 8));
    double* R = static_cast<double*>(ws.take((size_t)rp * rp * 8));
    double* Wt = static_cast<double*>(ws.take((size_t)rp * rp * 8));
    double* Zt = static_cast<double*>(ws.take((size_t)rp * rp * 8));
    double* Zs = static_cast<double*>(ws.take((size_t)rp * rp * 8));
    double* sv = static_cast<double*>(ws.take((size_t)rp * 8));
    double* Qzt = q > 0 ? static_cast<double*>(ws.take((size_t)rp * ldn * 8)) : nullptr;
    if (ws.overrun) return hipErrorOutOfMemory;
    const size_t mark = ws.used;
    hipError_t e;
#define LRC_STEP(call)                     \
    do {                                   \
        e = (call);                        \
        if (e != hipSuccess) return e;     \
        ws.used = mark;                    \
    } while (0)
    LRC_STEP(launch_gemm_nt(Om, ldo, l, A, lda, m, n, nullptr, Y, rp, rp, ws, st, "factor_sketch_f64"));
    LRC_STEP(launch_cholqr2(Y, m, l, Q, nullptr, flags, ws, st, "factor_cholqr2_f64", shifted));
    for (int it = 0; it < q; ++it) {
        LRC_STEP(launch_gemm_tn(Q, rp, l, A, lda, n, m, Bt, rp, rp, ws, st, "factor_project_f64",
                                "factor_project_finish_f64"));
        LRC_STEP(launch_cholqr2(Bt, n, l, Q2, nullptr, flags, ws, st, "factor_cholqr2_f64", shifted));
        {
            KernelTimer tm("factor_transpose_f64", st);
            hipLaunchKernelGGL(k_fact_transpose, dim3((unsigned)((ldn + 31) / 32), (unsigned)((rp + 31) / 32)),
                               dim3(256), 0, st, Q2, n, (int64_t)rp, (int64_t)rp, Qzt, ldn);
        }
        LRC_STEP(launch_gemm_nt(Qzt, ldn, l, A, lda, m, n, nullptr, Y, rp, rp, ws, st, "factor_sketch_f64"));
        LRC_STEP(launch_cholqr2(Y, m, l, Q, nullptr, flags, ws, st, "factor_cholqr2_f64", shifted));
    }
    LRC_STEP(launch_gemm_tn(Q, rp, l, A, lda, n, m, Bt, rp, rp, ws, st, "factor_project_f64",
                            "factor_project_finish_f64"));
    LRC_STEP(launch_cholqr2(Bt, n, l, Q2, R, flags + 1, ws, st, "factor_cholqr2_f64", shifted));
    {
        KernelTimer tm("factor_jacobi_f64", st);
        launch_jacobi<1>(R, l, rp, k, sv, s_out, Wt, Zt, Vts ? Zs : nullptr, flags + 2, st);
    }
    if (U) LRC_STEP(launch_gemm_nt(Wt, rp, k, Q, rp, m, l, nullptr, U, ldu, k, ws, st, "factor_vectors_f64"));
    if (V) LRC_STEP(launch_gemm_nt(Zt, rp, k, Q2, rp, n, l, nullptr, V, ldv, k, ws, st, "factor_vectors_f64"));
    if (Vts) LRC_STEP(launch_gemm_nt(Q2, rp, n, Zs, rp, k, l, nullptr, Vts, ldvt, n, ws, st, "factor_vectors_f64"));
#undef LRC_STEP
    return hipGetLastError();
}

// Padded copy (rows x cols -> rows x even pitch) when the source is not fit
// for 16-byte moves; returns the pointer and pitch to use.
static hipError_t fit(const double* src, int64_t rows, int64_t cols, Workspace& ws, hipStream_t st,
                      const double** out, int64_t* ld) {
    if (cols % 2 == 0 && reinterpret_cast<uintptr_t>(src) % 16 == 0) {
        *out = src;
        *ld = cols;
        return hipSuccess;
    }
    const int64_t p = round_up(cols, 2);
    double* d = static_cast<double*>(ws.take((size_t)rows * p * 8));
    if (ws.overrun) return hipErrorOutOfMemory;
    KernelTimer tm("factor_pad_f64", st);
    hipLaunchKernelGGL(k_fact_pad, dim3(fact_grid(rows * p)), dim3(256), 0, st, src, rows, cols, cols, d, rows, p);
    *out = d;
    *ld = p;
    return hipGetLastError();
}

static size_t fit_bytes(int64_t rows, int64_t cols) { return r256(rows * round_up(cols, 2) * 8); }

size_t matrix_rsvd_workspace_bytes(int64_t m, int64_t n, int l, int k, int q) {
    return 3 * 256 + fit_bytes(m, n) + fit_bytes(l, n) + rsvd_workspace_bytes(m, n, l, k, q, false);
}

hipError_t launch_matrix_rsvd(const double* A, int64_t m, int64_t n, const double* Om, int l, int q, int k, double* U,
                              double* s, double* V, int* flags, Workspace& ws, hipStream_t st, bool shifted) {
    hipLaunchKernelGGL(k_fact_zero, dim3(1), dim3(64), 0, st, flags, 3);
    const double *Af, *Of;
    int64_t lda, ldo;
    hipError_t e = fit(A, m, n, ws, st, &Af, &lda);
    if (e == hipSuccess) e = fit(Om, l, n, ws, st, &Of, &ldo);
    if (e != hipSuccess) return e;
    return launch_rsvd(Af, m, n, lda, Of, ldo, l, q, k, U, k, s, V, k, nullptr, 0, flags, ws, st, shifted);
}

// TT-SVD, step l of d - 1: C_l ((r_{l-1} n_l) x prod_{i>l} n_i) -> core l =
// U (pitch r_l), C_{l+1} = diag(s) V^T (r_l x cols, contiguous, which is
// C_{l+1} reshaped); the last step writes diag(s) V^T into the last core.
size_t tt_rsvd_workspace_bytes(const int64_t* dims, const int64_t* ranks, const int64_t* samples, int d, int q) {
    size_t need = 0, cbuf = 0;
    int64_t cols = 1;
    for (int i = 1; i < d; ++i) cols *= dims[i];
    for (int l = 0; l + 1 < d; ++l) {
        const int64_t rows = ranks[l] * dims[l];
        size_t b = fit_bytes(rows, cols) + fit_bytes(samples[l], cols) +
                   rsvd_workspace_bytes(rows, cols, (int)samples[l], (int)ranks[l + 1], q, true);
        need = std::max(need, b);
        if (l + 2 < d) cbuf = std::max(cbuf, r256(ranks[l + 1] * cols * 8));
        cols /= dims[l + 1];
    }
    return need + 2 * cbuf + r256(4 * 3 * (int64_t)d) + 1024;
}

hipError_t launch_tt_rsvd(const double* T, const int64_t* dims, const int64_t* ranks, const int64_t* samples, int d,
                          const double* const* omegas, int q, double* const* cores, double* sigma, int* flags,
                          Workspace& ws, hipStream_t st, bool shifted) {
    hipLaunchKernelGGL(k_fact_zero, dim3(1), dim3(64), 0, st, flags, 3 * (d - 1));
    int64_t cols = 1;
    for (int i = 1; i < d; ++i) cols *= dims[i];
    size_t cbuf = 0;
    {
        int64_t c = cols;
        for (int l = 0; l + 2 < d; ++l) {
            cbuf = std::max(cbuf, (size_t)(ranks[l + 1] * c * 8));
            c /= dims[l + 1];
        }
    }
    double* Cb[2] = {nullptr, nullptr};
    if (cbuf) {
        Cb[0] = static_cast<double*>(ws.take(cbuf));
        Cb[1] = static_cast<double*>(ws.take(cbuf));
        if (ws.overrun) return hipErrorOutOfMemory;
    }
    const double* C = T;
    int64_t soff = 0;
    for (int l = 0; l + 1 < d; ++l) {
        const int64_t rows = ranks[l] * dims[l];
        const int r = (int)ranks[l + 1];
        const bool last = l + 2 == d;
        double* next = last ? cores[d - 1] : Cb[l & 1];
        const size_t mark = ws.used;
        const double *Af, *Of;
        int64_t lda, ldo;
        hipError_t e = fit(C, rows, cols, ws, st, &Af, &lda);
        if (e == hipSuccess) e = fit(omegas[l], samples[l], cols, ws, st, &Of, &ldo);
        if (e == hipSuccess)
            e = launch_rsvd(Af, rows, cols, lda, Of, ldo, (int)samples[l], q, r, cores[l], r,
                            sigma ? sigma + soff : nullptr, nullptr, 0, next, cols, flags + 3 * l, ws, st, shifted);
        if (e != hipSuccess) return e;
        ws.used = mark;
        soff += r;
        C = next;
        cols /= dims[l + 1];
    }
    return hipSuccess;
}

}  // namespace lrc
