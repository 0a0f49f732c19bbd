// Small applies in one launch; part of apply.hip.
//
// The smallest calls are bound by their launches: phase 1, the sum of its
// splits and phase 2 take 3 to 6 us each on the device and as much on the
// host.  Here a workgroup forms the T' columns that it needs itself (V is read
// again by every row block, X by every row block too, all from the L2) and
// multiplies them with its 64 rows of U.  512 x 256, k = 20, batch 64: 14.7 ->
// 6.9 us a call in FP64, 12.6 -> 7.0 us in FP32, where the binding's own 6.5 us
// are the bound.  binary16 operands are widened to FP32 (exact) and take the FP32
// instruction, whose rate does not matter at these sizes.
#pragma once

template <typename T> struct SmallAcc { using type = float; };
template <> struct SmallAcc<double> { using type = double; };

constexpr int kSmallTile = 32;      // rank indices formed at a time
constexpr int kSmallBatch = 8;      // K steps of 4 rows whose loads are issued together
constexpr int kSmallWaves = 8;
constexpr int kSmallMaxK = 128;

// LDS pitch of K-contiguous rows: 4 times an odd number, so that the 64 lanes
// of a fragment read (16 rows, 4 K values) fall on distinct banks.
__host__ __device__ constexpr int small_pitch(int k) { return 4 * (((k + 3) / 4) | 1); }

// acc[f] += sum over rows i in [i0, i1) of V[i][k0 + 16 f + .] X[i][n0 + .]
// (i0, i1 uniform).  Whole batches of 4 BT rows take uniform row addresses
// and constant lane offsets, so that issuing their loads costs no vector
// arithmetic.
template <typename T>
__device__ __forceinline__ void small_rows(const T* __restrict__ V, int64_t k, int64_t k0, const T* __restrict__ X,
                                           int64_t b, int64_t n0, int64_t i0, int64_t i1, int lane,
                                           typename PrecTraits<typename SmallAcc<T>::type>::accv (&acc)[2]) {
    constexpr int BT = kSmallBatch;
    using Acc = typename SmallAcc<T>::type;
    const int r = lane & 15, g = lane >> 4;
    unsigned mc[2];
#pragma unroll
    for (int f = 0; f < 2; ++f) mc[f] = (unsigned)std::min(k0 + 16 * f + r, k - 1);
    const unsigned nc = (unsigned)std::min(n0 + r, b - 1);
    const unsigned gk = (unsigned)(g * k), gb = (unsigned)(g * b);
    T va[BT][2], xa[BT];
    int64_t ib = i0;
    for (; ib + 4 * BT <= i1; ib += 4 * BT) {
#pragma unroll
        for (int t = 0; t < BT; ++t) {
            const T *vr = V + (ib + 4 * t) * k, *xr = X + (ib + 4 * t) * b;
#pragma unroll
            for (int f = 0; f < 2; ++f) va[t][f] = vr[gk + mc[f]];
            xa[t] = xr[gb + nc];
        }
#pragma unroll
        for (int t = 0; t < BT; ++t)
#pragma unroll
            for (int f = 0; f < 2; ++f) acc[f] = mfma((Acc)va[t][f], (Acc)xa[t], acc[f]);
    }
    if (ib >= i1) return;
#pragma unroll
    for (int t = 0; t < BT; ++t) {
        const int64_t i = std::min(ib + 4 * t + g, i1 - 1);
#pragma unroll
        for (int f = 0; f < 2; ++f) va[t][f] = V[i * k + mc[f]];
        xa[t] = X[i * b + nc];
    }
#pragma unroll
    for (int t = 0; t < BT; ++t) {
        const bool in = ib + 4 * t + g < i1;
#pragma unroll
        for (int f = 0; f < 2; ++f) acc[f] = mfma(in ? (Acc)va[t][f] : Acc(0), in ? (Acc)xa[t] : Acc(0), acc[f]);
    }
}

// Y rows [64 y, 64 y + 64) by columns [16 x, 16 x + 16).  The rows of U (KC =
// ceil(k / 64) loads per lane and row) are requested first; then T' = s * (V^T
// X), each wave summing an eighth of the rows and the waves added in order,
// goes to LDS rounded to T, 32 rank indices at a time; then the products, one
// 16 x 16 fragment per wave of the first four.
template <typename T, int KC>
__global__ __launch_bounds__(64 * kSmallWaves) void k_apply_small(
    const T* __restrict__ U, const T* __restrict__ s, const T* __restrict__ V, const T* __restrict__ X,
    T* __restrict__ Y, int64_t m, int64_t n, int64_t k, int64_t b, int vec4) {
    using Acc = typename SmallAcc<T>::type;
    using AccV = typename PrecTraits<Acc>::accv;
    constexpr int W = kSmallWaves, RP = kSmallTile + 1, PMAX = small_pitch(64 * KC);
    __shared__ alignas(16) Acc Us[64 * PMAX];       // [64][P]
    __shared__ alignas(16) Acc Ts[16 * PMAX];       // [16][P]
    __shared__ Acc red[W * 16 * RP];                // [wave][column][rank index]
    const int P = small_pitch((int)k);
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int r = lane & 15, g = lane >> 4;
    const int64_t m0 = (int64_t)blockIdx.y * 64, n0 = (int64_t)blockIdx.x * 16;
    T u[8][KC];
#pragma unroll
    for (int q = 0; q < 8; ++q) {
        const T* row = U + std::min(m0 + wave * 8 + q, m - 1) * k;
#pragma unroll
        for (int c = 0; c < KC; ++c) u[q][c] = row[std::min<int64_t>(c * 64 + lane, k - 1)];
    }
    const int64_t per = (n + W - 1) / W, i0 = std::min<int64_t>(wave * per, n), i1 = std::min(i0 + per, n);
    for (int64_t k0 = 0; k0 < k; k0 += kSmallTile) {
        AccV acc[2] = {zero_accv<AccV>(), zero_accv<AccV>()};
        small_rows<T>(V, k, k0, X, b, n0, i0, i1, lane, acc);
        if (k0 > 0) __syncthreads();                // the previous block has been summed
#pragma unroll
        for (int f = 0; f < 2; ++f)
#pragma unroll
            for (int v = 0; v < 4; ++v) red[(wave * 16 + r) * RP + f * 16 + acc_row<Acc>(g, v)] = acc[f][v];
        __syncthreads();
        const int c = tid / kSmallTile, j = tid % kSmallTile;
        Acc x = red[c * RP + j];
#pragma unroll
        for (int w = 1; w < W; ++w) x += red[(w * 16 + c) * RP + j];
        if (k0 + j < P) Ts[c * P + k0 + j] = k0 + j < k ? (Acc)to_storage<T>((Acc)s[k0 + j] * x) : Acc(0);
    }
#pragma unroll
    for (int q = 0; q < 8; ++q) {
        Acc* row = Us + (wave * 8 + q) * P;         // the products read up to k rounded to 4
#pragma unroll
        for (int c = 0; c < KC; ++c)
            if (c * 64 + lane < P) row[c * 64 + lane] = c * 64 + lane < k ? (Acc)u[q][c] : Acc(0);
    }
    __syncthreads();
    if (wave >= 4) return;
    AccV acc = zero_accv<AccV>();
    const Acc *up = Us + (wave * 16 + r) * P + g, *tp = Ts + r * P + g;
    const int ke = ((int)k + 3) & ~3;
    int t = 0;
    for (; t + 32 <= ke; t += 32) {
        Acc uv[8], tv[8];
#pragma unroll
        for (int e = 0; e < 8; ++e) {
            uv[e] = up[t + 4 * e];
            tv[e] = tp[t + 4 * e];
        }
#pragma unroll
        for (int e = 0; e < 8; ++e) acc = mfma(tv[e], uv[e], acc);
    }
    for (; t < ke; t += 4) acc = mfma(tp[t], up[t], acc);
    const int64_t mm = m0 + wave * 16 + r;
    if (mm >= m) return;
    if (AccRowsContiguous<Acc>::value && vec4 && n0 + 4 * g + 4 <= b) {
        typedef T v4_t __attribute__((ext_vector_type(4)));
        v4_t w;
#pragma unroll
        for (int v = 0; v < 4; ++v) w[v] = to_storage<T>(acc[v]);
        *reinterpret_cast<v4_t*>(Y + mm * b + n0 + 4 * g) = w;
    } else {
#pragma unroll
        for (int v = 0; v < 4; ++v) {
            const int64_t c = n0 + acc_row<Acc>(g, v);
            if (c < b) Y[mm * b + c] = to_storage<T>(acc[v]);
        }
    }
}

// Where one launch pays: its time grows with the serial part, the batches of 32
// rows per wave times the blocks of 32 rank indices, and with the workgroups
// past one per compute unit; up to 4 of these it takes 7 to 15 us against 13 to
// 25 (200 sizes with n <= 700, k <= 100, 9 <= b <= 1024 in each precision: 1.1 to
// 2.8 times); at 6 the two are even (1024 x 700, k = 64: 17.3 against 16.8 us),
// beyond it loses.
static bool small_takes(int64_t m, int64_t n, int64_t k, int64_t b) {
    if (k > kSmallMaxK || n > 2048 || m > 32768 || b > 8192) return false;
    const int64_t wgs = ((m + 63) / 64) * ((b + 15) / 16);
    const int64_t batches = ((n + kSmallWaves - 1) / kSmallWaves + 4 * kSmallBatch - 1) / (4 * kSmallBatch);
    return wgs <= 512 && batches * ((k + kSmallTile - 1) / kSmallTile) * ((wgs + 255) / 256) <= 4;
}

template <typename T>
static hipError_t small_apply(const T* U, const T* s, const T* V, const T* X, T* Y, int64_t m, int64_t n, int64_t k,
                              int64_t b, hipStream_t stream) {
    KernelTimer t(p2_mfma_label<T>(), stream);
    const dim3 g((unsigned)((b + 15) / 16), (unsigned)((m + 63) / 64));
    const int vec4 = (b % 4 == 0 && reinterpret_cast<uintptr_t>(Y) % 16 == 0) ? 1 : 0;
    if (k <= 64)
        hipLaunchKernelGGL((k_apply_small<T, 1>), g, dim3(64 * kSmallWaves), 0, stream, U, s, V, X, Y, m, n, k, b, vec4);
    else
        hipLaunchKernelGGL((k_apply_small<T, 2>), g, dim3(64 * kSmallWaves), 0, stream, U, s, V, X, Y, m, n, k, b, vec4);
    return hipGetLastError();
}
