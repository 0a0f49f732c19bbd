// FP32 apply by split products on the bfloat16 matrix cores; part of
// apply.hip (uses its tile loads, stores and orders).
//
// The FP32 matrix cores run at 157 TFLOP/s, the bfloat16 ones (with the same
// FP32 accumulators) at 2500.  A binary32 value x is the exact sum of three
// bfloat16 values, x1 = bf16(x), x2 = bf16(x - x1), x3 = x - x1 - x2 (24 bits =
// 8 + 8 + 8, each rounded to nearest, every difference exact), so
//   a b = a1 b1 + (a1 b2 + a2 b1) + (a1 b3 + a2 b2 + a3 b1) + dropped,
// |dropped| <= |a2 b3| + |a3 b2| + |a3 b3| <= 2.01 * 2^-24 |a b| and of either
// sign.  Six bfloat16 products stand for one FP32 product, with one rounding
// of the accumulator per 32 K values and term instead of one per 4.
// The split is exact for 2^-100 <= |x| < 2^62 and for 0.  Any other value (of V,
// U or T': marked by the kernel that writes the planes; of X: checked where it
// is split) sends the K step that it belongs to, of one wave's columns in phase
// 1 and of one tile in phase 2, to the FP32 instruction.  So do accumulators that
// are not finite with all their steps, and infinities, NaN, overflow and underflow
// come out as they do there.  8192 x 8192, k = 257, b = 4096 takes 212 us, 352 on
// the FP32 instruction throughout; with 1e-33 in 1e-5 of the values of X, V or U
// 221 to 225, in 1e-3 of them 298 (U) to 373 (V), in every value of X 472 (phase
// 1 runs its loop for nothing).
#pragma once

typedef __bf16 bf2_t __attribute__((ext_vector_type(2)));
typedef __bf16 bf8_t __attribute__((ext_vector_type(8)));
typedef float f2_t __attribute__((ext_vector_type(2)));
typedef unsigned u32x2_t __attribute__((ext_vector_type(2)));

constexpr int kX3BK = 32;           // K step: one bfloat16 MFMA
constexpr float kX3Min = 0x1p-100f, kX3Max = 0x1p62f;
constexpr int kX3A[6] = {2, 0, 1, 1, 0, 0}, kX3B[6] = {0, 2, 1, 0, 1, 0};   // terms, smallest first

// The packed parts of two values.
__device__ __forceinline__ void x3_split2(float a, float b, unsigned (&p)[3]) {
    p[0] = __builtin_bit_cast(unsigned, __builtin_convertvector((f2_t){a, b}, bf2_t));
    const float ra = a - __builtin_bit_cast(float, p[0] << 16);
    const float rb = b - __builtin_bit_cast(float, p[0] & 0xFFFF0000u);
    p[1] = __builtin_bit_cast(unsigned, __builtin_convertvector((f2_t){ra, rb}, bf2_t));
    const float qa = ra - __builtin_bit_cast(float, p[1] << 16);
    const float qb = rb - __builtin_bit_cast(float, p[1] & 0xFFFF0000u);
    p[2] = __builtin_bit_cast(unsigned, __builtin_convertvector((f2_t){qa, qb}, bf2_t));
}

// A value outside the split's range.
__device__ __forceinline__ bool x3_outside(float x) {
    const float a = __builtin_fabsf(x);
    return !(a < kX3Max) | ((a < kX3Min) & (a != 0.0f));   // no branches: loads stay together
}

// Range of the values split on the way: largest magnitude and smallest
// nonzero one (as the value's bits, the sign shifted out, minus 1; zero
// wraps to the largest key).  The value itself decides, not its first part,
// which is zero for subnormals below 2^-134.
struct X3Range {
    float mx = 0.0f;
    unsigned mn = ~0u;
    __device__ __forceinline__ void add(float a, float b) {
        mx = __builtin_fmaxf(__builtin_fmaxf(mx, __builtin_fabsf(a)), __builtin_fabsf(b));
        mn = std::min(mn, std::min(__builtin_bit_cast(unsigned, a) * 2u - 1u, __builtin_bit_cast(unsigned, b) * 2u - 1u));
    }
    __device__ __forceinline__ bool bad() const {
        constexpr unsigned kKey = 2u * ((127u - 100u) << 23) - 1u;   // of 2^-100
        return !(mx < kX3Max) || mn < kKey;
    }
};

// Copies 16 bytes per lane from global memory straight into LDS: lane l's
// bytes land at lds + 16 l.  The caller waits (wait_loads, barrier) before
// reading them.
__device__ __forceinline__ void load_lds16(const void* g, void* lds) {
    __builtin_amdgcn_global_load_lds((const __attribute__((address_space(1))) void*)g,
                                     (__attribute__((address_space(3))) void*)lds, 16, 0, 0);
}
__device__ __forceinline__ void wait_loads() { asm volatile("s_waitcnt vmcnt(0)" ::: "memory"); }

// LDS tiles hold [rows][32] bfloat16 values per plane; the four 16-byte
// chunks of a row are XOR-swizzled by the row, so that eight neighbouring
// rows fall on distinct banks (counters: no conflicts).  A wave moves 16
// rows per load: lane l takes row l / 4 and the chunk that lives in slot l % 4.
__device__ __forceinline__ int x3_chunk(int lane) { return (lane & 3) ^ ((lane >> 3) & 3); }
__device__ __forceinline__ bf8_t x3_frag(const unsigned short* plane, int row0, int lane) {
    const int r = row0 + (lane & 15), c = (lane >> 4) ^ ((r >> 1) & 3);
    return *reinterpret_cast<const bf8_t*>(plane + r * kX3BK + c * 8);
}
__device__ __forceinline__ float4_t x3_mfma(bf8_t a, bf8_t b, float4_t c) {
    return __builtin_amdgcn_mfma_f32_16x16x32_bf16(a, b, c, 0, 0, 0);
}

// ---- planes of U and of V^T, one launch ----------------------------------------
// Workgroups [0, ublocks) write the planes of U (m x k, [m][ldk]), 256 chunks
// of 8 values each; the rest write those of V^T ([kpad][ldn] from V, n x k),
// a 64 x 64 tile each through LDS.  Both zero padded; any alignment.  Values
// outside the split's range: umask has one bit per chunk of U, vflag four bytes
// (one per wave) per 32 rows, one K step, of a tile of V.
// Bound by their 10 bytes per value: 65536 x 513 and 4096 x 513 in 62 us (5.8 TB/s).
__global__ __launch_bounds__(256) void k_x3_planes(const float* __restrict__ U, int64_t m, int64_t k,
                                                   unsigned short* __restrict__ Up, int64_t ldk, unsigned ublocks,
                                                   const float* __restrict__ V, int64_t n,
                                                   unsigned short* __restrict__ Vp, int64_t ldn, int64_t kpad,
                                                   unsigned ntiles, unsigned long long* __restrict__ umask,
                                                   unsigned char* __restrict__ vflag) {
    __shared__ float tile[64][65];
    const int tid = threadIdx.x;
    float v[8];
    if (blockIdx.x < ublocks) {
        const int64_t c = (int64_t)blockIdx.x * 256 + tid, cpr = ldk / 8, i = std::min(c / cpr, m - 1);
        const int64_t j0 = (c % cpr) * 8;
        const float* last = U + (m * k - 1);
        bool out = false;
#pragma unroll
        for (int h = 0; h < 2; ++h) {
            const int64_t j = j0 + 4 * h;
            MisChunk<float> mc;
            mc.fetch(U + i * k + (j < k ? j : k - 1), last);
            const float4_t w = mc.template value<float4_t>();
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                v[4 * h + q] = j + q < k ? w[q] : 0.0f;
                out |= x3_outside(v[4 * h + q]);
            }
        }
        if (c < m * cpr) {
            u32x4_t part[3];
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                unsigned p[3];
                x3_split2(v[2 * q], v[2 * q + 1], p);
#pragma unroll
                for (int t = 0; t < 3; ++t) part[t][q] = p[t];
            }
#pragma unroll
            for (int t = 0; t < 3; ++t) *reinterpret_cast<u32x4_t*>(Up + t * m * ldk + c * 8) = part[t];
        }
        const unsigned long long mask = __builtin_amdgcn_ballot_w64(out);
        if ((tid & 63) == 0) umask[c >> 6] = mask;
        return;
    }
    const unsigned b = blockIdx.x - ublocks;
    const int64_t n0 = (int64_t)(b % ntiles) * 64, k0 = (int64_t)(b / ntiles) * 64;
    const int tx = tid & 63, ty = tid >> 6;
    bool out[2] = {false, false};
#pragma unroll
    for (int u = 0; u < 16; ++u) {
        const int64_t i = n0 + ty + 4 * u, j = k0 + tx;
        const float x = V[(i < n ? i : n - 1) * k + (j < k ? j : k - 1)];
        tile[ty + 4 * u][tx] = (i < n && j < k) ? x : 0.0f;
        out[u / 8] |= x3_outside(x);   // past the edges: of the last row or column once more
    }
#pragma unroll
    for (int h = 0; h < 2; ++h) {
        const bool any = __builtin_amdgcn_ballot_w64(out[h]) != 0;
        if (tx == 0) vflag[8 * (int64_t)b + 4 * h + ty] = any ? 1 : 0;
    }
    __syncthreads();
#pragma unroll
    for (int e = 0; e < 2; ++e) {
        const int c = tid & 7, row = (tid >> 3) + 32 * e;    // 8 n values, rank index
        if (k0 + row >= kpad || n0 + 8 * c >= ldn) continue;
        u32x4_t part[3];
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            unsigned p[3];
            x3_split2(tile[8 * c + 2 * q][row], tile[8 * c + 2 * q + 1][row], p);
#pragma unroll
            for (int t = 0; t < 3; ++t) part[t][q] = p[t];
        }
#pragma unroll
        for (int t = 0; t < 3; ++t)
            *reinterpret_cast<u32x4_t*>(Vp + (t * kpad + k0 + row) * ldn + n0 + 8 * c) = part[t];
    }
}

// ---- phase 1 ---------------------------------------------------------------------
// Partial T'^T [split][b][kpad]: one workgroup of 4 waves per (rank tile of nf
// <= NF fragments, 128 columns of X, chunk of rows).  All waves read the V^T
// fragments from LDS (3 nf KB per K step of 32, moved there by direct loads);
// each wave keeps 32 columns of X (b columns at pitch ldx), loaded element by
// element along rows (64 contiguous bytes per 16 lanes, any pitch) and split
// in registers, so X is read and split once per rank tile and needs neither
// copy nor LDS.  Two workgroups per compute unit cover each other's load
// latency.  Bound by the matrix cores: 8192 x 8192, k = 257, b = 4096 runs in
// 96 us against 201 us on the FP32 instruction (split operands of both
// sides through LDS, 64 rank rows per tile: 191 us).  A wave leaves out the
// steps with a value outside the split's range and runs them after the loop on
// the FP32 instruction.
template <int NF>
__global__ __launch_bounds__(256, 2) void k_p1_x3(const unsigned short* __restrict__ Vp, int64_t ldn, int64_t kpad,
                                                  const float* __restrict__ V, int64_t k,
                                                  const float* __restrict__ X, int64_t ldx, int64_t n, int64_t b,
                                                  int64_t chunk, int nf, int tiles_m, int tiles_n, int splits,
                                                  const unsigned char* __restrict__ vflag,
                                                  float* __restrict__ part) {
    __shared__ alignas(16) unsigned short S[3 * NF * 16 * kX3BK];
    const int tid = threadIdx.x, lane = tid & 63, r = lane & 15, g = lane >> 4;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int64_t total = (int64_t)tiles_m * tiles_n * splits;
    const int64_t lt = xcd_tile(total);
    if (lt >= total) return;
    // rank tiles of the same columns and rows are neighbours, then column tiles
    const int64_t mt = lt % tiles_m, nt = (lt / tiles_m) % tiles_n, sp = lt / ((int64_t)tiles_m * tiles_n);
    const int64_t kbeg = sp * chunk, kend = std::min(kbeg + chunk, n);
    const int64_t mrow0 = mt * nf * 16;
    const int nsteps = (int)((kend - kbeg + kX3BK - 1) / kX3BK);

    const unsigned short* vp = Vp + (mrow0 + (lane >> 2)) * ldn + kbeg + x3_chunk(lane) * 8;
    auto move = [&](int j) {
        for (int t = wave; t < 3 * nf; t += 4) {
            const int q = t / nf, f = t - q * nf;
            load_lds16(vp + ((int64_t)q * kpad + f * 16) * ldn + (int64_t)j * kX3BK, S + (q * NF + f) * 16 * kX3BK);
        }
    };
    int64_t col[2];
    const float* xp[2];
#pragma unroll
    for (int h = 0; h < 2; ++h) {
        col[h] = nt * 128 + wave * 32 + h * 16 + r;
        xp[h] = X + (col[h] < b ? col[h] : b - 1);
    }
    // V's flags over this tile's ranks, four bytes per 64 ranks and step
    const int64_t kt0 = mrow0 >> 6, nkt = ((mrow0 + nf * 16 - 1) >> 6) - kt0 + 1;
    const int* vf = reinterpret_cast<const int*>(vflag) + (kt0 + (lane < nkt ? lane : 0)) * (((ldn + 63) >> 6) * 2);
    float xr[2][8];
    int flag;
    auto fetch = [&](int j) {
        const int64_t row0 = kbeg + (int64_t)j * kX3BK + 8 * g;
        flag = vf[kbeg / kX3BK + j];
        if (kbeg + (int64_t)(j + 1) * kX3BK <= n) {
#pragma unroll
            for (int h = 0; h < 2; ++h)
#pragma unroll
                for (int i = 0; i < 8; ++i) xr[h][i] = xp[h][(row0 + i) * ldx];
        } else {   // rows past n meet zeros of V^T; read the last row
#pragma unroll
            for (int h = 0; h < 2; ++h)
#pragma unroll
                for (int i = 0; i < 8; ++i) xr[h][i] = xp[h][(row0 + i < n ? row0 + i : n - 1) * ldx];
        }
    };
    float4_t acc[2][NF];
#pragma unroll
    for (int h = 0; h < 2; ++h)
#pragma unroll
        for (int f = 0; f < NF; ++f) acc[h][f] = zero_accv<float4_t>();
    unsigned left = 0;   // steps left out of the loop: bit j % 32 of lane j / 32
    move(0);
    fetch(0);
    for (int j = 0; j < nsteps; ++j) {
        wait_loads();
        __syncthreads();
        bf8_t v[2][3];   // fragment f and, read under its products, f + 1
#pragma unroll
        for (int q = 0; q < 3; ++q) v[0][q] = x3_frag(S + q * NF * 16 * kX3BK, 0, lane);
        X3Range range;
        bf8_t x[2][3];
#pragma unroll
        for (int h = 0; h < 2; ++h) {
            u32x4_t pk[3];
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                unsigned p[3];
                x3_split2(xr[h][2 * q], xr[h][2 * q + 1], p);
                range.add(xr[h][2 * q], xr[h][2 * q + 1]);
#pragma unroll
                for (int t = 0; t < 3; ++t) pk[t][q] = p[t];
            }
#pragma unroll
            for (int t = 0; t < 3; ++t) x[h][t] = __builtin_bit_cast(bf8_t, pk[t]);
        }
        const bool skip = __builtin_amdgcn_ballot_w64(flag != 0 || range.bad()) != 0;
        if (skip && lane == (j >> 5)) left |= 1u << (j & 31);
        if (j + 1 < nsteps) fetch(j + 1);
        if (!skip) {
#pragma unroll
            for (int f = 0; f < NF; ++f) {
                if (f < nf) {
                    if (f + 1 < NF) {
#pragma unroll
                        for (int q = 0; q < 3; ++q)
                            v[(f + 1) & 1][q] = x3_frag(S + q * NF * 16 * kX3BK, (f + 1) * 16, lane);
                    }
#pragma unroll
                    for (int t = 0; t < 6; ++t)
#pragma unroll
                        for (int h = 0; h < 2; ++h) acc[h][f] = x3_mfma(v[f & 1][kX3A[t]], x[h][kX3B[t]], acc[h][f]);
                }
            }
        }
        __syncthreads();
        if (j + 1 < nsteps) move(j + 1);
    }
    // The steps left out, on the FP32 instruction, operands straight from
    // memory: V requested one row per lane group ahead of its products, X four,
    // also from one step to the next.  Where the sums are not finite, all steps
    // once more that way.
    const unsigned m1 = (unsigned)(mrow0 + r), mk = (unsigned)(k - 1);
    for (bool all = false;;) {
        int word = -1;
        unsigned bits = 0;
        auto next = [&]() -> int64_t {   // first row of the next step left out, or -1
            while (bits == 0) {
                if (++word * 32 >= nsteps) return -1;
                bits = __builtin_amdgcn_readlane(left, word);
            }
            const int j = word * 32 + __builtin_ctz(bits);
            bits &= bits - 1;
            return kbeg + (int64_t)j * kX3BK;
        };
        float vn[NF], xn[4][2];
        auto get_v = [&](int64_t row) {
            const float* p = V + (row < n ? row : n - 1) * k;
#pragma unroll
            for (int f = 0; f < NF; ++f)   // ranks past k: sums that nothing reads
                if (f < nf) vn[f] = p[std::min(m1 + f * 16, mk)];
        };
        auto get_x = [&](int u, int64_t row) {
#pragma unroll
            for (int h = 0; h < 2; ++h) xn[u][h] = xp[h][(row < n ? row : n - 1) * ldx];
        };
        int64_t cur = next();
        if (cur >= 0) {
            get_v(cur + g);
#pragma unroll
            for (int u = 0; u < 4; ++u) get_x(u, cur + 4 * u + g);
        }
        while (cur >= 0) {
            const int64_t nxt = next(), nb = nxt >= 0 ? nxt : cur;
#pragma clang loop unroll(disable)
            for (int half = 0; half < 2; ++half) {
                const int64_t here = cur + 16 * half, then = half == 0 ? cur + 16 : nb;
#pragma unroll
                for (int u = 0; u < 4; ++u) {
                    const bool in = here + 4 * u + g < n;
                    float vc[NF], xc[2];
#pragma unroll
                    for (int f = 0; f < NF; ++f) vc[f] = in ? vn[f] : 0.0f;
#pragma unroll
                    for (int h = 0; h < 2; ++h) xc[h] = in ? xn[u][h] : 0.0f;
                    get_v((u < 3 ? here + 4 * (u + 1) : then) + g);
                    get_x(u, then + 4 * u + g);
#pragma unroll
                    for (int f = 0; f < NF; ++f) {
                        if (f < nf) {
                            acc[0][f] = mfma(vc[f], xc[0], acc[0][f]);
                            acc[1][f] = mfma(vc[f], xc[1], acc[1][f]);
                        }
                    }
                }
            }
            cur = nxt;
        }
        bool bad = false;
#pragma unroll
        for (int h = 0; h < 2; ++h)
#pragma unroll
            for (int f = 0; f < NF; ++f)
#pragma unroll
                for (int v = 0; v < 4; ++v) bad = bad || !(__builtin_fabsf(acc[h][f][v]) < __builtin_inff());
        if (__builtin_amdgcn_ballot_w64(bad) == 0 || all) break;
#pragma unroll
        for (int h = 0; h < 2; ++h)
#pragma unroll
            for (int f = 0; f < NF; ++f) acc[h][f] = zero_accv<float4_t>();
        const int mine = nsteps - 32 * lane;
        left = mine >= 32 ? ~0u : mine > 0 ? (1u << mine) - 1u : 0u;
        all = true;
    }
#pragma unroll
    for (int h = 0; h < 2; ++h) {
        if (col[h] >= b) continue;
        float* dst = part + (sp * b + col[h]) * kpad + mrow0 + 4 * g;
#pragma unroll
        for (int f = 0; f < NF; ++f)
            if (f < nf) *reinterpret_cast<float4_t*>(dst + f * 16) = acc[h][f];
    }
}

// T'^T[c][j] = s_j * (sum of the split partials in split order), as FP32
// (pitch ldt) and as planes (pitch ldk), zeros for j >= k: one thread per four
// consecutive j.  tmask: one bit per thread, set for a value outside the split's
// range.
__global__ __launch_bounds__(256) void k_x3_finish(const float* __restrict__ part, int64_t kpad, int splits,
                                                   const float* __restrict__ s, int64_t k, int64_t b,
                                                   float* __restrict__ Tt, int64_t ldt,
                                                   unsigned short* __restrict__ Tp, int64_t ldk,
                                                   unsigned long long* __restrict__ tmask) {
    const int64_t per = ldk / 4, idx = (int64_t)blockIdx.x * 256 + threadIdx.x;
    const int64_t c = idx / per, j = (idx - c * per) * 4;
    float4_t sum = zero_accv<float4_t>();
    if (c < b && j < k) {
        const float* src = part + c * kpad + j;
        const int64_t qs = b * kpad;
        int q = 0;
        for (; q + 8 <= splits; q += 8) {
            float4_t pv[8];
#pragma unroll
            for (int u = 0; u < 8; ++u) pv[u] = __builtin_nontemporal_load(reinterpret_cast<const float4_t*>(src + (q + u) * qs));
#pragma unroll
            for (int u = 0; u < 8; ++u) sum += pv[u];
        }
        for (; q < splits; ++q) sum += __builtin_nontemporal_load(reinterpret_cast<const float4_t*>(src + q * qs));
#pragma unroll
        for (int v = 0; v < 4; ++v) sum[v] = j + v < k ? s[j + v] * sum[v] : 0.0f;
    }
    const unsigned long long mask = __builtin_amdgcn_ballot_w64(x3_outside(sum[0]) | x3_outside(sum[1]) |
                                                                x3_outside(sum[2]) | x3_outside(sum[3]));
    if ((threadIdx.x & 63) == 0) tmask[idx >> 6] = mask;
    if (c >= b) return;
    if (j < ldt) *reinterpret_cast<float4_t*>(Tt + c * ldt + j) = sum;
    unsigned lo[3], hi[3];
    x3_split2(sum[0], sum[1], lo);
    x3_split2(sum[2], sum[3], hi);
#pragma unroll
    for (int t = 0; t < 3; ++t) *reinterpret_cast<u32x2_t*>(Tp + t * b * ldk + c * ldk + j) = (u32x2_t){lo[t], hi[t]};
}

// ---- phase 2 ---------------------------------------------------------------------
// Y[m][n] = sum_k U[m][k] T'^T[n][k] from the planes: one 128 x 128 tile per
// workgroup of 4 waves.  A K step of 32 moves 48 KB of planes straight into
// LDS; every wave reads its 24 fragments into registers, and the next step's
// loads run under the 96 products of this one (one LDS buffer, two
// workgroups per compute unit).  K steps with a marked value of U or T' are left
// out of the loop and run after it from the FP32 operands (U in place, T'^T with
// pitch ldt) on the FP32 instruction; a tile with more than half of its steps
// marked, or a mark among more than 64, or sums that are not finite, runs all
// of them that way.
// Bound by the matrix cores at the clock that their power leaves (1.6 to 1.8
// of 2.4 GHz here): 65536 x 4096, k = 513, b = 4096 in 1540 to 1580 us against
// 2160 us on the FP32 instruction; 8192 x 8192, k = 257 in 107 against 168 us
// (reading the marks costs 2 % of it).
// Measured before it: both operands split on their way to LDS 1650 us (the
// splits' vector work), fragments read as they are used and three workgroups
// per compute unit 1547 against 1366 us.
using X3C2 = Cfg<float, 128, 128, 16, 2, 2>;
__global__ __launch_bounds__(256, 2) void k_p2_x3(const unsigned short* __restrict__ Up,
                                                  const unsigned short* __restrict__ Tp, int64_t ldk,
                                                  const float* __restrict__ U, int64_t M, int64_t k,
                                                  const float* __restrict__ Tt, int64_t ldt, int64_t N, int tiles_m,
                                                  int tiles_n, const unsigned long long* __restrict__ umask,
                                                  const unsigned long long* __restrict__ tmask, float* __restrict__ Y,
                                                  int64_t ldy, int vec16) {
    using C = X3C2;
    constexpr int PLANE = 128 * kX3BK;
    static_assert(2 * (C::BM + C::BN) * C::LDK * 4 <= 6 * PLANE * 2 && (C::BM + C::BN) * 36 * 4 <= 6 * PLANE * 2,
                  "the FP32 loops and the store fit the planes' LDS");
    __shared__ alignas(16) unsigned short S[6 * PLANE];
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int wm = wave / C::WN, wn = wave % C::WN;
    const AbtOrder ord(tiles_m, tiles_n);
    const int64_t lt = xcd_tile(ord.total);
    if (lt >= ord.total) return;
    const int64_t mt = (lt % ord.per_group) / ord.G;
    const int64_t nt = (lt / ord.per_group) * ord.G + (lt % ord.per_group) % ord.G;
    if (nt >= tiles_n) return;
    const int64_t m0 = mt * C::BM, n0 = nt * C::BN;

    float4_t acc[C::FN][C::FM];
#pragma unroll
    for (int fn = 0; fn < C::FN; ++fn)
#pragma unroll
        for (int fm = 0; fm < C::FM; ++fm) acc[fn][fm] = zero_accv<float4_t>();

    // wave w moves rows [32 w, 32 w + 32) of every plane
    const unsigned short *pu[2], *pt[2];
#pragma unroll
    for (int h = 0; h < 2; ++h) {
        const int64_t ru = m0 + wave * 32 + 16 * h + (lane >> 2), rt = n0 + wave * 32 + 16 * h + (lane >> 2);
        pu[h] = Up + (ru < M ? ru : M - 1) * ldk + x3_chunk(lane) * 8;
        pt[h] = Tp + (rt < N ? rt : N - 1) * ldk + x3_chunk(lane) * 8;
    }
    auto move = [&](int j) {
#pragma unroll
        for (int q = 0; q < 3; ++q)
#pragma unroll
            for (int h = 0; h < 2; ++h) {
                unsigned short* d = S + q * PLANE + (wave * 32 + 16 * h) * kX3BK;
                load_lds16(pu[h] + q * M * ldk + j * kX3BK, d);
                load_lds16(pt[h] + q * N * ldk + j * kX3BK, d + 3 * PLANE);
            }
    };
    const int nsteps = (int)(ldk / kX3BK);
    // marks among this tile's rows of U (4 bits per K step of a row) and of T'^T
    // (8 bits); every wave reads them all, so that they agree without a barrier
    const int64_t u0 = m0 * (ldk / 8), u1 = std::min(m0 + C::BM, M) * (ldk / 8);
    const int64_t t0 = n0 * (ldk / 4), t1 = std::min(n0 + C::BN, N) * (ldk / 4);
    const unsigned long long *um = umask + (u0 >> 6), *tm = tmask + (t0 >> 6);
    const int ul = (int)(((u1 - 1) >> 6) - (u0 >> 6)), tl = (int)(((t1 - 1) >> 6) - (t0 >> 6));
    unsigned long long some = 0;   // neighbours' bits included; the first 1000 ranks in one round of loads
#pragma unroll
    for (int q = 0; q < 4; ++q) some |= um[std::min(lane + 64 * q, ul)];
#pragma unroll
    for (int q = 0; q < 8; ++q) some |= tm[std::min(lane + 64 * q, tl)];
    for (int i = lane + 256; i <= ul; i += 64) some |= um[i];
    for (int i = lane + 512; i <= tl; i += 64) some |= tm[i];
    move(0);
    unsigned long long marked = 0;   // K steps with marks
    bool all = false;                // every step on the FP32 instruction
    if (__builtin_amdgcn_ballot_w64(some != 0) != 0) {
        all = nsteps > 64;
        if (!all) {
            auto steps = [&](const unsigned long long* mask, int last, int64_t first, int64_t end, int per) {
                for (int i = lane; i <= last; i += 64) {
                    const int64_t c0 = ((first >> 6) + i) << 6;
                    unsigned long long bits = mask[i];
                    if (c0 < first) bits &= ~0ull << (first - c0);
                    if (end < c0 + 64) bits &= ~0ull >> (c0 + 64 - end);
                    for (int j = (int)(c0 / per % nsteps); bits; bits >>= per) {
                        if (bits & ((1 << per) - 1)) marked |= 1ull << j;
                        j = j + 1 < nsteps ? j + 1 : 0;
                    }
                }
            };
            steps(um, ul, u0, u1, 4);
            steps(tm, tl, t0, t1, 8);
#pragma unroll
            for (int d = 1; d < 64; d *= 2) marked |= __shfl_xor(marked, d, 64);
            const unsigned lo = __builtin_amdgcn_readfirstlane((unsigned)marked);
            marked = (unsigned long long)__builtin_amdgcn_readfirstlane((unsigned)(marked >> 32)) << 32 | lo;
            all = 2 * __builtin_popcountll(marked) > nsteps;
        }
    }
    float* smem = reinterpret_cast<float*>(S);
    if (!all) {
        for (int j = 0; j < nsteps; ++j) {
            wait_loads();
            __syncthreads();
            bf8_t u[C::FM][3], t[C::FN][3];
#pragma unroll
            for (int q = 0; q < 3; ++q) {
#pragma unroll
                for (int fm = 0; fm < C::FM; ++fm) u[fm][q] = x3_frag(S + q * PLANE, wm * C::WTM + fm * 16, lane);
#pragma unroll
                for (int fn = 0; fn < C::FN; ++fn) t[fn][q] = x3_frag(S + (3 + q) * PLANE, wn * C::WTN + fn * 16, lane);
            }
            __syncthreads();
            if (j + 1 < nsteps) move(j + 1);
            if (marked >> (j & 63) & 1) continue;
#pragma unroll
            for (int e = 0; e < 6; ++e)
#pragma unroll
                for (int fn = 0; fn < C::FN; ++fn)
#pragma unroll
                    for (int fm = 0; fm < C::FM; ++fm)
                        acc[fn][fm] = x3_mfma(t[fn][kX3A[e]], u[fm][kX3B[e]], acc[fn][fm]);
        }
        // the marked steps: 128 rows of U and of T'^T as FP32 in LDS, 36 floats apart,
        // the next step's values requested under the products
        const int kk = tid & 31, row0 = tid >> 5, q4 = (tid & 7) * 4, row4 = tid >> 3;
        float uv[16];
        float4_t tv[4];
        auto fetch = [&](int64_t k0) {
#pragma unroll
            for (int e = 0; e < 16; ++e) {
                const int64_t row = m0 + row0 + 8 * e;
                uv[e] = U[(row < M ? row : M - 1) * k + (k0 + kk < k ? k0 + kk : k - 1)];
            }
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                const int64_t row = n0 + row4 + 32 * e;
                tv[e] = *reinterpret_cast<const float4_t*>(Tt + (row < N ? row : N - 1) * ldt + (k0 + q4 < ldt ? k0 + q4 : 0));
            }
        };
        if (marked) fetch((int64_t)__builtin_ctzll(marked) * kX3BK);
        while (marked) {
            const int64_t k0 = (int64_t)__builtin_ctzll(marked) * kX3BK;
            __syncthreads();
#pragma unroll
            for (int e = 0; e < 16; ++e) smem[(row0 + 8 * e) * 36 + kk] = k0 + kk < k ? uv[e] : 0.0f;
#pragma unroll
            for (int e = 0; e < 4; ++e)
                *reinterpret_cast<float4_t*>(smem + (128 + row4 + 32 * e) * 36 + q4) =
                    k0 + q4 < ldt ? tv[e] : zero_accv<float4_t>();
            __syncthreads();
            marked &= marked - 1;
            if (marked) fetch((int64_t)__builtin_ctzll(marked) * kX3BK);
            const float* up = smem + (wm * C::WTM + (lane & 15)) * 36 + (lane >> 4);
            const float* tp = smem + (128 + wn * C::WTN + (lane & 15)) * 36 + (lane >> 4);
#pragma unroll
            for (int e = 0; e < 8; ++e) {
                float u[C::FM], t[C::FN];
#pragma unroll
                for (int fm = 0; fm < C::FM; ++fm) u[fm] = up[fm * 16 * 36 + 4 * e];
#pragma unroll
                for (int fn = 0; fn < C::FN; ++fn) t[fn] = tp[fn * 16 * 36 + 4 * e];
#pragma unroll
                for (int fn = 0; fn < C::FN; ++fn)
#pragma unroll
                    for (int fm = 0; fm < C::FM; ++fm) acc[fn][fm] = mfma(t[fn], u[fm], acc[fn][fm]);
            }
        }
        bool bad = false;
#pragma unroll
        for (int fn = 0; fn < C::FN; ++fn)
#pragma unroll
            for (int fm = 0; fm < C::FM; ++fm)
#pragma unroll
                for (int v = 0; v < 4; ++v) bad = bad || !(__builtin_fabsf(acc[fn][fm][v]) < __builtin_inff());
        all = __syncthreads_or(bad ? 1 : 0) != 0;
    }
    if (all) {
        wait_loads();   // the first step's, which land in the same LDS
        __syncthreads();
#pragma unroll
        for (int fn = 0; fn < C::FN; ++fn)
#pragma unroll
            for (int fm = 0; fm < C::FM; ++fm) acc[fn][fm] = zero_accv<float4_t>();
        abt_products<float, C, true>(U, k, m0, M, k, Tt, ldt, n0, N, ldt, ldt, smem, acc, wm, wn, lane, tid);
    }
    abt_store_staged<float, C>(acc, smem, tid, wm, wn, m0, n0, M, N, Y, ldy, vec16);
}

// ---- host ------------------------------------------------------------------------
// About the bytes of V's planes per split and of a column's partial sums; factors
// too large for both keep the FP32 instruction.  Panels of such sizes fit the
// allocation-free entry's scratch (x3_plan makes sure).
constexpr int64_t kX3MaxChunk = (int64_t)64 * 32 * kX3BK;   // rows whose steps fit the bits of a wave's lanes
constexpr int64_t kX3VBytes = (int64_t)16 << 20, kX3ColBytes = (int64_t)128 << 10;

// Sizes that gain from the split, times of the split over those of the FP32
// instruction's plan beside each line (grids of 512 <= m, n <= 65536, 4 <= k <= 513, 512
// <= b <= 8192).  What it saves grows with the (m + n) b values of X and Y and with
// the rank; what it costs is the planes' launch and 10 bytes per factor value.
// Odd batches gain by X read without a padded copy, odd ranks by U and V.
static bool x3_takes(int64_t m, int64_t n, int64_t k, int64_t b, int prec, const void* U, const void* V,
                     const void* X) {
    if (prec != P32 || b < 512 || m < 128) return false;   // batches below 512: 1.1 to 2
    // Sums of up to three products: the terms that six products leave out (2.01
    // 2^-24 of each) outweigh the roundings that they save (error of k = 1 in units
    // of 2^-24 |U| |T'|: 4.2 against 2.6, k = 3 4.1 against 3.9, k = 4 3.7 against 4.4).
    if (k < 4) return false;
    const int64_t kpad = round_up(k, 16) + 16 * 17;
    if ((double)n * kpad * 6.0 / kX3VBytes > (double)(kX3ColBytes / 4) / kpad) return false;
    const double values = (double)(m + n) * b;
    const bool xbad = needs_stage(X, b, prec), kbad = needs_stage(U, k, prec) || needs_stage(V, k, prec);
    const bool wide = n > 2 * m, tall = m > 2 * n;                // phase 1, bound by X, is the most or little of it
    const bool xgain = xbad && !tall && values >= (b >= 1536 ? 7.0e6 : 8.0e6);   // 0.44 to 0.94; else 0.92 to 1.20
    if (k <= 16) return xgain;                                    // else 1.0 to 1.23
    if (values >= 0x1p25) {
        if (k >= 96 || xbad) return true;                         // 0.47 to 1.02
        if (kbad) return k > 32 || !wide;                         // 0.79 to 1.01; else 0.99 to 1.05
        if (values < 0x1.2p25) return false;                      // 0.97 to 1.13
        return !wide || (k > 32 && values >= 0x1p27);             // 0.76 to 1.01; else 0.97 to 1.13
    }
    // 0.52 to 1.0; else 0.72 to 1.18
    if (values >= 0x1p24)
        return xgain || k >= 160 || (k >= 96 && (kbad || b >= 1536)) || (kbad && b >= (tall ? 1536 : 2048));
    // 0.76 to 0.97; else 0.84 to 1.20
    const double least = tall ? 7.0e6 : k >= 160 ? 7.5e6 : 1.2e7;
    return xgain || (kbad && k >= 96 && values >= least);
}

// Fragments per rank tile: at most 17, so that ranks 16 j + 1 (a compensated
// rank past a round one) up to 257 stay one tile.  Row chunks for about two
// workgroups per compute unit (256 instead of 512: 136 against 101 us at
// 8192 x 8192, k = 257, b = 4096), at least 128 rows each.  False (p unusable):
// a call that the allocation-free entry takes (p.scratch_bytes) would not fit
// its scratch; both entries then keep the FP32 instruction, with equal bits.
static bool x3_plan(ApplyPlan& p, int64_t m, int64_t n, int64_t k, int64_t b) {
    const int64_t frags = (k + 15) / 16;
    p.x3 = 1;
    p.mis1 = p.mis2 = p.misx = p.stage_u = p.stage_v = p.stage_x = 0;
    p.tiles_m = (int)((frags + 16) / 17);
    p.nf = (int)((frags + p.tiles_m - 1) / p.tiles_m);
    p.tiles_n = (int)((b + 127) / 128);
    p.kpad = (int64_t)p.tiles_m * p.nf * 16;
    p.ldk = round_up(k, kX3BK);
    const int64_t base = (int64_t)p.tiles_m * p.tiles_n;
    int64_t splits = std::min((512 + base - 1) / base, n / 128);
    splits = std::min(splits, kX3ColBytes / 4 / p.kpad);
    splits = std::max(splits, (n * p.kpad * 6 + kX3VBytes - 1) / kX3VBytes);
    splits = std::max(splits, (n + kX3MaxChunk - 1) / kX3MaxChunk);
    p.chunk = round_up((n + splits - 1) / splits, kX3BK);
    p.splits = (int)((n + p.chunk - 1) / p.chunk);
    const size_t noalloc = (size_t)LRC_NOALLOC_SCRATCH_BYTES;
    return (p.scratch_bytes > noalloc || x3_panels(p, m, b, noalloc)) && x3_panels(p, m, b, (size_t)1 << 30);
}

// Bytes of one panel's marks of values outside the split's range (whole workgroups of
// the kernels that write them).
static int64_t x3_umask_bytes(const ApplyPlan& p) { return (p.mpanel * (p.ldk / 8) + 255) / 256 * 32; }
static int64_t x3_tmask_bytes(const ApplyPlan& p) { return (p.bpanel * (p.ldk / 4) + 255) / 256 * 32; }
static int64_t x3_mark_bytes(const ApplyPlan& p) {
    return x3_umask_bytes(p) + x3_tmask_bytes(p) + ((p.vgroup * p.chunk + 63) / 64) * ((p.kpad + 63) / 64) * 8;
}

// Panels within `limit` bytes of scratch: splits whose planes of V^T are held
// at a time, columns of the batch and rows of U.  V takes up to a quarter (one
// split at least), columns and rows share two to one what it leaves.  Every
// output value is the same whatever the panels.  False: not even panels of 128
// columns and rows fit, the plan is not usable.
bool x3_panels(ApplyPlan& p, int64_t m, int64_t b, size_t limit) {
    // marks included: eight bytes per 64 x 64 of V, a bit per 8 values of U, 4 of T'
    const int64_t vsplit = 6 * p.kpad * p.chunk + 8 * ((p.chunk + 63) / 64) * ((p.kpad + 63) / 64);
    const int64_t col = (int64_t)p.splits * p.kpad * 4 + p.Kp * 4 + 6 * p.ldk + p.ldk / 32;
    const int64_t row = 6 * p.ldk + p.ldk / 64 + 1, room = (int64_t)limit - 4096;
    p.vgroup = p.splits;
    p.bpanel = b;
    p.mpanel = m;
    if (vsplit * p.vgroup + col * b + row * m > room) {
        p.vgroup = std::max<int64_t>(1, std::min<int64_t>(p.splits, room / 4 / vsplit));
        const int64_t left = room - p.vgroup * vsplit;
        p.bpanel = std::min(b, left / 3 * 2 / col / 128 * 128);
        p.mpanel = std::min(m, (left - p.bpanel * col) / row / 128 * 128);
        if (p.bpanel < std::min<int64_t>(b, 128) || p.mpanel < std::min<int64_t>(m, 128)) return false;
    }
    p.part_bytes = (size_t)p.splits * p.bpanel * p.kpad * 4;
    p.mid_bytes = (size_t)p.bpanel * p.Kp * 4;
    p.stage_bytes = round_up((size_t)6 * p.bpanel * p.ldk, 256) + round_up((size_t)6 * p.mpanel * p.ldk, 256) +
                    round_up((size_t)6 * p.kpad * p.chunk * p.vgroup, 256) + round_up((size_t)x3_mark_bytes(p), 256);
    return true;
}

static hipError_t x3_apply(const ApplyPlan& p, const float* U, const float* s, const float* V, const float* X,
                           float* Y, int64_t m, int64_t n, int64_t k, int64_t b, float* part, float* Tt,
                           Workspace& ws, hipStream_t stream) {
    unsigned short* Tp = static_cast<unsigned short*>(ws.take((size_t)6 * p.bpanel * p.ldk));
    unsigned short* Up = static_cast<unsigned short*>(ws.take((size_t)6 * p.mpanel * p.ldk));
    unsigned short* Vp = static_cast<unsigned short*>(ws.take((size_t)6 * p.kpad * p.chunk * p.vgroup));
    char* marks = static_cast<char*>(ws.take((size_t)x3_mark_bytes(p)));
    if (ws.overrun) return hipErrorOutOfMemory;
    auto* umask = reinterpret_cast<unsigned long long*>(marks);
    auto* tmask = reinterpret_cast<unsigned long long*>(marks + x3_umask_bytes(p));
    auto* vflag = reinterpret_cast<unsigned char*>(tmask) + x3_tmask_bytes(p);
    // planes of `rows` rows of U and of `cols` rows of V (0: none)
    auto planes = [&](const float* u, int64_t rows, const float* v, int64_t cols, int64_t ldn) {
        KernelTimer t("apply_planes_f32", stream);
        const unsigned ub = (unsigned)((rows * (p.ldk / 8) + 255) / 256), nt = (unsigned)((ldn + 63) / 64);
        hipLaunchKernelGGL(k_x3_planes, dim3(ub + nt * (unsigned)((p.kpad + 63) / 64)), dim3(256), 0, stream, u, rows, k,
                           Up, p.ldk, ub, v, cols, Vp, ldn, p.kpad, nt, umask, vflag);
    };
    const bool whole_u = p.mpanel >= m, whole_v = p.vgroup >= p.splits;
    const int vec16 = vec_ok<float>(Y, b) ? 1 : 0;
    for (int64_t b0 = 0; b0 < b; b0 += p.bpanel) {
        const int64_t bw = std::min(p.bpanel, b - b0);
        const int tn = (int)((bw + 127) / 128);
        for (int64_t s0 = 0; s0 < p.splits; s0 += p.vgroup) {
            const int64_t ns = std::min<int64_t>(p.vgroup, p.splits - s0), r0 = s0 * p.chunk;
            const int64_t rows = std::min(ns * p.chunk, n - r0), ldn = round_up(rows, kX3BK);
            if (b0 == 0 || !whole_v) planes(U, whole_u && b0 == 0 && s0 == 0 ? m : 0, V + r0 * k, rows, ldn);
            KernelTimer t("apply_p1_mfma_f32", stream);
            const dim3 g(xcd_grid((int64_t)p.tiles_m * tn * ns));
#define LRC_P1X(NF)                                                                                                 \
    hipLaunchKernelGGL(k_p1_x3<NF>, g, dim3(256), 0, stream, Vp, ldn, p.kpad, V + r0 * k, k, X + r0 * b + b0, b, rows, \
                       bw, p.chunk, p.nf, p.tiles_m, tn, (int)ns, vflag, part + s0 * bw * p.kpad)
            if (p.nf <= 5) LRC_P1X(5); else if (p.nf <= 9) LRC_P1X(9); else LRC_P1X(17);
#undef LRC_P1X
        }
        {
            KernelTimer t("apply_p1_finish_f32", stream);
            hipLaunchKernelGGL(k_x3_finish, dim3((unsigned)((bw * (p.ldk / 4) + 255) / 256)), dim3(256), 0, stream,
                               part, p.kpad, p.splits, s, k, bw, Tt, p.Kp, Tp, p.ldk, tmask);
        }
        for (int64_t m0 = 0; m0 < m; m0 += p.mpanel) {
            const int64_t mw = std::min(p.mpanel, m - m0);
            if (!whole_u) planes(U + m0 * k, mw, V, 0, 0);
            KernelTimer t("apply_p2_mfma_f32", stream);
            const int tm = (int)((mw + 127) / 128);
            hipLaunchKernelGGL(k_p2_x3, dim3(xcd_grid(AbtOrder(tm, tn).total)), dim3(256), 0, stream, Up, Tp, p.ldk,
                               U + m0 * k, mw, k, Tt, p.Kp, bw, tm, tn, umask, tmask, Y + m0 * b + b0, b, vec16);
        }
        const hipError_t e = hipGetLastError();
        if (e != hipSuccess) return e;
    }
    return hipSuccess;
}
