// FP16 phase 2 for large outputs; part of apply.hip.
#pragma once

// Y[m][n] = sum_k U[m][k] T'^T[n][k] in binary16 with FP32 accumulation: one
// 256 x 128 tile per workgroup of 4 waves (128 x 64 each).  The K steps of 32
// move 24 KB straight into one of three LDS buffers, two steps ahead of the
// products, without registers or vector work; rows of 64 bytes with their
// 16-byte chunks XOR-swizzled on the global side (see x3_frag).
// U: 16-byte aligned rows of pitch ldu, k values each (k a multiple of 8);
// T'^T: pitch ldt, a multiple of 32, zero from k on, which also stands in
// for U's columns past k.
// 65536 x 4096, b = 4096: k = 512 417 -> 320 us, k = 513 500 -> 365 us, k = 65
// 172 -> 120 us (4.5 TB/s of output); the tiles it replaced staged operands
// through registers into rows whose pad left 0.4 of the LDS time to bank
// conflicts.  Now the matrix cores are busy 41 % of the time at 2.0 GHz
// and the address units 56 %.  Within 2 %: 192 x 128 tiles with K steps of 64
// (128 contiguous bytes per row, two buffers); slower: 256 x 128 with K steps
// of 64 and one buffer (400 us, one workgroup per compute unit).
using HalfC2 = Cfg<half_t, 256, 128, 32, 2, 2>;
constexpr int kHalfBufs = 3;
__global__ __launch_bounds__(256, 2) void k_p2_half(const half_t* __restrict__ U, int64_t ldu, int64_t M, int64_t k,
                                                    const half_t* __restrict__ Tt, int64_t ldt, int64_t N,
                                                    int tiles_m, int tiles_n, half_t* __restrict__ Y, int64_t ldy,
                                                    int vec16) {
    using C = HalfC2;
    constexpr int TA = C::BM * C::BK, TB = C::BN * C::BK, BUF = TA + TB;
    static_assert(kHalfBufs * BUF >= 2 * (C::BM + C::BN) * C::LDK, "the store's staging fits the buffers");
    __shared__ alignas(16) half_t S[kHalfBufs * BUF];
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

    // wave w moves rows [64 w, 64 w + 64) of U and [32 w, 32 w + 32) of T'^T
    const int ch = x3_chunk(lane) * 8;
    const half_t *pu[4], *pt[2];
#pragma unroll
    for (int h = 0; h < 4; ++h) {
        const int64_t r = m0 + wave * 64 + 16 * h + (lane >> 2);
        pu[h] = U + (r < M ? r : M - 1) * ldu + ch;
    }
#pragma unroll
    for (int h = 0; h < 2; ++h) {
        const int64_t r = n0 + wave * 32 + 16 * h + (lane >> 2);
        pt[h] = Tt + (r < N ? r : N - 1) * ldt + ch;
    }
    const int nsteps = (int)((k + C::BK - 1) / C::BK);
    auto move = [&](int j, int buf) {
        half_t* d = S + buf * BUF;
        const bool past = j * C::BK + ch >= k;
#pragma unroll
        for (int h = 0; h < 4; ++h)
            load_lds16(past ? Tt + k : pu[h] + j * C::BK, d + (wave * 64 + 16 * h) * C::BK);
#pragma unroll
        for (int h = 0; h < 2; ++h) load_lds16(pt[h] + j * C::BK, d + TA + (wave * 32 + 16 * h) * C::BK);
    };
    move(0, 0);
    if (nsteps > 1) move(1, 1);
    int buf = 0;
    for (int j = 0; j < nsteps; ++j) {
        // this step's loads have landed (the next step's six may be in flight),
        // and so have everyone's once past the barrier; a plain barrier, since
        // __syncthreads would wait for all loads
        if (j + 1 < nsteps) asm volatile("s_waitcnt vmcnt(6) lgkmcnt(0)" ::: "memory");
        else asm volatile("s_waitcnt vmcnt(0) lgkmcnt(0)" ::: "memory");
        __builtin_amdgcn_s_barrier();
        asm volatile("" ::: "memory");
        if (j + 2 < nsteps) move(j + 2, buf == 0 ? 2 : buf - 1);
        const unsigned short* As = reinterpret_cast<const unsigned short*>(S + buf * BUF);
        half8_t a[C::FN], b[C::FM];
#pragma unroll
        for (int fn = 0; fn < C::FN; ++fn) a[fn] = __builtin_bit_cast(half8_t, x3_frag(As + TA, wn * C::WTN + fn * 16, lane));
#pragma unroll
        for (int fm = 0; fm < C::FM; ++fm) b[fm] = __builtin_bit_cast(half8_t, x3_frag(As, wm * C::WTM + fm * 16, lane));
#pragma unroll
        for (int fm = 0; fm < C::FM; ++fm)
#pragma unroll
            for (int fn = 0; fn < C::FN; ++fn) acc[fn][fm] = mfma(a[fn], b[fm], acc[fn][fm]);
        buf = buf == 2 ? 0 : buf + 1;
    }
    __syncthreads();
    abt_store_staged<half_t, C>(acc, S, tid, wm, wn, m0, n0, M, N, Y, ldy, vec16);
}

// Outputs of at least two tiles per compute unit; below, the 128 x 128 tiles
// spread better (4096 x 1024, k = 256: 10.4 against 12.2 us; 8192 x 512, k = 128:
// 9.4 against 9.8 us; from 13505 x 1795, 795 tiles, on this kernel gains).
// Odd pitches are copied first (stage_u) unless they are small.
static bool half_takes(const ApplyPlan& p, int64_t m, int64_t b) {
    return p.big2 && !p.mis2 && !forced_tile() &&
           tiles_of(m, HalfC2::BM) * tiles_of(b, HalfC2::BN) >= 512;
}
