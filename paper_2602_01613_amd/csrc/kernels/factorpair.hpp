// Both factors on a side of a Tucker core applied to every token, a workgroup to a token.
// Part of the tn_linear library's single translation unit: included by tn_linear.hip inside its
// anonymous namespace, after kernels/common.hpp.
#pragma once

// ---------------------------------------------------------------------------------------------
// With U1 [A][P] and U2 [B][Q] the factors, Y [A][B] a token on the side of the modes and G [Q][P] the one on the side of the core:
//     in:   S = Y U2,        G = (U1^T S)^T          out:  T = U1 G^T,       Y = T U2^T
// The same two products either way, out[c1][c2] = sum_r (sum_k in[r][k] first[c1][k]) second[c2][r] with a bf16 intermediate; the forms differ
// in what is large, what comes in or what leaves.
//
// Bound by memory: 18 KB and 51 KB a token for 3.9 million multiply-adds (160 x 160, ranks of 96), 1 us of a compute unit's matrix
// cores beside 3.5 of its share of the memory's rate. So a workgroup does a whole token between a load and a store of whole rows, and two
// or three of them on a compute unit cover each other's:
//   * the token goes to LDS through registers, requested while the one before is multiplied; four waves 2 x 2. A wave's share of the
//     factors stays in registers where that takes kFactorHeld of them (64 x 80 to ranks of 48, 8192 tokens from memory: 25 us, read from L2
//     for every token 31), else it is requested ahead of the barrier behind which it is used;
//   * the intermediate, in the registers of an accumulator along what the second product contracts, goes to LDS in 8-byte pieces. LDS
//     decides how many workgroups there are, so it takes the place of what has been read: in, of Y; out, of nothing yet, but Y then of
//     it and of G, and leaves in rows of 16-byte pieces;
//   * rows in LDS are 16 bytes longer than the data, an odd number of 16-byte units; extents are padded to multiples of 32 with zeros.
// us at 8192 tokens, a wave to a token (step_chain2_kernel) / so: 64 x 80 to ranks of 48 40 / 25, ranks of 96 to 160 x 160 154 / 125; at
// 500 tokens 5.4 / 4.8 and 19.5 / 12. 160 x 160 to ranks of 96, which that kernel has no registers for, at 500 tokens 24.7 as two launches / 13.
// ---------------------------------------------------------------------------------------------
struct FactorPairArgs {
    const bf16_t* in;
    bf16_t* out;
    const bf16_t *first, *second;           // packed fragment-major: in: columns q, k = b; columns p, k = a. out: columns a, k = p; columns b, k = q
    int32_t nks_first, nks_second;          // k-steps of 16 of those
    int32_t size_first, size_second;        // bytes of those
    int32_t A, B, P, Q;                     // multiples of 16
    int32_t tokens;
};

// What the two kernels share: a matrix [R][C] on its way to LDS through registers, and the operands of a 16 x 16 x 32 product.
template <int R, int C>
struct FactorTile {
    static constexpr int PITCH = C + 8, PIECES = C / 8, ROWS = 256 / PIECES, N = (R + ROWS - 1) / ROWS;      // rows that 256 threads bring at a time
};

typedef uint32_t factor_u32x4 __attribute__((ext_vector_type(4)));
constexpr uint32_t kFactorNowhere = 0x80000000u;
constexpr int kFactorHeld = 90;             // registers that a workgroup's share of both factors may take to be held throughout

__device__ __forceinline__ bf16x8 factor_fetch(const bf16_t* p, int size, uint32_t at) {
#ifdef __HIP_DEVICE_COMPILE__
    const __amdgpu_buffer_rsrc_t r = __builtin_amdgcn_make_buffer_rsrc(const_cast<bf16_t*>(p), 0, size, 0x00020000);
    return __builtin_bit_cast(bf16x8, __builtin_amdgcn_raw_buffer_load_b128(r, int(at), 0, 0));
#else
    return bf16x8{};
#endif
}

// Lane l: column tile * 16 + l % 16, k = 32 * ks + 8 * (l / 16) .. + 7 (bfrag_offset); zeros past the tensor's end.
__device__ __forceinline__ bf16x8 factor_operand(const bf16_t* src, int size, int nks, int tile, int ks, int lane) {
    const int l16 = lane & 15, h = lane >> 4;
    uint32_t at = uint32_t((h >> 1) * 1024 + (l16 + 32 * (h & 1)) * 16);
    asm volatile("" : "+v"(at));                                   // (not one register per load throughout)
    at += uint32_t(((tile >> 1) * nks + ks * 2) * 1024 + (tile & 1) * 256);
    return factor_fetch(src, size, ks * 2 + (h >> 1) < nks ? at : kFactorNowhere);
}

template <int A32, int B32, int P32, int Q32>
constexpr size_t factor_in_smem() { return size_t(32 * A32) * FactorTile<32 * A32, 32 * B32>::PITCH * 2; }

template <int A32, int B32, int P32, int Q32>
__global__ void __launch_bounds__(256, 2) factor_in_kernel(FactorPairArgs g0, FactorPairArgs g1) {
#ifdef __HIP_DEVICE_COMPILE__
    const FactorPairArgs& g = blockIdx.y ? g1 : g0;
    constexpr int LA = 32 * A32, LB = 32 * B32;
    using Ty = FactorTile<LA, LB>;
    constexpr int PY = Ty::PITCH, PS = LA + 8;
    static_assert(32 * Q32 * PS <= LA * PY, "S takes Y's place");
    typedef __bf16 bf16x4_t __attribute__((ext_vector_type(4)));
    extern __shared__ __attribute__((aligned(16))) unsigned char dyn_smem[];
    bf16_t* sY = reinterpret_cast<bf16_t*>(dyn_smem);
    const int tid = threadIdx.x, lane = tid & 63, l16 = lane & 15, h = lane >> 4;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6), wr = wave >> 1, wc = wave & 1;
    auto plain = [&](int pitch, int tile, int ks) { return *reinterpret_cast<const bf16x8*>(sY + (tile * 16 + l16) * pitch + ks * 32 + 8 * h); };
    auto mma = [&](bf16x8 a, bf16x8 b, floatx4 c) { return __builtin_amdgcn_mfma_f32_16x16x32_bf16(a, b, c, 0, 0, 0); };
    auto round4 = [&](floatx4 v) {
        bf16x4_t r;
#pragma unroll
        for (int e = 0; e < 4; ++e) r[e] = bf16_t(v[e]);
        return r;
    };
    bf16x8 ry[Ty::N];
    const int y_row = tid / Ty::PIECES, y_col = (tid - y_row * Ty::PIECES) * 8;
    const uint32_t y_at = y_row < Ty::ROWS && y_col < g.B ? uint32_t(y_row * g.B + y_col) * 2 : kFactorNowhere;
    auto request = [&](int t) {
        uint32_t yo = y_at;
        asm volatile("" : "+v"(yo));
#pragma unroll
        for (int n = 0; n < Ty::N; ++n) ry[n] = factor_fetch(g.in + int64_t(t) * g.A * g.B, g.A * g.B * 2, yo + uint32_t(n * Ty::ROWS * g.B * 2));
    };
    constexpr bool HOLD = (Q32 * B32 + P32 * A32) * 4 <= kFactorHeld;
    bf16x8 u2[Q32][B32], u1[P32][A32];
    auto request_first = [&]() {
#pragma unroll
        for (int j = 0; j < Q32; ++j)
#pragma unroll
            for (int ks = 0; ks < B32; ++ks) u2[j][ks] = factor_operand(g.first, g.size_first, g.nks_first, wc * Q32 + j, ks, lane);
    };
    auto request_second = [&]() {
#pragma unroll
        for (int i = 0; i < P32; ++i)
#pragma unroll
            for (int ks = 0; ks < A32; ++ks) u1[i][ks] = factor_operand(g.second, g.size_second, g.nks_second, wr * P32 + i, ks, lane);
    };
    const floatx4 none = {0.f, 0.f, 0.f, 0.f};
    if (int(blockIdx.x) >= g.tokens) return;
    request(blockIdx.x);
    if constexpr (HOLD) {
        request_first();
        request_second();
    }
    for (int t = blockIdx.x; t < g.tokens; t += gridDim.x) {
        if (y_row < Ty::ROWS) {
#pragma unroll
            for (int n = 0; n < Ty::N; ++n)
                if ((n + 1) * Ty::ROWS <= LA || n * Ty::ROWS + y_row < LA) *reinterpret_cast<bf16x8*>(sY + (n * Ty::ROWS + y_row) * PY + y_col) = ry[n];
        }
        floatx4 acc[A32][Q32];
#pragma unroll
        for (int i = 0; i < A32; ++i)
#pragma unroll
            for (int j = 0; j < Q32; ++j) acc[i][j] = none;
        {
            if constexpr (!HOLD) request_first();
            __syncthreads();
            if (t + int(gridDim.x) < g.tokens) request(t + gridDim.x);
            bf16x8 f[2][A32];
#pragma unroll
            for (int i = 0; i < A32; ++i) f[0][i] = plain(PY, wr * A32 + i, 0);
#pragma unroll
            for (int s = 0; s < B32; ++s) {
                if (s + 1 < B32) {
#pragma unroll
                    for (int i = 0; i < A32; ++i) f[(s + 1) & 1][i] = plain(PY, wr * A32 + i, s + 1);
                }
                __builtin_amdgcn_sched_barrier(0);
#pragma unroll
                for (int i = 0; i < A32; ++i)
#pragma unroll
                    for (int j = 0; j < Q32; ++j) acc[i][j] = mma(f[s & 1][i], u2[j][s], acc[i][j]);
                __builtin_amdgcn_sched_barrier(0);
            }
        }
        if constexpr (!HOLD) request_second();
        __syncthreads();                                            // Y has been read: S, [q][a], takes its place
#pragma unroll
        for (int i = 0; i < A32; ++i)
#pragma unroll
            for (int j = 0; j < Q32; ++j)
                *reinterpret_cast<bf16x4_t*>(sY + ((wc * Q32 + j) * 16 + l16) * PS + (wr * A32 + i) * 16 + 4 * h) = round4(acc[i][j]);
        __syncthreads();
        floatx4 o[P32][Q32];
#pragma unroll
        for (int i = 0; i < P32; ++i)
#pragma unroll
            for (int j = 0; j < Q32; ++j) o[i][j] = none;
        {
            bf16x8 f[2][Q32];
#pragma unroll
            for (int j = 0; j < Q32; ++j) f[0][j] = plain(PS, wc * Q32 + j, 0);
#pragma unroll
            for (int s = 0; s < A32; ++s) {
                if (s + 1 < A32) {
#pragma unroll
                    for (int j = 0; j < Q32; ++j) f[(s + 1) & 1][j] = plain(PS, wc * Q32 + j, s + 1);
                }
                __builtin_amdgcn_sched_barrier(0);
#pragma unroll
                for (int i = 0; i < P32; ++i)
#pragma unroll
                    for (int j = 0; j < Q32; ++j) o[i][j] = mma(u1[i][s], f[s & 1][j], o[i][j]);
                __builtin_amdgcn_sched_barrier(0);
            }
        }
        bf16_t* G = g.out + int64_t(t) * g.Q * g.P;
#pragma unroll
        for (int i = 0; i < P32; ++i)
#pragma unroll
            for (int j = 0; j < Q32; ++j) {
                const int p = (wr * P32 + i) * 16 + 4 * h, q = (wc * Q32 + j) * 16 + l16;
                if (p < g.P && q < g.Q) *reinterpret_cast<bf16x4_t*>(G + q * g.P + p) = round4(o[i][j]);
            }
        __syncthreads();                                            // S has been read
    }
#endif
}

template <int A32, int B32, int P32, int Q32>
constexpr size_t factor_out_smem() {
    const size_t in = size_t(2) * (32 * Q32 * FactorTile<32 * Q32, 32 * P32>::PITCH + 32 * A32 * (32 * Q32 + 8)), out = size_t(2) * 32 * A32 * (32 * B32 + 8);
    return in > out ? in : out;
}

template <int A32, int B32, int P32, int Q32>
__global__ void __launch_bounds__(256, 2) factor_out_kernel(FactorPairArgs g0, FactorPairArgs g1) {
#ifdef __HIP_DEVICE_COMPILE__
    const FactorPairArgs& g = blockIdx.y ? g1 : g0;
    constexpr int LA = 32 * A32, LB = 32 * B32, LP = 32 * P32, LQ = 32 * Q32;
    using Tg = FactorTile<LQ, LP>;
    using Ty = FactorTile<LA, LB>;
    constexpr int PG = Tg::PITCH, PT = LQ + 8, PY = Ty::PITCH;
    typedef __bf16 bf16x4_t __attribute__((ext_vector_type(4)));
    extern __shared__ __attribute__((aligned(16))) unsigned char dyn_smem[];
    bf16_t* sG = reinterpret_cast<bf16_t*>(dyn_smem);
    bf16_t* sT = sG + LQ * PG;
    bf16_t* sY = sG;                                                // once T has been read
    const int tid = threadIdx.x, lane = tid & 63, l16 = lane & 15, h = lane >> 4;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6), wr = wave >> 1, wc = wave & 1;
    auto plain = [&](const bf16_t* s, int pitch, int tile, int ks) { return *reinterpret_cast<const bf16x8*>(s + (tile * 16 + l16) * pitch + ks * 32 + 8 * h); };
    auto mma = [&](bf16x8 a, bf16x8 b, floatx4 c) { return __builtin_amdgcn_mfma_f32_16x16x32_bf16(a, b, c, 0, 0, 0); };
    auto round4 = [&](floatx4 v) {
        bf16x4_t r;
#pragma unroll
        for (int e = 0; e < 4; ++e) r[e] = bf16_t(v[e]);
        return r;
    };
    bf16x8 rg[Tg::N];
    const int g_row = tid / Tg::PIECES, g_col = (tid - g_row * Tg::PIECES) * 8;
    const uint32_t g_at = g_row < Tg::ROWS && g_col < g.P ? uint32_t(g_row * g.P + g_col) * 2 : kFactorNowhere;
    auto request = [&](int t) {
        uint32_t go = g_at;
        asm volatile("" : "+v"(go));
#pragma unroll
        for (int n = 0; n < Tg::N; ++n) rg[n] = factor_fetch(g.in + int64_t(t) * g.Q * g.P, g.Q * g.P * 2, go + uint32_t(n * Tg::ROWS * g.P * 2));
    };
    const int y_row = tid / Ty::PIECES, y_col = (tid - y_row * Ty::PIECES) * 8;
    constexpr bool HOLD = (A32 * P32 + B32 * Q32) * 4 <= kFactorHeld;
    bf16x8 u1[A32][P32], u2[B32][Q32];
    auto request_first = [&]() {
#pragma unroll
        for (int i = 0; i < A32; ++i)
#pragma unroll
            for (int ks = 0; ks < P32; ++ks) u1[i][ks] = factor_operand(g.first, g.size_first, g.nks_first, wr * A32 + i, ks, lane);
    };
    auto request_second = [&]() {
#pragma unroll
        for (int j = 0; j < B32; ++j)
#pragma unroll
            for (int ks = 0; ks < Q32; ++ks) u2[j][ks] = factor_operand(g.second, g.size_second, g.nks_second, wc * B32 + j, ks, lane);
    };
    const floatx4 none = {0.f, 0.f, 0.f, 0.f};
    if (int(blockIdx.x) >= g.tokens) return;
    request(blockIdx.x);
    if constexpr (HOLD) {
        request_first();
        request_second();
    }
    for (int t = blockIdx.x; t < g.tokens; t += gridDim.x) {
        if (g_row < Tg::ROWS) {
#pragma unroll
            for (int n = 0; n < Tg::N; ++n)
                if ((n + 1) * Tg::ROWS <= LQ || n * Tg::ROWS + g_row < LQ) *reinterpret_cast<bf16x8*>(sG + (n * Tg::ROWS + g_row) * PG + g_col) = rg[n];
        }
        {
            bf16x8 f[P32][Q32];
            if constexpr (!HOLD) request_first();
            __syncthreads();
            if (t + int(gridDim.x) < g.tokens) request(t + gridDim.x);
            floatx4 acc[A32][Q32];
#pragma unroll
            for (int i = 0; i < A32; ++i)
#pragma unroll
                for (int j = 0; j < Q32; ++j) acc[i][j] = none;
#pragma unroll
            for (int ks = 0; ks < P32; ++ks)
#pragma unroll
                for (int j = 0; j < Q32; ++j) f[ks][j] = plain(sG, PG, wc * Q32 + j, ks);
#pragma unroll
            for (int ks = 0; ks < P32; ++ks)
#pragma unroll
                for (int i = 0; i < A32; ++i)
#pragma unroll
                    for (int j = 0; j < Q32; ++j) acc[i][j] = mma(f[ks][j], u1[i][ks], acc[i][j]);
            // T [a][q], its q in the registers of an accumulator
#pragma unroll
            for (int i = 0; i < A32; ++i)
#pragma unroll
                for (int j = 0; j < Q32; ++j)
                    *reinterpret_cast<bf16x4_t*>(sT + ((wr * A32 + i) * 16 + l16) * PT + (wc * Q32 + j) * 16 + 4 * h) = round4(acc[i][j]);
        }
        if constexpr (!HOLD) request_second();
        __syncthreads();
        floatx4 o[A32][B32];
#pragma unroll
        for (int i = 0; i < A32; ++i)
#pragma unroll
            for (int j = 0; j < B32; ++j) o[i][j] = none;
        {
#pragma unroll
            for (int s = 0; s < Q32; ++s) {
                bf16x8 f[A32];
#pragma unroll
                for (int i = 0; i < A32; ++i) f[i] = plain(sT, PT, wr * A32 + i, s);
#pragma unroll
                for (int i = 0; i < A32; ++i)
#pragma unroll
                    for (int j = 0; j < B32; ++j) o[i][j] = mma(u2[j][s], f[i], o[i][j]);
                __builtin_amdgcn_sched_barrier(0);
            }
        }
        __syncthreads();                                            // G and T have been read: Y takes their place
#pragma unroll
        for (int i = 0; i < A32; ++i)
#pragma unroll
            for (int j = 0; j < B32; ++j)
                *reinterpret_cast<bf16x4_t*>(sY + ((wr * A32 + i) * 16 + l16) * PY + (wc * B32 + j) * 16 + 4 * h) = round4(o[i][j]);
        __syncthreads();
        bf16_t* Y = g.out + int64_t(t) * g.A * g.B;
        if (y_row < Ty::ROWS && y_col < g.B) {
#pragma unroll
            for (int n = 0; n < Ty::N; ++n)
                if (n * Ty::ROWS + y_row < g.A) *reinterpret_cast<bf16x8*>(Y + (n * Ty::ROWS + y_row) * g.B + y_col) = *reinterpret_cast<const bf16x8*>(sY + (n * Ty::ROWS + y_row) * PY + y_col);
        }
        __syncthreads();                                            // Y has left
    }
#endif
}
