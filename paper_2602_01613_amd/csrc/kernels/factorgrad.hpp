// Gradients of the two factors on one side of a Tucker core, in one pass over the tokens.
// Part of the tn_linear library's single translation unit: included by tn_linear.hip inside its
// anonymous namespace, after kernels/grad.hpp.
#pragma once

// ---------------------------------------------------------------------------------------------
// A factor pair applies U1 [A][P] and U2 [B][Q] to a token's matrix from both sides: with Y [A][B] the token on the side of the
// modes and G [Q][P] the one on the side of the core, Y_t = U1 G_t^T U2^T for the out-factors (Y: dY, G: the core's output), and
// G_t^T = U1^T Y_t U2 for the in-factors (Y: x, G: the gradient of the core's input). Either way the gradients are
//     S_t = Y_t U2 [A][Q]      T_t = U1 G_t^T [A][Q]
//     dU1 = sum_t S_t G_t      dU2 = sum_t Y_t^T T_t      and, for the out-factors, dG_t = (U1^T S_t)^T
// with S and T rounded to bf16 as the step-by-step walk rounds them (they are a step's saved input and a step's gradient there).
//
// Bound by latency and memory at the token counts a fine-tuning step has, a few tokens per compute unit: 500 tokens of 160 x 160
// with ranks of 96 are 9.3 GFLOP (7 us of the matrix cores), 44 MB in and out and 31 MB of sums. 25 us here, and 8 for the in-factors
// (64 x 80, ranks 48); step by step every product was a launch, T went through memory and the gradients' rows through LDS 32 at a
// time: 102 us and 47.
//   * a workgroup takes a token at a time: Y and G go to LDS through registers (requested while the token before is multiplied),
//     S and T pass through LDS between the two halves of the work, both transposed ([q][a]), which is how the accumulators leave in
//     8-byte pieces and what the products that contract a read in 16-byte ones; the others use the transposing read;
//   * four waves 2 x 2: each holds its quarter of dU1 and dU2 in accumulators over all of its tokens; its share of the factors is
//     read from L2 for every token, ahead of its use (all three forms of them kept in registers spilled). Eight waves, one product
//     of each half of the work to four of them, took 29 us: 256 registers do not hold the token that is on its way;
//   * the operands of a k-step are requested ahead of the products of the one before (as the compiler orders them by itself every
//     three products wait for a read: 13 us a token instead of 8.5);
//   * rows in LDS are 16 bytes longer than the data, an odd number of 16-byte units: sixteen rows of a read lie on all banks;
//   * extents are padded to multiples of 32 with zeros (in LDS and in the factors' registers), nothing of which is stored.
// Every workgroup leaves its sums; grad_reduce_many_kernel adds them in workgroup order.
// ---------------------------------------------------------------------------------------------
struct FactorGradArgs {
    const bf16_t *Y, *G;                    // [token][A][B], [token][Q][P]
    bf16_t* dG;                             // [token][Q][P], or null
    const bf16_t *u2t, *u1, *u1t;           // packed fragment-major: columns q, k = b; columns a, k = p; columns p, k = a (with dG)
    int32_t nks_u2t, nks_u1, nks_u1t;       // k-steps of 16 of those
    int32_t size_u2t, size_u1, size_u1t;    // bytes of those
    float *sums1, *sums2;                   // [workgroup][A][P], [workgroup][B][Q]
    int32_t A, B, P, Q;                     // multiples of 16
    int32_t tokens;
};

template <int A32, int B32, int P32, int Q32>
constexpr size_t factor_grad_smem() {
    return size_t(2) * (32 * A32 * (32 * B32 + 8) + 32 * Q32 * (32 * P32 + 8) + 2 * 32 * Q32 * (32 * A32 + 8));
}

template <int A32, int B32, int P32, int Q32>
__global__ void __launch_bounds__(256, 1) factor_grad_kernel(FactorGradArgs g) {
#ifdef __HIP_DEVICE_COMPILE__
    constexpr int LA = 32 * A32, LB = 32 * B32, LP = 32 * P32, LQ = 32 * Q32;
    constexpr int PY = LB + 8, PG = LP + 8, PS = LA + 8;           // LDS rows, in elements
    constexpr int CY = LB / 8, CG = LP / 8;                        // 16-byte pieces of a row
    constexpr int RY = 256 / CY, RG = 256 / CG;                    // rows that the workgroup brings at a time
    constexpr int NY = (LA + RY - 1) / RY, NG = (LQ + RG - 1) / RG;
    typedef short shortx4 __attribute__((ext_vector_type(4)));
    typedef __bf16 bf16x4_t __attribute__((ext_vector_type(4)));
    typedef __attribute__((address_space(3))) shortx4 lds_x4;
    extern __shared__ __attribute__((aligned(16))) unsigned char dyn_smem[];
    bf16_t* sY = reinterpret_cast<bf16_t*>(dyn_smem);
    bf16_t* sG = sY + LA * PY;
    bf16_t* sS = sG + LQ * PG;
    bf16_t* sT = sS + LQ * PS;
    const int tid = threadIdx.x, lane = tid & 63, l16 = lane & 15, h = lane >> 4;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6), wr = wave >> 1, wc = wave & 1;
    // loads through a buffer descriptor: what lies past the end is zero
    typedef uint32_t uintx4 __attribute__((ext_vector_type(4)));
    constexpr uint32_t NOWHERE = 0x80000000u;
    auto fetch = [](const bf16_t* p, int size, uint32_t at) {
        const __amdgpu_buffer_rsrc_t r = __builtin_amdgcn_make_buffer_rsrc(const_cast<bf16_t*>(p), 0, size, 0x00020000);
        union { uintx4 u; bf16x8 v; } x;
        x.u = __builtin_amdgcn_raw_buffer_load_b128(r, int(at), 0, 0);
        return x.v;
    };
    // operands of a 16 x 16 x 32 product: lane l supplies row (column) l % 16, k = 8 * (l / 16) .. + 7; see bfrag_offset
    auto factor = [&](const bf16_t* src, int size, int nks, int tile, int ks) {
        uint32_t at = uint32_t((h >> 1) * 1024 + (l16 + 32 * (h & 1)) * 16);
        asm volatile("" : "+v"(at));                               // (not one register per load throughout)
        at += uint32_t(((tile >> 1) * nks + ks * 2) * 1024 + (tile & 1) * 256);
        return fetch(src, size, ks * 2 + (h >> 1) < nks ? at : NOWHERE);
    };
    bf16x8 u2t[Q32][B32], u1[A32][P32];
    auto request_u2 = [&]() {
#pragma unroll
        for (int j = 0; j < Q32; ++j)
#pragma unroll
            for (int ks = 0; ks < B32; ++ks) u2t[j][ks] = factor(g.u2t, g.size_u2t, g.nks_u2t, wc * Q32 + j, ks);
    };
    auto request_u1 = [&]() {
#pragma unroll
        for (int i = 0; i < A32; ++i)
#pragma unroll
            for (int ks = 0; ks < P32; ++ks) u1[i][ks] = factor(g.u1, g.size_u1, g.nks_u1, wr * A32 + i, ks);
    };

    auto plain = [&](const bf16_t* s, int pitch, int tile, int ks) {
        return *reinterpret_cast<const bf16x8*>(s + (tile * 16 + l16) * pitch + ks * 32 + 8 * h);
    };
    // rows are k: four rows of 16 columns per 16 lanes and read
    auto turned = [&](const bf16_t* s, int pitch, int tile, int ks) {
        const bf16_t* p = s + (ks * 32 + 8 * h + (l16 >> 2)) * pitch + tile * 16 + 4 * (l16 & 3);
        union { shortx4 u[2]; bf16x8 v; } r;
        r.u[0] = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_x4*)(p));
        r.u[1] = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_x4*)(p + 4 * pitch));
        return r.v;
    };
    auto mma = [&](bf16x8 a, bf16x8 b, floatx4 c) { return __builtin_amdgcn_mfma_f32_16x16x32_bf16(a, b, c, 0, 0, 0); };
    auto round4 = [&](floatx4 v) {
        bf16x4_t r;
#pragma unroll
        for (int e = 0; e < 4; ++e) r[e] = bf16_t(v[e]);
        return r;
    };

    bf16x8 ry[NY], rg[NG];
    const int y_row = tid / CY, y_col = (tid - y_row * CY) * 8, g_row = tid / CG, g_col = (tid - g_row * CG) * 8;
    const uint32_t y_at = y_row < RY && y_col < g.B ? uint32_t(y_row * g.B + y_col) * 2 : NOWHERE;
    const uint32_t g_at = g_row < RG && g_col < g.P ? uint32_t(g_row * g.P + g_col) * 2 : NOWHERE;
    auto request = [&](int t) {
        uint32_t yo = y_at, go = g_at;
        asm volatile("" : "+v"(yo), "+v"(go));
#pragma unroll
        for (int n = 0; n < NY; ++n) ry[n] = fetch(g.Y + int64_t(t) * g.A * g.B, g.A * g.B * 2, yo + uint32_t(n * RY * g.B * 2));
#pragma unroll
        for (int n = 0; n < NG; ++n) rg[n] = fetch(g.G + int64_t(t) * g.Q * g.P, g.Q * g.P * 2, go + uint32_t(n * RG * g.P * 2));
    };
    auto deposit = [&]() {
        if (y_row < RY) {
#pragma unroll
            for (int n = 0; n < NY; ++n)
                if ((n + 1) * RY <= LA || n * RY + y_row < LA) *reinterpret_cast<bf16x8*>(sY + (n * RY + y_row) * PY + y_col) = ry[n];
        }
        if (g_row < RG) {
#pragma unroll
            for (int n = 0; n < NG; ++n)
                if ((n + 1) * RG <= LQ || n * RG + g_row < LQ) *reinterpret_cast<bf16x8*>(sG + (n * RG + g_row) * PG + g_col) = rg[n];
        }
    };

    floatx4 d1[A32][P32], d2[B32][Q32];
    const floatx4 none = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int i = 0; i < A32; ++i)
#pragma unroll
        for (int j = 0; j < P32; ++j) d1[i][j] = none;
#pragma unroll
    for (int i = 0; i < B32; ++i)
#pragma unroll
        for (int j = 0; j < Q32; ++j) d2[i][j] = none;

    request(blockIdx.x);
    request_u2();
    for (int t = blockIdx.x; t < g.tokens; t += gridDim.x) {
        deposit();
        request_u1();
        __syncthreads();
        if (t + int(gridDim.x) < g.tokens) request(t + gridDim.x);
        // S and T, their a in the registers of an accumulator: [q][a] in 8-byte pieces.
        {
            floatx4 acc[A32][Q32];
            bf16x8 f[2][A32 > Q32 ? A32 : Q32];
            auto clear = [&]() {
#pragma unroll
                for (int i = 0; i < A32; ++i)
#pragma unroll
                    for (int j = 0; j < Q32; ++j) acc[i][j] = none;
            };
            auto leave = [&](bf16_t* to) {
#pragma unroll
                for (int i = 0; i < A32; ++i)
#pragma unroll
                    for (int j = 0; j < Q32; ++j)
                        *reinterpret_cast<bf16x4_t*>(to + ((wc * Q32 + j) * 16 + l16) * PS + (wr * A32 + i) * 16 + 4 * h) = round4(acc[i][j]);
            };
            auto read = [&](int s) {
                if (s < B32) {
#pragma unroll
                    for (int i = 0; i < A32; ++i) f[s & 1][i] = plain(sY, PY, wr * A32 + i, s);
                } else if (s < B32 + P32) {
#pragma unroll
                    for (int j = 0; j < Q32; ++j) f[s & 1][j] = plain(sG, PG, wc * Q32 + j, s - B32);
                }
            };
            clear();
            read(0);
#pragma unroll
            for (int s = 0; s < B32 + P32; ++s) {
                read(s + 1);
                __builtin_amdgcn_sched_barrier(0);
#pragma unroll
                for (int i = 0; i < A32; ++i)
#pragma unroll
                    for (int j = 0; j < Q32; ++j)
                        acc[i][j] = s < B32 ? mma(f[s & 1][i], u2t[j][s], acc[i][j]) : mma(u1[i][s - B32], f[s & 1][j], acc[i][j]);
                if (s == B32 - 1) {
                    leave(sS);
                    clear();
                }
                __builtin_amdgcn_sched_barrier(0);
            }
            leave(sT);
        }
        __syncthreads();
        bf16x8 u1t[P32][A32];
        if (g.dG) {
#pragma unroll
            for (int i = 0; i < P32; ++i)
#pragma unroll
                for (int ks = 0; ks < A32; ++ks) u1t[i][ks] = factor(g.u1t, g.size_u1t, g.nks_u1t, wr * P32 + i, ks);
        }
        // dU1, dG and dU2
        {
            constexpr int S1 = Q32, S2 = Q32 + A32, S3 = Q32 + 2 * A32, WIDE = A32 > B32 ? A32 : B32, NARROW = P32 > Q32 ? P32 : Q32;
            floatx4 acc[P32][Q32];
            bf16x8 fw[2][WIDE], fn[2][NARROW];
#pragma unroll
            for (int i = 0; i < P32; ++i)
#pragma unroll
                for (int j = 0; j < Q32; ++j) acc[i][j] = none;
            auto read = [&](int s) {
                if (s < S1) {
#pragma unroll
                    for (int j = 0; j < P32; ++j) fn[s & 1][j] = turned(sG, PG, wc * P32 + j, s);
#pragma unroll
                    for (int i = 0; i < A32; ++i) fw[s & 1][i] = turned(sS, PS, wr * A32 + i, s);
                } else if (s < S2) {
#pragma unroll
                    for (int j = 0; j < Q32; ++j) fn[s & 1][j] = plain(sS, PS, wc * Q32 + j, s - S1);
                } else if (s < S3) {
#pragma unroll
                    for (int j = 0; j < Q32; ++j) fn[s & 1][j] = plain(sT, PS, wc * Q32 + j, s - S2);
#pragma unroll
                    for (int i = 0; i < B32; ++i) fw[s & 1][i] = turned(sY, PY, wr * B32 + i, s - S2);
                }
            };
            read(0);
#pragma unroll
            for (int s = 0; s < S3; ++s) {
                read(s + 1);
                __builtin_amdgcn_sched_barrier(0);
                if (s < S1) {
#pragma unroll
                    for (int i = 0; i < A32; ++i)
#pragma unroll
                        for (int j = 0; j < P32; ++j) d1[i][j] = mma(fw[s & 1][i], fn[s & 1][j], d1[i][j]);
                } else if (s < S2) {
                    if (g.dG) {
#pragma unroll
                        for (int i = 0; i < P32; ++i)
#pragma unroll
                            for (int j = 0; j < Q32; ++j) acc[i][j] = mma(u1t[i][s - S1], fn[s & 1][j], acc[i][j]);
                    }
                } else {
#pragma unroll
                    for (int i = 0; i < B32; ++i)
#pragma unroll
                        for (int j = 0; j < Q32; ++j) d2[i][j] = mma(fw[s & 1][i], fn[s & 1][j], d2[i][j]);
                }
                if (s == S2 - 1 && g.dG) {
                    bf16_t* dG = g.dG + int64_t(t) * g.Q * g.P;
#pragma unroll
                    for (int i = 0; i < P32; ++i)
#pragma unroll
                        for (int j = 0; j < Q32; ++j) {
                            const int p = (wr * P32 + i) * 16 + 4 * h, q = (wc * Q32 + j) * 16 + l16;
                            if (p < g.P && q < g.Q) *reinterpret_cast<bf16x4_t*>(dG + q * g.P + p) = round4(acc[i][j]);
                        }
                }
                __builtin_amdgcn_sched_barrier(0);
            }
        }
        __builtin_amdgcn_sched_barrier(0);
        if (t + int(gridDim.x) < g.tokens) request_u2();
        __syncthreads();                                            // everyone has read this token
    }

    // lane l, register v: row 4 * (l / 16) + v, column l % 16
    float* s1 = g.sums1 + int64_t(blockIdx.x) * g.A * g.P;
    float* s2 = g.sums2 + int64_t(blockIdx.x) * g.B * g.Q;
#pragma unroll
    for (int i = 0; i < A32; ++i)
#pragma unroll
        for (int j = 0; j < P32; ++j) {
            const int a = (wr * A32 + i) * 16 + 4 * h, p = (wc * P32 + j) * 16 + l16;
#pragma unroll
            for (int v = 0; v < 4; ++v)
                if (a < g.A && p < g.P) s1[(a + v) * g.P + p] = d1[i][j][v];
        }
#pragma unroll
    for (int i = 0; i < B32; ++i)
#pragma unroll
        for (int j = 0; j < Q32; ++j) {
            const int b = (wr * B32 + i) * 16 + 4 * h, q = (wc * Q32 + j) * 16 + l16;
#pragma unroll
            for (int v = 0; v < 4; ++v)
                if (b < g.B && q < g.Q) s2[(b + v) * g.Q + q] = d2[i][j][v];
        }
#endif
}
