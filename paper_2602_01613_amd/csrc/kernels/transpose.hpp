// Transposed copies that make an operand of the matrix-product kernel out of a matrix whose slow index is contracted.
// Part of the tn_linear library's single translation unit: included by tn_linear.hip inside its
// anonymous namespace, after kernels/common.hpp.
#pragma once

// ---------------------------------------------------------------------------------------------
// src [T][D] row-major, D % 8 == 0 -> dst with rows d and k = t, zeros for t in [T, Tp): row-major [D][Tp], or packed
// fragment-major (columns d). With a table, d goes to row or column to[d] instead. Tp % 64 == 0. Bound by memory: a workgroup takes 64 x 64 elements through LDS, reads rows of
// 128 bytes and writes rows of 128 bytes (packed: 16-byte chunks of 8 t, 32 neighbouring d = 512 bytes together). The LDS
// rows are 65 words of 4 bytes (two neighbouring t) long, so that the 8 d of a loaded piece and the t of a stored chunk both
// go over different banks.
// ---------------------------------------------------------------------------------------------
struct TransposeArgs {
    const bf16_t* src;
    bf16_t* dst;
    int64_t T, D, Tp;
    int32_t packed;
    const int32_t* to;
};

// Up to kTransposeMany matrices in one launch, blockIdx.y says which.
constexpr int kTransposeMany = 4;
struct TransposeMany {
    TransposeArgs m[kTransposeMany];
};

__global__ void __launch_bounds__(256) transpose_kernel(TransposeMany many) {
    __shared__ uint32_t tile[32][65];                    // [t / 2][d]: t even in the low half
    const TransposeArgs& p = many.m[blockIdx.y];
    const uint32_t across = uint32_t((p.D + 63) >> 6), down = blockIdx.x / across;
    const int64_t t0 = int64_t(down) * 64, d0 = int64_t(blockIdx.x - down * across) * 64;
    if (t0 >= p.Tp) return;
    const int tid = threadIdx.x;
    {
        // a thread: rows t0 + 2 * (tid / 8), + 1, eight d
        const int tp = tid >> 3, dp = (tid & 7) * 8;
        const int64_t t = t0 + 2 * tp, d = d0 + dp;
        typedef uint16_t u16x8 __attribute__((ext_vector_type(8)));
        u16x8 v[2] = {u16x8(0), u16x8(0)};
#pragma unroll
        for (int j = 0; j < 2; ++j)
            if (t + j < p.T && d < p.D) v[j] = *reinterpret_cast<const u16x8*>(p.src + (t + j) * p.D + d);
#pragma unroll
        for (int e = 0; e < 8; ++e) tile[tp][dp + e] = uint32_t(v[0][e]) | uint32_t(v[1][e]) << 16;
    }
    __syncthreads();
#pragma unroll
    for (int j = 0; j < 2; ++j) {
        // a chunk: one d, eight t. Packed: lanes along d; row-major: eight lanes along t
        const int i = tid + 256 * j;
        const int dl = p.packed ? i & 63 : i >> 3, tq = p.packed ? i >> 6 : i & 7;
        uint4 o;
        o.x = tile[4 * tq][dl];
        o.y = tile[4 * tq + 1][dl];
        o.z = tile[4 * tq + 2][dl];
        o.w = tile[4 * tq + 3][dl];
        const int64_t d = d0 + dl, t = t0 + 8 * tq;
        if (d < p.D) {
            const int64_t to = p.to ? p.to[d] : d;
            *reinterpret_cast<uint4*>(p.dst + (p.packed ? bfrag_offset(int(to), int(t), int(p.Tp >> 4)) : to * p.Tp + t)) = o;
        }
    }
}
