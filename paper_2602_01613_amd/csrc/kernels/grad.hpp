// Gradients with respect to the parameter tensors: the contraction step with the token index contracted.
// Part of the tn_linear library's single translation unit: included by tn_linear.hip inside its
// anonymous namespace, after kernels/stream.hpp.
#pragma once

// ---------------------------------------------------------------------------------------------
// A forward step computes Out[t, r, c] = sum_k In[t, r, k] P[c][k]. With dOut the gradient of the loss with
// respect to the step's output (Section 3.4: the factors are fine-tuned, so the loss is back-propagated through
// every contraction), the gradient with respect to the step's parameter tensor is the same contraction with the
// rows (tokens and row indices) summed instead of k:
//     dP[c][k] = sum_{t, r} dOut[t, r, c] * In[t, r, k]
// and the gradient with respect to its input, dIn[t, r, k] = sum_c dOut[t, r, c] P[c][k], is an ordinary step
// with the packed tensor transposed, which the step kernels run as they are (dOut is read through the forward
// step's scatter tables as gather tables).
// grad_param_kernel: a workgroup owns a 64 x 64 tile of (c, k) and a range of rows; rows go through LDS 16 at a
// time, plain fp32 FMA, any dtype, any addressing. The row range is split over workgroups when C*K alone would not
// fill the chip; every split writes its own fp32 tile and grad_reduce_kernel adds them in split order (no
// atomics: results are bit-reproducible) and scatters the sum to the caller's tensor layout.
// ---------------------------------------------------------------------------------------------
struct GradArgs {
    const void* dOut;
    const void* In;
    float* partial;            // [n_split][C][K]
    const int32_t* crow;       // position of (r, c) in a token of dOut: crow[r] + ccol[c]
    const int32_t* ccol;
    const int32_t* arow;       // position of (r, k) in a token of In: arow[r] + acol[k]; null: r*K + k
    const int32_t* acol;
    int64_t c_tok_stride, a_tok_stride;
    uint32_t total_rows, R;
    int32_t K, C;
    uint32_t rows_per_split;
    int32_t c_tiles, k_tiles, n_split;      // grad_param_mfma_kernel: a one-dimensional grid of c_tiles * k_tiles * n_split workgroups
    int32_t d_mode, i_mode;                 // grad_param_mfma_kernel: how dOut and In are loaded (see there)
};

template <typename T>
__global__ void __launch_bounds__(256) grad_param_kernel(GradArgs a) {
    constexpr int BC = 64, BK = 64, BG = 16;
    __shared__ float sD[BG][BC + 4];
    __shared__ float sI[BG][BK + 4];
    const T* dOut = static_cast<const T*>(a.dOut);
    const T* In = static_cast<const T*>(a.In);
    const int tid = threadIdx.x;
    const int c0 = blockIdx.x * BC, k0 = blockIdx.y * BK;
    const uint32_t g_begin = blockIdx.z * a.rows_per_split;
    const uint32_t g_end = min(a.total_rows, g_begin + a.rows_per_split);
    const int tx = tid & 15, ty = tid >> 4;            // thread: c = c0 + 4*ty .. +3, k = k0 + 4*tx .. +3
    float acc[4][4] = {};
    for (uint32_t g0 = g_begin; g0 < g_end; g0 += BG) {
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            const int e = tid + 256 * j;
            const int gg = e >> 6, cc = e & 63;
            const uint32_t g = g0 + gg;
            float vd = 0.f, vi = 0.f;
            if (g < g_end) {
                const uint32_t t = g / a.R;
                const uint32_t r = g - t * a.R;
                if (c0 + cc < a.C) vd = to_float(dOut[int64_t(t) * a.c_tok_stride + a.crow[r] + a.ccol[c0 + cc]]);
                if (k0 + cc < a.K)
                    vi = to_float(In[int64_t(t) * a.a_tok_stride +
                                     (a.arow ? int64_t(a.arow[r]) + a.acol[k0 + cc] : int64_t(r) * a.K + k0 + cc)]);
            }
            sD[gg][cc] = vd;
            sI[gg][cc] = vi;
        }
        __syncthreads();
#pragma unroll
        for (int gg = 0; gg < BG; ++gg) {
            float dv[4], iv[4];
#pragma unroll
            for (int i = 0; i < 4; ++i) dv[i] = sD[gg][ty * 4 + i];
#pragma unroll
            for (int j = 0; j < 4; ++j) iv[j] = sI[gg][tx * 4 + j];
#pragma unroll
            for (int i = 0; i < 4; ++i)
#pragma unroll
                for (int j = 0; j < 4; ++j) acc[i][j] = fmaf(dv[i], iv[j], acc[i][j]);
        }
        __syncthreads();
    }
    float* out = a.partial + int64_t(blockIdx.z) * a.C * a.K;
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        const int c = c0 + ty * 4 + i;
        if (c >= a.C) continue;
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            const int k = k0 + tx * 4 + j;
            if (k < a.K) out[int64_t(c) * a.K + k] = acc[i][j];
        }
    }
}

// The same contraction on the matrix cores, for bf16 layers: a workgroup owns a 128 x 128 tile of (c, k), each of
// its four waves a 64 x 64 quarter (2 x 2 MFMA tiles, fp32 accumulators). The contracted index is the row g, which
// is the slow index of both operands in memory, while an MFMA lane supplies 8 consecutive values of the contracted
// index: so the rows go through LDS 32 at a time, stored transposed ([column][g]), and a fragment is one 16-byte LDS
// read. Waves 0-1 bring the 128 x 32 block of dOut, waves 2-3 that of In, each through the forward step's own tables,
// in the widest pieces the operand's layout allows (GradArgs::d_mode, i_mode):
//   1  8 consecutive columns of a row are one aligned 16-byte piece: a thread loads 4 rows x 8 columns, transposes
//      them in registers and writes 8 pieces of 4 consecutive g;
//   2  8 consecutive rows of a column are one aligned 16-byte piece (dOut of a step whose output runs along the row
//      index; R % 8 == 0): such a piece is 8 consecutive g as it stands;
//   0  neither: one element per lane and load, lanes along the columns of one row (the row of a load is the same
//      for the whole wave, so its token and table entry sit in scalar registers).
// The loads of the next 32 rows are requested before the current ones are multiplied. Row ranges start at multiples
// of 32. Partial tiles as in grad_param_kernel.
__global__ void __launch_bounds__(256) grad_param_mfma_kernel(GradArgs a) {
    // LDS row of column x: 32 + 8 bf16 (80 bytes), and every 8 columns 16 bytes more, so that the 8-byte writes of
    // mode 1 (lanes 8 columns = 640 bytes apart) do not all fall on one bank
    constexpr int BT = 128, BG = 32, PITCH = BG + 8, LDS_ELEMS = BT * PITCH + (BT / 8) * 8;
    auto row_of = [](int x) { return x * PITCH + ((x >> 3) << 3); };
    __shared__ __attribute__((aligned(16))) bf16_t sD[LDS_ELEMS];
    __shared__ __attribute__((aligned(16))) bf16_t sI[LDS_ELEMS];
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    // workgroup -> (tile, split). With a multiple of 8 splits, all tiles of one split run on one XCD (workgroups are
    // dealt to the 8 XCDs in turn): the rows of a split then come from memory once, into that XCD's L2, for all of its
    // tiles, instead of once per XCD.
    const int tiles = a.c_tiles * a.k_tiles;
    int tile, split;
    if ((a.n_split & 7) == 0) {
        const int xcd = blockIdx.x & 7, j = blockIdx.x >> 3;
        tile = j % tiles;
        split = (j / tiles) * 8 + xcd;
    } else {
        tile = blockIdx.x % tiles;
        split = blockIdx.x / tiles;
    }
    const int c0 = (tile % a.c_tiles) * BT, k0 = (tile / a.c_tiles) * BT;
    const uint32_t g_begin = min(a.total_rows, uint32_t(split) * a.rows_per_split);
    const uint32_t g_end = min(a.total_rows, g_begin + a.rows_per_split);

    // ---- this wave's operand (wave-uniform)
    const bool is_d = wave < 2;
    const bf16_t* src = static_cast<const bf16_t*>(is_d ? a.dOut : a.In);
    const int32_t* rowtab = is_d ? a.crow : a.arow;             // null: plain In, row r at r*K
    const int32_t* coltab = is_d ? a.ccol : a.acol;             // null: plain In, column k at k
    const int64_t tok_stride = is_d ? a.c_tok_stride : a.a_tok_stride;
    const int mode = is_d ? a.d_mode : a.i_mode;
    const int ext = is_d ? a.C : a.K, x0 = is_d ? c0 : k0;
    bf16_t* sdst = is_d ? sD : sI;
    const int u = tid & 127;
    // modes 0 and 2: thread -> column u; mode 1: thread -> (columns 8*(u%16) .. +7, rows 4*(u/16) .. +3 of the 32)
    const int col = x0 + (mode == 1 ? 8 * (u & 15) : u);
    const bool vcol = col < ext;                                // mode 1: ext % 8 == 0, the whole piece is inside
    // table entries are offsets inside one token: non-negative, below 2^31 (checked when the plan is built)
    const uint32_t coff = vcol ? (coltab ? uint32_t(coltab[col]) : uint32_t(col)) : 0u;
    bf16x8 reg[4];
    auto request = [&](uint32_t g0) {
        bf16x8 zero;
#pragma unroll
        for (int e = 0; e < 8; ++e) zero[e] = bf16_t(0.f);
        if (mode == 1) {
            // per-lane rows: g0 + 4*(u/16) + j
            uint32_t g = g0 + 4u * uint32_t(u >> 4);
            uint32_t t = g / a.R, r = g - t * a.R;
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                reg[j] = zero;
                if (g + uint32_t(j) < g_end && vcol) {
                    const int64_t ro = rowtab ? int64_t(rowtab[r]) : int64_t(r) * a.K;
                    reg[j] = *reinterpret_cast<const bf16x8*>(src + int64_t(t) * tok_stride + ro + coff);
                }
                if (++r == a.R) {
                    r = 0;
                    ++t;
                }
            }
        } else if (mode == 2) {
            // rows g0 + 8q .. +7: one token, one aligned run of the row table (R % 8 == 0, g0 % 8 == 0)
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                const uint32_t g = g0 + 8u * uint32_t(q);       // wave-uniform
                reg[q] = zero;
                if (g < g_end && vcol) {
                    const uint32_t t = g / a.R, r = g - t * a.R;
                    reg[q] = *reinterpret_cast<const bf16x8*>(src + (int64_t(t) * tok_stride + rowtab[r]) + coff);
                }
            }
        } else {
            uint32_t t = g0 / a.R, r = g0 - t * a.R;            // wave-uniform
            // all 32 row offsets first (scalar table reads, one wait), then the loads back to back
            int64_t ro[BG];
#pragma unroll
            for (int j = 0; j < BG; ++j) {
                ro[j] = g0 + uint32_t(j) < g_end ? int64_t(t) * tok_stride + (rowtab ? int64_t(rowtab[r]) : int64_t(r) * a.K) : -1;
                if (++r == a.R) {
                    r = 0;
                    ++t;
                }
            }
#pragma unroll
            for (int j = 0; j < BG; ++j)
                reg[j >> 3][j & 7] = (ro[j] >= 0 && vcol) ? (src + ro[j])[coff] : bf16_t(0.f);
        }
    };
    auto deposit = [&]() {
        if (mode == 1) {
            typedef __bf16 bf16x4_t __attribute__((ext_vector_type(4)));
            const int cl = 8 * (u & 15), gq = 4 * (u >> 4);
#pragma unroll
            for (int e = 0; e < 8; ++e) {
                bf16x4_t v;
#pragma unroll
                for (int j = 0; j < 4; ++j) v[j] = reg[j][e];
                *reinterpret_cast<bf16x4_t*>(sdst + row_of(cl + e) + gq) = v;
            }
        } else {
#pragma unroll
            for (int q = 0; q < 4; ++q) *reinterpret_cast<bf16x8*>(sdst + row_of(u) + 8 * q) = reg[q];
        }
    };
    // wave -> quarter (wc, wk); MFMA row operand: c, column operand: k; lane l supplies g = 8*(l/32) .. +7 of a k-step
    const int wc = wave >> 1, wk = wave & 1;
    floatx16 acc[2][2];
#pragma unroll
    for (int i = 0; i < 2; ++i)
#pragma unroll
        for (int j = 0; j < 2; ++j)
#pragma unroll
            for (int v = 0; v < 16; ++v) acc[i][j][v] = 0.f;
    if (g_begin < g_end) request(g_begin);
    for (uint32_t g0 = g_begin; g0 < g_end; g0 += BG) {
        deposit();
        __syncthreads();
        if (g0 + BG < g_end) request(g0 + BG);
#pragma unroll
        for (int ks = 0; ks < 2; ++ks) {
            bf16x8 fd[2], fi[2];
#pragma unroll
            for (int i = 0; i < 2; ++i) {
                fd[i] = *reinterpret_cast<const bf16x8*>(sD + row_of(64 * wc + 32 * i + (lane & 31)) + 16 * ks + 8 * (lane >> 5));
                fi[i] = *reinterpret_cast<const bf16x8*>(sI + row_of(64 * wk + 32 * i + (lane & 31)) + 16 * ks + 8 * (lane >> 5));
            }
#pragma unroll
            for (int i = 0; i < 2; ++i)
#pragma unroll
                for (int j = 0; j < 2; ++j) acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(fd[i], fi[j], acc[i][j], 0, 0, 0);
        }
        __syncthreads();                                        // everyone has read the group before it is overwritten
    }
    // lane l, register v of acc[i][j]: c = c0 + 64*wc + 32*i + 8*(v/4) + 4*(l/32) + v%4, k = k0 + 64*wk + 32*j + l%32
    float* out = a.partial + int64_t(split) * a.C * a.K;
#pragma unroll
    for (int i = 0; i < 2; ++i)
#pragma unroll
        for (int j = 0; j < 2; ++j) {
            const int k = k0 + 64 * wk + 32 * j + (lane & 31);
#pragma unroll
            for (int v = 0; v < 16; ++v) {
                const int c = c0 + 64 * wc + 32 * i + 8 * (v >> 2) + 4 * (lane >> 5) + (v & 3);
                if (c < a.C && k < a.K) out[int64_t(c) * a.K + k] = acc[i][j][v];
            }
        }
}

// ---------------------------------------------------------------------------------------------
// Both halves' gradients towards a narrow bond in one pass over dW. With D [F0][F1] the gradient of the matrix with its modes
// ordered by halves (stored [F1 / 32][F0][32]), in two bf16 parts (high, low: see step_gemm_kernel), and the halves P0 [F0][S], P1 [F1][S]:
//     dH0[f0][s] = sum_f1 D[f0][f1] P1[f1][s]        dH1[f1][s] = sum_f0 D[f0][f1] P0[f0][s]
// each as the fp32 product but for terms of 2^-16: D high and low with P high, D high with P low.
// Bound by memory: D (168 MB for 5120 x 8192) is larger than what the products, 2 S MACs an element of it, take on the matrix
// cores. As two products of step_gemm_kernel it was read twice, and for the second one transposed through memory first: 180 us at
// S = 64 for 4096 x 10240, 68 here with the launches that add the sums (51 for this one: 168 MB read and 59 MB of
// sums written, 4.4 TB/s).
//   * a workgroup owns 256 rows of D and walks over tiles of 32 columns of its range: 3 or 4 stages of (16 KB of each part of D and
//     the 32 columns' P1), direct to LDS. dW's product leaves D tile by tile, [F1 / 32][F0][32], so that a
//     workgroup's 16 KB lie together (as pieces of 64 bytes of row-major D, 3 stages: 69 us instead of 51). A wave holds the sums of dH0 for 64 rows in registers throughout;
//   * the 32 rows of dH1 that a tile gives are shared out to the waves, (16 columns) x (half of the bond), so that no sums cross
//     waves. D is contracted along its rows there: the operand is read with the transposing LDS read (ds_read_b64_tr_b16), and the
//     wave's 256 rows x half a bond of P0 stay in registers for the whole walk;
//   * 256 rows: the sums of dH1 leave per 256 rows of D, S/256 of D's fp32 size written and read again; with 512 there is no room for
//     P0 next to the sums;
//   * a 16-byte chunk c of a row of 64 bytes sits at c ^ (row / 4 % 4): the 16 rows of a read (or the 8 of a transposing one)
//     then fall on different banks.
// Columns of a range past its end load nothing (out of bounds).
// ---------------------------------------------------------------------------------------------
constexpr int kBondRows = 256, kBondCols = 32;
struct BondGradArgs {
    const void *D, *P0, *P1;               // D [F1 / 32][F0][32]; P0, P1 packed fragment-major, columns s, k = f0 (f1)
    int64_t d_lo, p0_lo, p1_lo;            // from a matrix to its low part, in elements
    float *sums0, *sums1;                  // [ranges][F0][S], [row panels][F1][S]
    int64_t F0, F1;                        // multiples of 64
    int32_t S;                             // 32 * S32
    int32_t tiles, tiles_per_range, ranges;      // of 32 columns; no range is empty
};

template <int S32>
struct BondGradShape {
    static constexpr int ST = 2 * S32;                              // 16-wide tiles of the bond
    static constexpr int D_BYTES = kBondRows * kBondCols * 2, P_BYTES = ST * 1024;
    static constexpr int STAGE = 2 * (D_BYTES + P_BYTES), NS = S32 < 3 ? 4 : 3;
    static constexpr size_t SMEM = size_t(NS) * STAGE;
};

template <int S32>
__global__ void __launch_bounds__(256, 1) bond_grad_kernel(BondGradArgs a) {
#ifdef __HIP_DEVICE_COMPILE__
    using Sh = BondGradShape<S32>;
    constexpr int ST = Sh::ST, SH = S32, STAGE = Sh::STAGE, NS = Sh::NS, D_BYTES = Sh::D_BYTES;
    constexpr int L = 8 + SH;                            // 1 KB loads per wave and stage: 4 of each part of D, SH of P1
    constexpr int KS = kBondRows / 32;
    typedef __attribute__((address_space(3))) void lds_t;
    typedef short shortx4 __attribute__((ext_vector_type(4)));
    extern __shared__ __attribute__((aligned(16))) unsigned char dyn_smem[];
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int panel = blockIdx.x / a.ranges, range = blockIdx.x - panel * a.ranges;
    const int64_t row0 = int64_t(panel) * kBondRows;
    const int tile0 = range * a.tiles_per_range, n = min(a.tiles, tile0 + a.tiles_per_range) - tile0;
    const int nks0 = int(a.F0 >> 4), nks1 = int(a.F1 >> 4);

    // P0: rows s of the wave's half of the bond, k-steps of 32 rows of D
    const int s_tile0 = (wave >> 1) * SH;
    bf16x8 p0[2][KS][SH];
    {
        const bf16_t* P0 = static_cast<const bf16_t*>(a.P0);
        bf16x8 zero;
#pragma unroll
        for (int e = 0; e < 8; ++e) zero[e] = bf16_t(0.f);
#pragma unroll
        for (int ks = 0; ks < KS; ++ks)
#pragma unroll
            for (int j = 0; j < SH; ++j) {
                p0[0][ks][j] = p0[1][ks][j] = zero;
                if (row0 + ks * 32 < a.F0) {             // a multiple of 64 rows: k-steps are whole
                    const bf16_t* src = P0 + bfrag_offset((s_tile0 + j) * 16 + (lane & 15), int(row0) + ks * 32 + 8 * (lane >> 4), nks0);
                    p0[0][ks][j] = *reinterpret_cast<const bf16x8*>(src);
                    p0[1][ks][j] = *reinterpret_cast<const bf16x8*>(src + a.p0_lo);
                }
            }
        // they have landed before the loop, whose waits count its own loads only
#pragma unroll
        for (int ks = 0; ks < KS; ++ks)
#pragma unroll
            for (int j = 0; j < SH; ++j) asm volatile("" : "+v"(p0[0][ks][j]), "+v"(p0[1][ks][j]));
    }

    // rows past the end load nothing, which leaves zeros: 64 rows of a wave are all there or none is
    const bf16_t* D = static_cast<const bf16_t*>(a.D) + row0 * kBondCols;
    const int d_tile = int(a.F0) * kBondCols * 2;
    const __amdgpu_buffer_rsrc_t rd = __builtin_amdgcn_make_buffer_rsrc(const_cast<bf16_t*>(D), 0, 0x7fffffff, 0x00020000);
    const __amdgpu_buffer_rsrc_t rl = __builtin_amdgcn_make_buffer_rsrc(const_cast<bf16_t*>(D + a.d_lo), 0, 0x7fffffff, 0x00020000);
    const int vd = row0 + wave * 64 < a.F0 ? wave * 4096 + (lane >> 2) * 64 + ((lane & 3) ^ ((lane >> 4) & 3)) * 16 : int(0x80000000u);
    const bf16_t* P1 = static_cast<const bf16_t*>(a.P1);
    const int p_size = a.S * int(a.F1) * 2;
    auto issue = [&](int t, int stage) {
        unsigned char* s = dyn_smem + stage * STAGE;
        const int off = t < n ? 0 : int(0x80000000u), tile = tile0 + t;
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            const int so = tile * d_tile + q * 1024;
            __builtin_amdgcn_raw_ptr_buffer_load_lds(rd, (lds_t*)(s + (wave * 4 + q) * 1024), 16, vd | off, so, 0, 0);
            __builtin_amdgcn_raw_ptr_buffer_load_lds(rl, (lds_t*)(s + D_BYTES + (wave * 4 + q) * 1024), 16, vd | off, so, 0, 0);
        }
#pragma unroll
        for (int q = 0; q < SH; ++q) {
            // block j % ST: (32 columns of the bond) x (16 k), of the high part, then of the low one
            const int j = wave + 4 * q, b = j < ST ? j : j - ST;
            __builtin_amdgcn_raw_ptr_buffer_load_lds(
                __builtin_amdgcn_make_buffer_rsrc(const_cast<bf16_t*>(P1 + (j < ST ? 0 : a.p1_lo)), 0, p_size, 0x00020000),
                (lds_t*)(s + 2 * D_BYTES + j * 1024), 16, (lane * 16) | off, ((b >> 1) * nks1 + tile * 2 + (b & 1)) * 1024, 0, 0);
        }
    };

    // fragments: lane l supplies row (column) l%16 and k = 8*(l/16) .. +7
    const int od = (wave * 64 + (lane & 15)) * 64 + (((lane >> 4) ^ ((lane >> 2) & 3)) * 16);
    const int op = 2 * D_BYTES + (lane >> 5) * 1024 + ((lane & 15) + 32 * ((lane >> 4) & 1)) * 16;
    int ot[2];                                           // transposing read: four rows of 16 columns per 16 lanes
#pragma unroll
    for (int h = 0; h < 2; ++h) {
        const int row = 8 * (lane >> 4) + 4 * h + ((lane & 15) >> 2), chunk = 2 * (wave & 1) + ((lane & 3) >> 1);
        ot[h] = row * 64 + ((chunk ^ ((row >> 2) & 3)) * 16) + (lane & 1) * 8;
    }
    auto read8 = [&](const unsigned char* p) { return *reinterpret_cast<const bf16x8*>(p); };
    // four k-steps of both parts, [k-step][part]. (One block with its own wait: before the builtin of this read the compiler waits
    // for every load to LDS that is in flight, the next tiles' among them.)
    const uint32_t lds0 = uint32_t(uintptr_t((lds_t*)dyn_smem));
    auto read_t4 = [&](int at, bf16x8 (&f)[4][2]) {
        shortx4 u[16];
        const uint32_t a0 = lds0 + uint32_t(at + ot[0]), a1 = lds0 + uint32_t(at + ot[1]);
        static_assert(D_BYTES == 16384 && kBondCols * 64 == 2048, "offsets below");
        asm volatile(
            "ds_read_b64_tr_b16 %0, %16\n\tds_read_b64_tr_b16 %1, %17\n\t"
            "ds_read_b64_tr_b16 %2, %16 offset:16384\n\tds_read_b64_tr_b16 %3, %17 offset:16384\n\t"
            "ds_read_b64_tr_b16 %4, %16 offset:2048\n\tds_read_b64_tr_b16 %5, %17 offset:2048\n\t"
            "ds_read_b64_tr_b16 %6, %16 offset:18432\n\tds_read_b64_tr_b16 %7, %17 offset:18432\n\t"
            "ds_read_b64_tr_b16 %8, %16 offset:4096\n\tds_read_b64_tr_b16 %9, %17 offset:4096\n\t"
            "ds_read_b64_tr_b16 %10, %16 offset:20480\n\tds_read_b64_tr_b16 %11, %17 offset:20480\n\t"
            "ds_read_b64_tr_b16 %12, %16 offset:6144\n\tds_read_b64_tr_b16 %13, %17 offset:6144\n\t"
            "ds_read_b64_tr_b16 %14, %16 offset:22528\n\tds_read_b64_tr_b16 %15, %17 offset:22528\n\t"
            "s_waitcnt lgkmcnt(0)"
            : "=&v"(u[0]), "=&v"(u[1]), "=&v"(u[2]), "=&v"(u[3]), "=&v"(u[4]), "=&v"(u[5]), "=&v"(u[6]), "=&v"(u[7]), "=&v"(u[8]),
              "=&v"(u[9]), "=&v"(u[10]), "=&v"(u[11]), "=&v"(u[12]), "=&v"(u[13]), "=&v"(u[14]), "=&v"(u[15])
            : "v"(a0), "v"(a1)
            : "memory");
#pragma unroll
        for (int q = 0; q < 8; ++q)
            f[q >> 1][q & 1] = __builtin_bit_cast(bf16x8, __builtin_shufflevector(u[2 * q], u[2 * q + 1], 0, 1, 2, 3, 4, 5, 6, 7));
    };

    floatx4 acc[4][ST];
#pragma unroll
    for (int i = 0; i < 4; ++i)
#pragma unroll
        for (int j = 0; j < ST; ++j) acc[i][j] = floatx4{0.f, 0.f, 0.f, 0.f};
    float* out1 = a.sums1 + (int64_t(panel) * a.F1 + (wave & 1) * 16 + (lane & 15)) * a.S + s_tile0 * 16 + 4 * (lane >> 4);

#pragma unroll
    for (int q = 0; q < NS - 1; ++q) issue(q, q);
    int st = 0;
    for (int t = 0; t < n; ++t) {
        __builtin_amdgcn_s_waitcnt(0xC07F);              // lgkmcnt(0): this wave has read the tile before
        wait_vmcnt<(NS - 2) * L>();                      // its loads of this tile have landed (those of the next NS - 2 may not have)
        __builtin_amdgcn_s_barrier();
        __builtin_amdgcn_sched_barrier(0);
        issue(t + NS - 1, st == 0 ? NS - 1 : st - 1);
        const int at = st * STAGE;
        const unsigned char* s = dyn_smem + at;
        st = st == NS - 1 ? 0 : st + 1;
        // dH0: sums of 64 rows
        {
            bf16x8 h[4], l[4];
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                h[i] = read8(s + od + i * 1024);
                l[i] = read8(s + D_BYTES + od + i * 1024);
            }
#pragma unroll
            for (int j = 0; j < ST; ++j) {
                const bf16x8 ph = read8(s + op + (j >> 1) * 2048 + (j & 1) * 256);
#pragma unroll
                for (int i = 0; i < 4; ++i) acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(ph, h[i], acc[i][j], 0, 0, 0);
#pragma unroll
                for (int i = 0; i < 4; ++i) acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(ph, l[i], acc[i][j], 0, 0, 0);
                const bf16x8 pl = read8(s + op + Sh::P_BYTES + (j >> 1) * 2048 + (j & 1) * 256);
#pragma unroll
                for (int i = 0; i < 4; ++i) acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(pl, h[i], acc[i][j], 0, 0, 0);
            }
        }
        // dH1: 16 rows of it from 256 rows of D, in two chains of sums
        floatx4 acc1[2][SH];
#pragma unroll
        for (int c = 0; c < 2; ++c)
#pragma unroll
            for (int j = 0; j < SH; ++j) acc1[c][j] = floatx4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int k4 = 0; k4 < KS / 4; ++k4) {
            bf16x8 f[4][2];
            read_t4(at + k4 * 8192, f);
#pragma unroll
            for (int k = 0; k < 4; ++k)
#pragma unroll
                for (int j = 0; j < SH; ++j) {
                    acc1[0][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(p0[0][4 * k4 + k][j], f[k][0], acc1[0][j], 0, 0, 0);
                    acc1[1][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(p0[0][4 * k4 + k][j], f[k][1], acc1[1][j], 0, 0, 0);
                    acc1[1][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(p0[1][4 * k4 + k][j], f[k][0], acc1[1][j], 0, 0, 0);
                }
        }
        float* o = out1 + int64_t(tile0 + t) * kBondCols * a.S;
#pragma unroll
        for (int j = 0; j < SH; ++j) *reinterpret_cast<floatx4*>(o + j * 16) = acc1[0][j] + acc1[1][j];
        // keep the accumulators in the accumulation registers across the back edge
#pragma unroll
        for (int i = 0; i < 4; ++i)
#pragma unroll
            for (int j = 0; j < ST; ++j) asm volatile("" : "+a"(acc[i][j]));
    }
    wait_vmcnt<0>();                                     // no load into LDS outlives the workgroup
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        const int64_t r = row0 + wave * 64 + i * 16 + (lane & 15);
        if (r >= a.F0) continue;
        float* o = a.sums0 + (int64_t(range) * a.F0 + r) * a.S + 4 * (lane >> 4);
#pragma unroll
        for (int j = 0; j < ST; ++j) *reinterpret_cast<floatx4*>(o + j * 16) = acc[i][j];
    }
#endif
}

// grad[position of (c, k) in the caller's tensor] (+)= sum over splits of partial[split][c][k]. The position follows the
// step's packing recipe (PackArgs: digits of k and c times their strides); a tensor with a traced index pair (a
// ring of one core) receives the value at every diagonal position and keeps zeros elsewhere (the caller's buffer
// is cleared first by grad_fill_kernel).
// Y waves share 64 neighbouring elements, each takes every Y-th split (one wave walking 512 splits of a 96 x 160 tensor took
// 117 us, bound by the latency of its loads), and their sums are added in wave order: the order of the additions depends on
// n_split alone.
struct GradOutArgs {
    const float* partial;
    float* grad;
    int64_t ld, split_stride;               // partial: elements from c to c + 1, from split to split
    uint32_t c0, C, K;                      // rows c0 .. c0 + C - 1
    int32_t n_split, accumulate;
    int32_t nk, nc;
    uint32_t kext[tn::kMaxGatherDims], cext[tn::kMaxGatherDims];
    int64_t kstr[tn::kMaxGatherDims], cstr[tn::kMaxGatherDims];
    int64_t trace_extent, trace_stride;
};

// V: neighbouring elements of a row that a lane takes (K, ld and split_stride are multiples of it).
template <int Y, int V>
__device__ __forceinline__ void grad_reduce(const GradOutArgs& a) {
    typedef float floats __attribute__((ext_vector_type(V)));
    constexpr int GROUPS = Y >= 4 ? 1 : 4 / Y;                 // sets of 64 V elements a workgroup takes at a time
    __shared__ floats red[Y > 1 ? GROUPS * Y * 64 : 1];
    const uint32_t total = a.C * a.K;                          // below 2^31 (checked by the host)
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, y = wave % Y, group = wave / Y;
    for (uint32_t e0 = (blockIdx.x * GROUPS + group) * 64u * V; e0 - uint32_t(group) * 64u * V < total; e0 += gridDim.x * GROUPS * 64u * V) {
        const uint32_t e = e0 + lane * V;
        uint32_t c = e / a.K;
        const uint32_t k0 = e - c * a.K;
        c += a.c0;
        floats sum = {};
        if (e < total) {
            const float* p = a.partial + int64_t(c) * a.ld + k0;
#pragma unroll 8
            for (int s = y; s < a.n_split; s += Y) sum += *reinterpret_cast<const floats*>(p + int64_t(s) * a.split_stride);
        }
        if (Y > 1) {
            red[(group * Y + y) * 64 + lane] = sum;
            __syncthreads();
            if (y == 0) {
                sum = floats{};
#pragma unroll
                for (int j = 0; j < Y; ++j) sum += red[(group * Y + j) * 64 + lane];
            }
            __syncthreads();
        }
        if (y != 0 || e >= total) continue;
        int64_t c_off = 0;
        for (int j = a.nc - 1; j >= 0; --j) {
            const uint32_t q = c / a.cext[j];
            c_off += int64_t(c - q * a.cext[j]) * a.cstr[j];
            c = q;
        }
#pragma unroll
        for (int v = 0; v < V; ++v) {
            uint32_t k = k0 + v;
            int64_t off = c_off;
            for (int j = a.nk - 1; j >= 0; --j) {
                const uint32_t q = k / a.kext[j];
                off += int64_t(k - q * a.kext[j]) * a.kstr[j];
                k = q;
            }
            for (int64_t d = 0; d < a.trace_extent; ++d) {
                float* p = a.grad + off + d * a.trace_stride;
                *p = a.accumulate ? *p + sum[v] : sum[v];
            }
        }
    }
}

template <int Y>
__global__ void __launch_bounds__(Y > 4 ? 64 * Y : 256) grad_reduce_kernel(GradOutArgs a) {
    grad_reduce<Y, 1>(a);
}

// Several tensors in one launch, blockIdx.y says which; two elements a lane, as a launch of several has workgroups enough without
// one element to each.
constexpr int kGradOutMany = 4;
struct GradOutMany {
    GradOutArgs o[kGradOutMany];
};

template <int Y, int V>
__global__ void __launch_bounds__(256) grad_reduce_many_kernel(GradOutMany m) {
    if (Y == 4 && m.o[blockIdx.y].n_split < 4) grad_reduce<1, V>(m.o[blockIdx.y]);      // no splits to share out
    else grad_reduce<Y, V>(m.o[blockIdx.y]);
}

__global__ void __launch_bounds__(256) grad_fill_kernel(float* p, int64_t n) {
    for (int64_t e = int64_t(blockIdx.x) * 256 + threadIdx.x; e < n; e += int64_t(gridDim.x) * 256) p[e] = 0.f;
}
