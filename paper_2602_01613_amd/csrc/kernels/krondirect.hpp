// Kronecker-sum kernel for one token, slices made on chip: both halves' cores in, one token's output (or partial sums) out.
// Part of the tn_linear library's single translation unit: included by tn_linear.hip inside its
// anonymous namespace, after kernels/kronsum.hpp.
#pragma once

// ---------------------------------------------------------------------------------------------
// The same sum over the bond as kernels/kronsum.hpp,
//     Y[o1][o2] = sum_rho sum_a ( sum_k X[k][a] * B0_rho[o1][k] ) * B1_rho[o2][a],
// for calls of a few tokens. There the slices B0_rho, B1_rho are an array in memory (300 MB for a rank-96 ring 5120 -> 8192),
// and writing and reading it is what a one-token call takes its time with. Each slice is a small product of two cores,
// B_rho[(m, m')][(n, n')] = sum_s P[(m, n)][s] * Q[(m', n')][s], a few tens of KB; here it goes to LDS and no further:
//   * a workgroup takes a block of values of the bond, (values of one bond index) x (values of the other). The cores that carry
//     the first index are held ("resident": in registers, or in LDS where X takes the registers), the slabs of the others are
//     fetched from L2 per value, straight into MFMA operand registers, a value ahead;
//   * the four waves make the next value's two slices (16 x 16 tiles of the products, dealt out over a grid of waves) while they
//     use the current one's, in two LDS stages with one barrier per value;
//   * a tile's accumulator holds 4 consecutive rows (m, n) with n innermost: 4 consecutive k (or a) of one column of a slice, 8
//     bytes of an operand chunk. Where each goes is a table of one LDS position per tile and lane, made on the host;
//   * a wave owns O1W tiles of o1 (and, where o1 has fewer than four tiles, a share of o2). D = X^T B0_rho lands in the
//     accumulators, whose registers, rounded to bf16, are the operand of the second product (a numbered within 32 as
//     16 * (j / 4) + 4 * (lane / 16) + j % 4).
// What is rounded is what the kernel with stored slices rounds: slices and D to bf16, sums in fp32. Which half D is made with is the
// instantiation's choice here: for 5120 -> 1024 and 8192 -> 5120 it is the other one, and outputs of a few tokens are 3.1e-3 (2-norm) from those of
// that kernel, each 3.3e-3 from 64 bits; elsewhere a few 1e-5.
//
// What bounds it: what a wave issues. A value of the rank-96 ring 5120 -> 8192 is 76 MFMAs of a wave (1216 cycles, 42 of them the
// slices), 1280 cycles of the CU's LDS (a third of it the 8-byte stores, two to a bank) and 150 vector instructions, beside each other
// in 1.0 us (2100 cycles); as loops left to the compiler 1.9 us, in groups of MFMAs and groups of roundings 1.25.
// ---------------------------------------------------------------------------------------------
struct KronDirectArgs {
    const void* X;
    void* Y;                   // bf16 output, or fp32 partial sums [split][token][tile][lane][4] when n_splits > 1
    const void* src[2][2];     // per half: the resident and the streamed core, [value of its bond index][rows] x S, packed operands
    const uint16_t* unit[2];   // per half: LDS position / 8 of [row tile][column tile][lane]
    const int32_t *xrow, *xcol, *yrow, *ycol;      // offsets of a, k in a token of x, of o1, o2 in one of y
    int64_t N, M;
    int32_t tokens, A, K0, O1, C1;
    int32_t tiles[2][2];       // 16-row tiles of a slab: resident, streamed
    int32_t n_res, n_str;      // values of the two bond indices
    int32_t res_per, str_per;  // of them per workgroup
    int32_t str_blocks, n_splits;
    int32_t x_vec8;
};

template <int CFG, int SS>
struct KronDirectShape {
    static constexpr const int* C = tn::kDirectConfig[CFG];
    static constexpr int AT = C[0], KS = C[1], O1W = C[2], O2W = C[3], W1 = C[4], W2 = 4 / W1;
    static constexpr int WS0 = C[5], F0 = C[6], C0 = C[7], WS1 = C[8], F1 = C[9], C1 = C[10];
    static constexpr bool ROWS1_STR = C[11] != 0, RES_LDS = C[12] != 0;
    static constexpr int AS = (AT + 1) / 2;                          // steps of 32 values of a
    static constexpr int B0_BYTES = W1 * O1W * KS * 1024, B1_BYTES = W2 * O2W * AS * 1024, STAGE = B0_BYTES + B1_BYTES;
    static constexpr int RES_TILES = RES_LDS ? (4 / WS0) * C0 + (4 / WS1) * C1 : 0;
    static constexpr int CB0 = F0 == 1 ? 5 : 2, CB1 = F1 == 1 ? 5 : 2;      // resident tiles to a group of MFMAs
    static constexpr int GT = CB0 * F0 > CB1 * F1 ? CB0 * F0 : CB1 * F1;
    static constexpr int YB = O1W > 1 ? 4 : 8;                       // fragments of the second slice read at a time
    static constexpr size_t SMEM = size_t(2) * STAGE + size_t(RES_TILES) * SS * 1024;
};

// A lane's four sums of a tile to a token's output.
__device__ __forceinline__ void store_direct(const KronDirectArgs& p, bf16_t* y, int t1, int t2, int lane, const floatx4& v) {
    const int o1 = 16 * t1 + (lane & 15), o2 = 16 * t2 + 4 * (lane >> 4);
    if (o1 >= p.O1) return;
    const int yr = p.yrow[o1];
#pragma unroll
    for (int e = 0; e < 4; ++e)
        if (o2 + e < p.C1) y[yr + p.ycol[o2 + e]] = bf16_t(v[e]);
}

template <int CFG, int SS>
__global__ void __launch_bounds__(256, 1) step_krondirect_kernel(KronDirectArgs p) {
#ifdef __HIP_DEVICE_COMPILE__
    using S = KronDirectShape<CFG, SS>;
    constexpr int AT = S::AT, KS = S::KS, O1W = S::O1W, O2W = S::O2W, W1 = S::W1, W2 = S::W2, AS = S::AS;
    constexpr int F0 = S::F0, C0 = S::C0, F1 = S::F1, C1 = S::C1, STAGE = S::STAGE;
    constexpr bool RES_LDS = S::RES_LDS, ROWS1_STR = S::ROWS1_STR;
    extern __shared__ __attribute__((aligned(16))) unsigned char dyn_smem[];
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);

    // workgroup -> (token, block of the bond): the streamed blocks fastest, so that an XCD's workgroups fetch the same slabs
    const int t = blockIdx.x / p.n_splits, split = blockIdx.x - t * p.n_splits;
    const int res_block = split / p.str_blocks, str_block = split - res_block * p.str_blocks;
    const int r0 = res_block * p.res_per, r1 = min(p.n_res, r0 + p.res_per);
    const int s0 = str_block * p.str_per, n_s = min(p.n_str, s0 + p.str_per) - s0;
    const int n_it = (r1 - r0) * n_s;                                // >= 1 by construction of the grid

    // tiles of the cores this wave multiplies; past the end the last one again (the same values to the same place)
    const int ws0 = wave % S::WS0, wr0 = wave / S::WS0, ws1 = wave % S::WS1, wr1 = wave / S::WS1;
    auto tile_of = [](int first, int step, int i, int n) { return min(first + step * i, n - 1); };
    // a packed operand of 32 * SS columns: blocks of 32 rows x 16 k; lane l of a fragment takes row l % 16, k = 8 * (l / 16) ..
    const int frag_lane = (lane >> 5) * 512 + ((lane & 15) + 32 * ((lane >> 4) & 1)) * 8;
    auto frag = [&](const void* src, int tile, int s) -> bf16x8 {
        const bf16_t* q = static_cast<const bf16_t*>(src) + (int64_t(tile >> 1) * (2 * SS) + 2 * s) * 512 + (tile & 1) * 128 + frag_lane;
        return *reinterpret_cast<const bf16x8*>(q);
    };
    bf16x8 str0[F0][SS], str1[F1][SS];
    auto fetch_streamed = [&](auto half, int rs) {
        if constexpr (decltype(half)::value == 0) {
#pragma unroll
            for (int f = 0; f < F0; ++f)
#pragma unroll
                for (int s = 0; s < SS; ++s) str0[f][s] = frag(p.src[0][1], rs * p.tiles[0][1] + tile_of(ws0, S::WS0, f, p.tiles[0][1]), s);
        } else {
#pragma unroll
            for (int f = 0; f < F1; ++f)
#pragma unroll
                for (int s = 0; s < SS; ++s) str1[f][s] = frag(p.src[1][1], rs * p.tiles[1][1] + tile_of(ws1, S::WS1, f, p.tiles[1][1]), s);
        }
    };
    constexpr int HELD0 = RES_LDS ? 1 : C0, HELD1 = RES_LDS ? 1 : C1;
    bf16x8 res0[HELD0][SS], res1[HELD1][SS];
    unsigned char* res_lds = dyn_smem + 2 * STAGE;
    auto load_resident = [&](int rr) {
        if constexpr (RES_LDS) {
            const int n0 = p.tiles[0][0], n = n0 + p.tiles[1][0];
            for (int i = wave; i < n * SS; i += 4) {
                const int tile = i / SS, s = i - tile * SS;
                const bf16x8 v = tile < n0 ? frag(p.src[0][0], rr * n0 + tile, s) : frag(p.src[1][0], rr * p.tiles[1][0] + tile - n0, s);
                *reinterpret_cast<bf16x8*>(res_lds + i * 1024 + lane * 16) = v;
            }
        } else {
#pragma unroll
            for (int c = 0; c < C0; ++c)
#pragma unroll
                for (int s = 0; s < SS; ++s)
                    res0[c][s] = frag(p.src[0][0], rr * p.tiles[0][0] + tile_of(wr0, 4 / S::WS0, c, p.tiles[0][0]), s);
#pragma unroll
            for (int c = 0; c < C1; ++c)
#pragma unroll
                for (int s = 0; s < SS; ++s)
                    res1[c][s] = frag(p.src[1][0], rr * p.tiles[1][0] + tile_of(wr1, 4 / S::WS1, c, p.tiles[1][0]), s);
        }
    };
    fetch_streamed(std::integral_constant<int, 0>(), s0);
    fetch_streamed(std::integral_constant<int, 1>(), s0);
    load_resident(r0);

    // where this lane's 4 rows of every tile go in a stage
    int at0[F0][C0], at1[F1][C1];
#pragma unroll
    for (int f = 0; f < F0; ++f)
#pragma unroll
        for (int c = 0; c < C0; ++c) {
            const int ts = tile_of(ws0, S::WS0, f, p.tiles[0][1]), tr = tile_of(wr0, 4 / S::WS0, c, p.tiles[0][0]);
            at0[f][c] = int(p.unit[0][(ts * p.tiles[0][0] + tr) * 64 + lane]) * 8;
        }
#pragma unroll
    for (int f = 0; f < F1; ++f)
#pragma unroll
        for (int c = 0; c < C1; ++c) {
            const int ts = tile_of(ws1, S::WS1, f, p.tiles[1][1]), tr = tile_of(wr1, 4 / S::WS1, c, p.tiles[1][0]);
            at1[f][c] = S::B0_BYTES + int(p.unit[1][(ROWS1_STR ? ts * p.tiles[1][0] + tr : tr * p.tiles[1][1] + ts) * 64 + lane]) * 8;
        }

    // the token as row operands: tile i, step ks: lane l holds a = 16 * i + l % 16, k = 32 * ks + 8 * (l / 16) .. +7
    bf16x8 xa[AT][KS];
    {
        const bf16_t* xt = static_cast<const bf16_t*>(p.X) + int64_t(t) * p.N;
        int ro[AT];
#pragma unroll
        for (int i = 0; i < AT; ++i) ro[i] = p.xrow[min(16 * i + (lane & 15), p.A - 1)];
#pragma unroll
        for (int ks = 0; ks < KS; ++ks) {
            const int k = 32 * ks + 8 * (lane >> 4);
            if (p.x_vec8) {
                const int co = p.xcol[min(k, p.K0 - 8)];
#pragma unroll
                for (int i = 0; i < AT; ++i) xa[i][ks] = *reinterpret_cast<const bf16x8*>(xt + ro[i] + co);
            } else {
                int co[8];
#pragma unroll
                for (int e = 0; e < 8; ++e) co[e] = p.xcol[min(k, p.K0 - 8) + e];
#pragma unroll
                for (int i = 0; i < AT; ++i)
#pragma unroll
                    for (int e = 0; e < 8; ++e) xa[i][ks][e] = xt[ro[i] + co[e]];
            }
        }
        bf16x8 zero;
#pragma unroll
        for (int e = 0; e < 8; ++e) zero[e] = bf16_t(0.f);
#pragma unroll
        for (int i = 0; i < AT; ++i)
#pragma unroll
            for (int ks = 0; ks < KS; ++ks)
                if (16 * i + (lane & 15) >= p.A || 32 * ks + 8 * (lane >> 4) >= p.K0) xa[i][ks] = zero;
    }
    // what no tile writes (padding of o1, k, o2, a) is read all the same: zeros
    {
        floatx4 z = {0.f, 0.f, 0.f, 0.f};
        for (int i = tid; i < 2 * STAGE / 16; i += 256) *reinterpret_cast<floatx4*>(dyn_smem + i * 16) = z;
    }
    floatx4 acc[O1W][O2W];
#pragma unroll
    for (int o = 0; o < O1W; ++o)
#pragma unroll
        for (int j = 0; j < O2W; ++j)
#pragma unroll
            for (int v = 0; v < 4; ++v) acc[o][j][v] = 0.f;

    // One value's turn: D and Y of the value in `stage`, and between them the tiles of the next value into `next` (MAKE). One wave per
    // SIMD has nobody to hide behind, so the order is written out: phases of MFMAs that do not wait for each other, with the
    // rounding, the stores and the LDS reads of other phases dealt out between them one by one.
    constexpr int CB0 = S::CB0, CB1 = S::CB1, NG0 = (C0 + CB0 - 1) / CB0, NG = NG0 + (C1 + CB1 - 1) / CB1;
    constexpr int YF = O2W * AS, YB = S::YB, NY = (YF + YB - 1) / YB;
    auto phase = [](auto n_mfmas, auto&& mfma, auto n_items, auto&& item) {
        constexpr int M = decltype(n_mfmas)::value, I = decltype(n_items)::value;
        if constexpr (M == 0) {
            for_constants(item, std::make_integer_sequence<int, I>());
        } else {
            auto slot = [&](auto index) {
                constexpr int m = decltype(index)::value, i0 = (m * I + M - 1) / M, i1 = ((m + 1) * I + M - 1) / M;
                mfma(index);
                for_constants([&](auto q) { item(std::integral_constant<int, i0 + decltype(q)::value>()); },
                              std::make_integer_sequence<int, i1 - i0>());
                __builtin_amdgcn_sched_barrier(0);
            };
            for_constants(slot, std::make_integer_sequence<int, M>());
        }
    };
    // group q of tiles: half, first resident tile, how many, streamed tiles
#define TN_GROUP(q)                                                                                                          \
    constexpr int w = (q) >= NG0, first = w ? ((q) - NG0) * CB1 : (q) * CB0, F = w ? F1 : F0, C = w ? C1 : C0, CB = w ? CB1 : CB0, \
                  n = C - first < CB ? C - first : CB
    floatx4 g[S::GT];
    bf16x8 r[RES_LDS ? (CB0 > CB1 ? CB0 : CB1) : 1][SS];
    auto group_size = [](auto group) {
        constexpr int q = decltype(group)::value;
        if constexpr (q >= NG) return std::integral_constant<int, 0>();
        else {
            TN_GROUP(q);
            return std::integral_constant<int, n * F>();
        }
    };
    auto read_resident = [&](auto group) {                           // RES_LDS: a group's resident tiles
        if constexpr (RES_LDS && decltype(group)::value < NG) {
            TN_GROUP(decltype(group)::value);
#pragma unroll
            for (int c = 0; c < n; ++c)
#pragma unroll
                for (int s = 0; s < SS; ++s) {
                    const int tile = w ? p.tiles[0][0] + tile_of(wr1, 4 / S::WS1, first + c, p.tiles[1][0])
                                       : tile_of(wr0, 4 / S::WS0, first + c, p.tiles[0][0]);
                    r[c][s] = *reinterpret_cast<const bf16x8*>(res_lds + (tile * SS + s) * 1024 + lane * 16);
                }
        }
    };
    auto make_tile = [&](auto group, auto index) {                   // MFMA `index` of a group: its steps outermost
        constexpr int q = decltype(group)::value;
        if constexpr (q < NG) {
            TN_GROUP(q);
            constexpr int s = decltype(index)::value / (n * F), i = decltype(index)::value % (n * F), c = i / F, f = i % F;
            floatx4 z = {0.f, 0.f, 0.f, 0.f};
            if constexpr (s > 0) z = g[i];
            bf16x8 st, rs;
            if constexpr (w) st = str1[f][s];
            else st = str0[f][s];
            if constexpr (RES_LDS) rs = r[c][s];
            else if constexpr (w) rs = res1[first + c][s];
            else rs = res0[first + c][s];
            g[i] = w == 0 || ROWS1_STR ? __builtin_amdgcn_mfma_f32_16x16x32_bf16(st, rs, z, 0, 0, 0)
                                       : __builtin_amdgcn_mfma_f32_16x16x32_bf16(rs, st, z, 0, 0, 0);
        }
    };
    auto put_tile = [&](auto group, auto index, unsigned char* next) {
        constexpr int q = decltype(group)::value, i = decltype(index)::value;
        if constexpr (q < NG) {
            TN_GROUP(q);
            typedef __bf16 bf16x4_t __attribute__((ext_vector_type(4)));
            bf16x4_t h;
#pragma unroll
            for (int v = 0; v < 4; ++v) h[v] = bf16_t(g[i][v]);
            int at;
            if constexpr (w) at = at1[i % F][first + i / F];
            else at = at0[i % F][first + i / F];
            *reinterpret_cast<bf16x4_t*>(next + at) = h;
        }
    };
#undef TN_GROUP
    const int w1 = wave % W1, w2 = wave / W1;
    const int lane16 = lane * 16;
    auto turn = [&](auto make_next, const unsigned char* stage, unsigned char* next, int fetch) {
        constexpr bool MAKE = decltype(make_next)::value;
        bf16x8 b0[O1W][KS], y[2][YB], zb[O1W][AS];
        floatx4 d[O1W][2 * AS];
        const std::integral_constant<int, 0> none;
        auto size_of = [&](auto group) {                             // tiles of a group, where any are made
            if constexpr (MAKE) return group_size(group);
            else return std::integral_constant<int, 0>();
        };
        auto steps_of = [&](auto group) { return std::integral_constant<int, decltype(size_of(group))::value * SS>(); };
        auto read_y = [&](auto batch, auto index) {
            constexpr int e = decltype(batch)::value * YB + decltype(index)::value, s = e / O2W, j = e % O2W;
            if constexpr (e < YF)
                y[decltype(batch)::value & 1][decltype(index)::value] =
                    *reinterpret_cast<const bf16x8*>(stage + S::B0_BYTES + ((w2 + W2 * j) * AS + s) * 1024 + lane16);
        };
        const std::integral_constant<int, 0> q0;
#pragma unroll
        for (int o = 0; o < O1W; ++o)
#pragma unroll
            for (int ks = 0; ks < KS; ++ks) b0[o][ks] = *reinterpret_cast<const bf16x8*>(stage + ((w1 + W1 * o) * KS + ks) * 1024 + lane16);
        if constexpr (MAKE) read_resident(q0);
        __builtin_amdgcn_sched_barrier(0);
        // tiles of group 0, meanwhile the first fragments of B1
        phase(steps_of(q0), [&](auto m) { make_tile(q0, m); }, std::integral_constant<int, YB>(), [&](auto i) { read_y(q0, i); });
        if constexpr (MAKE) read_resident(std::integral_constant<int, 1>());
        // D, meanwhile group 0 goes to LDS
        phase(std::integral_constant<int, O1W * AT * KS>(), [&](auto index) {
            constexpr int m = decltype(index)::value, ks = m / (O1W * AT), o = m / AT % O1W, i = m % AT;
            floatx4 z = {0.f, 0.f, 0.f, 0.f};
            if constexpr (ks > 0) z = d[o][i];
            d[o][i] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(xa[i][ks], b0[o][ks], z, 0, 0, 0);
        }, size_of(q0), [&](auto i) { put_tile(q0, i, next); });
        auto round_d = [&](auto index) {
            constexpr int o = decltype(index)::value / AS, s = decltype(index)::value % AS;
#pragma unroll
            for (int e = 0; e < 8; ++e) {
                const int i = 2 * s + (e >> 2);
                zb[o][s][e] = i < AT ? bf16_t(d[o][i < AT ? i : 0][e & 3]) : bf16_t(0.f);
            }
        };
        auto step = [&](auto index) {
            constexpr int q = decltype(index)::value;
            const std::integral_constant<int, q> now;
            const std::integral_constant<int, q + 1> then;
            if constexpr (MAKE && q + 1 == NG0) fetch_streamed(none, fetch);             // the first half's slabs are used up
            // tiles of the next group, meanwhile D is rounded
            phase(steps_of(then), [&](auto m) { make_tile(then, m); }, std::integral_constant<int, q == 0 ? O1W * AS : 0>(), round_d);
            if constexpr (MAKE) read_resident(std::integral_constant<int, q + 2>());
            // Y, meanwhile that group goes to LDS and the next fragments of B1 are read
            constexpr int n_put = decltype(size_of(then))::value, n_read = q + 1 < NY ? YB : 0, left = q < NY ? (YF - q * YB < YB ? YF - q * YB : YB) : 0;
            phase(std::integral_constant<int, left * O1W>(), [&](auto m) {
                constexpr int i = decltype(m)::value / O1W, o = decltype(m)::value % O1W, s = (q * YB + i) / O2W, j = (q * YB + i) % O2W;
                acc[o][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(y[q & 1][i], zb[o][s], acc[o][j], 0, 0, 0);
            }, std::integral_constant<int, n_put + n_read>(), [&](auto i) {
                if constexpr (decltype(i)::value < n_read) read_y(then, i);
                else put_tile(then, std::integral_constant<int, decltype(i)::value - n_read>(), next);
            });
        };
        for_constants(step, std::make_integer_sequence<int, (NY > NG - 1 ? NY : NG - 1)>());
        if constexpr (MAKE) fetch_streamed(std::integral_constant<int, 1>(), fetch);
    };

    __syncthreads();                                                 // the zeros (and the resident cores) are in LDS
    for_constants([&](auto q) {
        constexpr int n = decltype(group_size(q))::value;
        read_resident(q);
        for_constants([&](auto m) { make_tile(q, m); }, std::make_integer_sequence<int, n * SS>());
        for_constants([&](auto i) { put_tile(q, i, dyn_smem); }, std::make_integer_sequence<int, n>());
    }, std::make_integer_sequence<int, NG>());
    int rs = 1, rr = r0;                                             // of the value after the one made last
    if (rs == n_s) rs = 0, ++rr;
    fetch_streamed(std::integral_constant<int, 0>(), s0 + rs);
    fetch_streamed(std::integral_constant<int, 1>(), s0 + rs);
    __syncthreads();
    for (int it = 0; it + 1 < n_it; ++it) {
        if (rs == 0) {                                               // the next value of the resident index
            load_resident(rr);
            if constexpr (RES_LDS) __syncthreads();                  // (every wave has made its tiles of the last value before the barrier above)
        }
        if (++rs == n_s) rs = 0, ++rr;
        turn(std::true_type(), dyn_smem + (it & 1) * STAGE, dyn_smem + ((it + 1) & 1) * STAGE, s0 + rs);
        __syncthreads();
    }
    turn(std::false_type(), dyn_smem + ((n_it - 1) & 1) * STAGE, nullptr, 0);

    // lane l, register v of acc[o][j]: o1 = 16 * tile + l % 16, o2 = 16 * tile + 4 * (l / 16) + v. Partial sums are kept as they lie in
    // the registers, a tile's 1 KB in one piece; krondirect_reduce_kernel knows the order.
    const int o1_tiles = (p.O1 + 15) / 16, o2_tiles = (p.C1 + 15) / 16;
    float* yf = static_cast<float*>(p.Y) + (int64_t(split) * p.tokens + t) * (o1_tiles * o2_tiles * 256);
    bf16_t* yb = static_cast<bf16_t*>(p.Y) + int64_t(t) * p.M;
#pragma unroll
    for (int o = 0; o < O1W; ++o) {
        const int t1 = w1 + W1 * o;
        if (t1 >= o1_tiles) continue;
#pragma unroll
        for (int j = 0; j < O2W; ++j) {
            const int t2 = w2 + W2 * j;
            if (t2 >= o2_tiles) continue;
            if (p.n_splits > 1) *reinterpret_cast<floatx4*>(yf + (t1 * o2_tiles + t2) * 256 + lane * 4) = acc[o][j];
            else store_direct(p, yb, t1, t2, lane, acc[o][j]);
        }
    }
#endif
}

// The partial sums of the kernel above, added in the order of the splits: a workgroup takes 16 pieces of 4 values of a token, its 16 rows of
// threads a sixteenth of the splits each.
__global__ void __launch_bounds__(256) krondirect_reduce_kernel(KronDirectArgs p, const float* partial) {
    __shared__ floatx4 part[16][16];
    const int g = threadIdx.x & 15, q = threadIdx.x >> 4;
    const int o2_tiles = (p.C1 + 15) / 16, per_token = (p.O1 + 15) / 16 * o2_tiles * 64;       // pieces: a multiple of 64
    const int64_t n = int64_t(p.tokens) * per_token * 4;
    const int64_t piece = int64_t(blockIdx.x) * 16 + g;
    floatx4 s = {0.f, 0.f, 0.f, 0.f};
#pragma unroll 8
    for (int k = q; k < p.n_splits; k += 16) s += *reinterpret_cast<const floatx4*>(partial + int64_t(k) * n + piece * 4);
    part[q][g] = s;
    __syncthreads();
    if (q == 0) {
        floatx4 v = part[0][g];
#pragma unroll
        for (int k = 1; k < 16; ++k) v += part[k][g];
        const int64_t t = piece / per_token;
        const int in = int(piece - t * per_token), tile = in >> 6, t1 = tile / o2_tiles;
        store_direct(p, static_cast<bf16_t*>(p.Y) + t * p.M, t1, tile - t1 * o2_tiles, in & 63, v);
    }
}
