// Matrix-product step kernel: wide bf16 steps whose input is a plain row-major matrix, more than a row tile of it.
// Part of the tn_linear library's single translation unit: included by tn_linear.hip inside its
// anonymous namespace, after kernels/tiled.hpp.
#pragma once

// ---------------------------------------------------------------------------------------------
// Out[r][c] = sum_k A[r][k] * B[c][k], A row-major with K % 64 == 0, B packed fragment-major, output through the
// step's scatter tables in aligned pieces of 8 columns (TRANS = 0) or of 8 rows (TRANS = 1).
//
// What bounds it: on large shapes the power the chip may draw. With every wait hidden the clock settles at what the
// energy of a K tile allows, so what counts is energy per product (measured at 8192 x 8192 x 5120):
//   * v_mfma_f32_16x16x32_bf16 instead of 32x32x16: half the accumulator traffic per product. The same loop ran at
//     1.99 GHz instead of 1.72 (1.52 instead of 1.42 PFLOP/s without its stores);
//   * four waves, each a quarter (up to 128 x 128) of the tile, instead of eight: 64 instead of 96 KB of fragments read
//     from LDS per 32 k. One wave per SIMD then has to keep its matrix core busy alone, so the order of the loop is
//     written out: one LDS read or one direct-to-LDS load at a time between two MFMAs (bunched, 1.33 PFLOP/s; one by
//     one, 1.58, without stores);
//   * both operands go from memory to LDS without passing through registers. A row of a stage is 128 bytes (64 k),
//     and its 16-byte chunk c sits at position c ^ ((row / 2) % 8), so that the 16 rows a read touches at a time
//     fall on 16 different slots of the 64 banks (with c ^ (row % 8) 40 % of the LDS cycles were conflicts); B's
//     packed blocks lie in fragment order already and are copied as they are.
// NS stages of 64 k. Once the fragments of a tile's second half are in registers its stage is free: one barrier per tile (two
// stages: and one where the next is read) lets the loads of the tile NS further on into it. The largest tiles leave LDS for two
// stages; a third, and the loads dealt out evenly over the whole of a tile instead of over its second half, is worth 17 to 21 %
// to the smaller ones, which move more bytes per product and do not cover the memory's latency with one tile (us with two
// stages and bunched loads / as it is: 1024 x 8192 x 5120 on 128 x 256 tiles 98 / 77, 777 x 25600 x 5120 on 160 x 256 206 / 170,
// 2500 x 8192 x 5120 195 / 159). Tiles of which a CU holds two workgroups keep to half of its LDS. Loads past the last tile are
// out of bounds and read no memory.
// The sums leave straight from registers: two lane swaps turn the accumulator layout (4 consecutive values per lane)
// into 16-byte pieces of 64-byte runs, with no second trip through LDS; the output offsets of the tile's rows and
// columns are fetched into LDS when the tile starts.
// 8192 x 8192 x 5120 in 466 us = 1.47 PFLOP/s (the 256 x 256 ping-pong kernel this replaces: 565 us), 8192 x 9216 x
// 2304 in 270 us (340).
//
// Tile sizes: 32*TM x 32*TN, TM <= 8, TN 8, 4 or 2; the host picks the one (and the number of K ranges) with the least
// time by gemm_choice. XCD x takes a contiguous eighth of the tiles in bands of four row tiles (row fastest), so that
// the 32 tiles an XCD runs at a time share 4 + 8 operand panels in its L2 and no XCD has a row tile more than another
// (dealing whole row tiles to XCDs left 2500 rows at 10 tiles over 8 XCDs: 281 us, now 160).
// ---------------------------------------------------------------------------------------------
struct GemmArgs {
    int32_t n_row, n_col;          // output tiles
    int32_t n_split;               // ranges of K
    int32_t ktiles_per_split;      // K tiles of 64 per range, at least one in every range
    int32_t scalar_out;            // GEMM_ANY, TRANS = 1: outputs in no aligned pieces
    float* partial;                // not null: fp32 sums [split][rows_pad][ld] instead of the output (TRANS = 0, C % 4 == 0)
    int64_t rows_pad, ld;
    // GEMM_PARTS, in elements, 0: there is none
    int64_t a_lo, b_lo;            // from an operand to its low part
    int64_t out_lo;                // from the output to where its low part goes
};

template <int TM, int TN, int NS>
struct GemmShape {
    static constexpr int BM = 32 * TM, BN = 32 * TN;
    static constexpr int STAGE_BYTES = (BM + BN) * 128;
    static constexpr int TAB_ROWS = (BM + 63) / 64 * 64;                 // crow of the tile's rows, ccol of its columns: 64 entries per load
    static constexpr size_t SMEM = size_t(NS) * STAGE_BYTES + size_t(TAB_ROWS + BN) * 4;
};

// Forms of the kernel, instantiations of their own so that the loop above stays as it was measured (with the second and third as
// branches in it, launches of 10 us took 0.2 to 0.5 longer: the arguments are fetched later).
//   GEMM_PARTS  a matrix of fp32 significance as a sum of two of bf16, high = bf16(v) and low = bf16(v - high), which leaves 2^-17
//               of v. With low parts the K tiles are walked two or three times, (A, B), (A low, B), (A, B low), into the same
//               sums, which is the fp32 product but for terms of 2^-16: sums over tokens have to pass through here without
//               losing what averaging over the tokens gained.
//   GEMM_SHORT  K of one or two tiles, NS of them: bound by the stores and by how many workgroups have theirs under way, so as
//               little as possible is held by one. Every K tile has its stage and all are loaded at once, one set of
//               fragments: 36 KB of LDS (one tile) and 118 registers at 160 x 128, three or four workgroups on a CU instead of two.
//   GEMM_ANY    K % 8 == 0: B holds zeros from K to whole tiles, and chunks of A past it read as zeros; and outputs in neither
//               kind of piece (TRANS = 1, scalar_out): one value at a time, 16 neighbouring columns per store.
enum GemmForm : int { GEMM_PLAIN = 1, GEMM_PARTS = 2, GEMM_ANY = 3, GEMM_SHORT = 4 };

template <typename F, int... Q>
__device__ __forceinline__ void for_constants(F&& f, std::integer_sequence<int, Q...>) {
    (f(std::integral_constant<int, Q>()), ...);
}

#ifdef __HIP_DEVICE_COMPILE__
template <int TM, int TN, int NS, int TRANS, int FORM>
__device__ __forceinline__ void gemm_tile(const StepArgs& a, const GemmArgs& g) {
    using S = GemmShape<TM, TN, NS>;
    constexpr int NW = 4, BM = S::BM, BN = S::BN, STAGE = S::STAGE_BYTES, A_BYTES = BM * 128;
    constexpr int L = TM + TN;                           // 1 KB direct-to-LDS loads per wave and stage: TM of A, then TN of B
    static_assert(TN % 2 == 0 && (!TRANS || TM % 2 == 0), "stores pair neighbouring tiles");
    typedef __attribute__((address_space(3))) void lds_t;
    typedef unsigned int uintx4 __attribute__((ext_vector_type(4)));
    extern __shared__ __attribute__((aligned(16))) unsigned char dyn_smem[];
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int wm = wave >> 1, wn = wave & 1;

    // workgroup -> (tile, range of K): see above
    int row_tile, col_tile, split;
    {
        constexpr int BAND = 4;
        const int n_items = g.n_row * g.n_col * g.n_split, xcd = blockIdx.x & 7;
        const int item = int(int64_t(n_items) * xcd >> 3) + int(blockIdx.x >> 3);
        if (item >= int(int64_t(n_items) * (xcd + 1) >> 3)) return;
        const int tile = item / g.n_split;
        split = item - tile * g.n_split;
        const int band = tile / (BAND * g.n_col), in_band = tile - band * (BAND * g.n_col);
        const int band_rows = min(BAND, g.n_row - band * BAND);
        col_tile = in_band / band_rows;
        row_tile = band * BAND + in_band - col_tile * band_rows;
    }
    const uint32_t row0 = uint32_t(row_tile) * BM;
    const int col0 = col_tile * BN, nks = a.Kp >> 4;
    const int kt0 = split * g.ktiles_per_split;
    const int nk_seg = a.Kp >> 6, n_seg = FORM != GEMM_PARTS ? 1 : 1 + (g.a_lo != 0) + (g.b_lo != 0);
    const int nk = min(nk_seg * n_seg, kt0 + g.ktiles_per_split) - kt0;  // >= 1

    // rows past the end read as zeros (bounds of the buffer)
    const int row_bytes = a.K * 2;
    const bf16_t* pa = static_cast<const bf16_t*>(a.A) + int64_t(row0) * a.K;
    const bf16_t* pb = static_cast<const bf16_t*>(a.B) + int64_t(col0 >> 5) * nks * 512;
    const int a_size = int(min(int64_t(a.total_rows) - int64_t(row0), int64_t(BM))) * row_bytes, b_size = (BN / 32) * nks * 1024;
    const __amdgpu_buffer_rsrc_t ra = __builtin_amdgcn_make_buffer_rsrc(const_cast<bf16_t*>(pa), 0, a_size, 0x00020000);
    const __amdgpu_buffer_rsrc_t rb = __builtin_amdgcn_make_buffer_rsrc(const_cast<bf16_t*>(pb), 0, b_size, 0x00020000);
    // a load of A covers 8 rows x 128 bytes: lane l fills position l%8 of row l/8
    const int chunk = (lane & 7) ^ ((wave * 4 + (lane >> 4)) & 7);
    int va = (wave * 8 + (lane >> 3)) * row_bytes + chunk * 16;
    // in a last tile that K does not fill, chunks past it read as zeros too: what follows them is the next row
    const int va_last = (FORM == GEMM_ANY && (a.K & 63) && kt0 + nk == nk_seg * n_seg && chunk * 8 >= (a.K & 63)) ? int(0x80000000u) : va;
    const int vb = wave * 1024 + lane * 16;              // the four waves bring the four k-step blocks of a column block
    // tiles past the range: out of bounds, no memory is read
    auto past = [&](int kt) -> int { return kt < nk ? 0 : int(0x80000000u); };
    auto load1 = [&](int j, int kt, int off, unsigned char* s) {
        if (FORM == GEMM_PARTS) {
            const int t = kt0 + kt, seg = (t >= nk_seg) + (t >= 2 * nk_seg), tk = t - seg * nk_seg;
            const bool a_low = seg == 1 && g.a_lo, b_low = seg && !a_low;
            if (j < TM)
                __builtin_amdgcn_raw_ptr_buffer_load_lds(
                    __builtin_amdgcn_make_buffer_rsrc(const_cast<bf16_t*>(pa + (a_low ? g.a_lo : 0)), 0, a_size, 0x00020000),
                    (lds_t*)(s + (j * NW + wave) * 1024), 16, va | off, tk * 128 + j * (NW * 8) * row_bytes, 0, 0);
            else
                __builtin_amdgcn_raw_ptr_buffer_load_lds(
                    __builtin_amdgcn_make_buffer_rsrc(const_cast<bf16_t*>(pb + (b_low ? g.b_lo : 0)), 0, b_size, 0x00020000),
                    (lds_t*)(s + A_BYTES + ((j - TM) * NW + wave) * 1024), 16, vb | off, tk * 4096 + (j - TM) * nks * 1024, 0, 0);
        } else if (j < TM)
            __builtin_amdgcn_raw_ptr_buffer_load_lds(ra, (lds_t*)(s + (j * NW + wave) * 1024), 16, va | off,
                                                     (kt0 + kt) * 128 + j * (NW * 8) * row_bytes, 0, 0);
        else
            __builtin_amdgcn_raw_ptr_buffer_load_lds(rb, (lds_t*)(s + A_BYTES + ((j - TM) * NW + wave) * 1024), 16, vb | off,
                                                     (kt0 + kt) * 4096 + (j - TM) * nks * 1024, 0, 0);
    };
    // output offsets of the tile's rows and columns; entries past the end repeat a valid one and are not used
    unsigned char* tab = dyn_smem + NS * STAGE;
    if (!g.partial) {
        const __amdgpu_buffer_rsrc_t rr = __builtin_amdgcn_make_buffer_rsrc(const_cast<int32_t*>(a.crow), 0, int(a.R) * 4, 0x00020000);
        const __amdgpu_buffer_rsrc_t rc = __builtin_amdgcn_make_buffer_rsrc(const_cast<int32_t*>(a.ccol), 0, a.C * 4, 0x00020000);
        if (wave * 64 < S::TAB_ROWS) {
            const uint32_t r = row0 + wave * 64 + lane;
            __builtin_amdgcn_raw_ptr_buffer_load_lds(rr, (lds_t*)(tab + wave * 256), 4, int((a.R == 1 ? 0u : r % a.R) * 4), 0, 0, 0);
        }
        if (wave * 64 < BN)
            __builtin_amdgcn_raw_ptr_buffer_load_lds(rc, (lds_t*)(tab + S::TAB_ROWS * 4 + wave * 256), 4,
                                                     min(col0 + wave * 64 + lane, a.C - 1) * 4, 0, 0, 0);
    }
    // One K tile is 2 * TM * TN MFMAs. The reads of the second half's fragments are dealt out over the first RS * NR of them and
    // are followed by the barrier (BAR); the loads of the tile NS further on into the stage that is free from there on are
    // dealt out over what is left of the tile, or, with a stage to spare, over a whole tile's length: the last of them
    // go with the first MFMAs of the next tile. A load keeps the vector-memory path of the CU for 16 cycles, an MFMA its
    // SIMD's matrix core: all of them in the second half of a tile (4 x 8: 48 loads, 768 cycles, beside 512 of MFMAs) stall it.
    constexpr int NM = TM * TN, NR = TM + TN;
    constexpr int RS = NM * 3 / 4 / NR > 1 ? NM * 3 / 4 / NR : 1, BAR = RS * NR + 4 < NM ? RS * NR + 4 : NM;
    constexpr int SPAN = NS > 2 ? 2 * NM : 2 * NM - BAR;
    constexpr int L_NOW = NS > 2 ? ((2 * NM - BAR) * L + SPAN - 1) / SPAN : L;      // loads l with BAR + l * SPAN / L < 2 * NM
    // With two stages the next tile's loads get until its first fragment is read (a barrier of its own, after the EARLY first loads of
    // the tile after it), or the last of them would have 37 MFMAs' time on 6 x 8 tiles. (Two products of 1321 x 25600 x 5120, 6 x 8 tiles:
    // 631 us with one wait, 576 so; rank-32 ring 25600 -> 5120 at 8192 tokens, 7 x 8: 1901 / 1797; 8192 x 9216 x 2304, 8 x 8: 1.5 % of it.)
    constexpr bool LATE = NS == 2 && BAR < NM;
    constexpr int EARLY = ((NM - BAR) * L + SPAN - 1) / SPAN;      // loads l with BAR + l * SPAN / L < NM
    static_assert(FORM == GEMM_SHORT || !LATE || (BAR + (EARLY - 1) * SPAN / L < NM && BAR + EARLY * SPAN / L >= NM), "early loads");
    static_assert(FORM == GEMM_SHORT || (L_NOW <= L && BAR + (L_NOW - 1) * SPAN / L < 2 * NM && (L_NOW == L || BAR + L_NOW * SPAN / L >= 2 * NM)), "load slots");
    if constexpr (FORM == GEMM_SHORT) {
#pragma unroll
        for (int q = 0; q < NS; ++q)
#pragma unroll
            for (int l = 0; l < L; ++l) load1(l, q, 0, dyn_smem + q * STAGE);
    } else {
#pragma unroll
        for (int q = 0; q < NS; ++q) {
            if (FORM == GEMM_ANY && nk == q + 1) va = va_last;
#pragma unroll
            for (int l = 0; l < (q == NS - 1 ? L_NOW : L); ++l) load1(l, q, past(q), dyn_smem + q * STAGE);
        }
    }

    // fragments: lane l supplies row (A) or column (B) l%16 and k = 32*ks + 8*(l/16) .. +7
    int oa[2], ob[2];
#pragma unroll
    for (int ks = 0; ks < 2; ++ks) {
        const int r = lane & 15, c = 4 * ks + (lane >> 4);
        oa[ks] = (wm * TM * 16 + r) * 128 + ((c ^ ((r >> 1) & 7)) * 16);
        ob[ks] = A_BYTES + (wn * TN / 2) * 4096 + (2 * ks + (lane >> 5)) * 1024 + ((lane & 15) + 32 * ((lane >> 4) & 1)) * 16;
    }
    floatx4 acc[TM][TN];
    bf16x8 fa[2][TM], fb[2][TN];
    auto read1 = [&](int q, int set, const unsigned char* s, int ks) {       // the columns first: every row of MFMAs needs them all
        if (q < TN) fb[set][q] = *reinterpret_cast<const bf16x8*>(s + ob[ks] + (q >> 1) * 4096 + (q & 1) * 256);
        else fa[set][q - TN] = *reinterpret_cast<const bf16x8*>(s + oa[ks] + (q - TN) * 2048);
    };
#pragma unroll
    for (int i = 0; i < TM; ++i)
#pragma unroll
        for (int j = 0; j < TN; ++j) {
#pragma unroll
            for (int v = 0; v < 4; ++v) acc[i][j][v] = 0.f;
            asm volatile("" : "+a"(acc[i][j]));
        }
    if constexpr (FORM == GEMM_SHORT) {
#pragma unroll
        for (int kt = 0; kt < NS; ++kt) {
            if (kt + 1 < NS) wait_vmcnt<(NS - 1) * L>();
            else wait_vmcnt<0>();
            __builtin_amdgcn_s_barrier();
#pragma unroll
            for (int ks = 0; ks < 2; ++ks) {
#pragma unroll
                for (int q = 0; q < NR; ++q) read1(q, 0, dyn_smem + kt * STAGE, ks);
#pragma unroll
                for (int i = 0; i < TM; ++i)
#pragma unroll
                    for (int j = 0; j < TN; ++j)
                        acc[i][j] = TRANS ? __builtin_amdgcn_mfma_f32_16x16x32_bf16(fa[0][i], fb[0][j], acc[i][j], 0, 0, 0)
                                          : __builtin_amdgcn_mfma_f32_16x16x32_bf16(fb[0][j], fa[0][i], acc[i][j], 0, 0, 0);
            }
        }
    } else {
        wait_vmcnt<(NS - 2) * L + L_NOW>();                  // the tables and the first K tile have landed
        __builtin_amdgcn_s_barrier();
#pragma unroll
        for (int q = 0; q < NR; ++q) read1(q, 0, dyn_smem, 0);
        int at = 0, at_prev = (NS - 1) * STAGE;              // byte offsets of this tile's stage and of the one before
        for (int kt = 0; kt < nk; ++kt) {
            unsigned char *s = dyn_smem + at, *sp = dyn_smem + at_prev;
            at_prev = at;
            at = at == (NS - 1) * STAGE ? 0 : at + STAGE;
            const unsigned char* sn = dyn_smem + at;
            const int off_prev = past(kt + NS - 1), off = past(kt + NS);
            __builtin_amdgcn_sched_barrier(0);
            // (slots as compile-time constants: as a loop, 128 of them are not unrolled in time to keep the fragments in registers)
            auto slot = [&](auto slot_index) {
                constexpr int q = decltype(slot_index)::value, half = q / NM, m = q % NM, i = m / TN, j = m % TN;
                if constexpr (q == BAR) {
                    __builtin_amdgcn_s_waitcnt(0xC07F);      // lgkmcnt(0): this wave has read the whole stage
                    if constexpr (!LATE) wait_vmcnt<(NS - 2) * L>();      // its loads of the next stage have landed
                    __builtin_amdgcn_s_barrier();
                    if (FORM == GEMM_ANY && kt + NS + 1 == nk) va = va_last;
                    __builtin_amdgcn_sched_barrier(0);
                }
                if constexpr (LATE && q == NM) {
                    wait_vmcnt<EARLY>();                     // the next stage is read from here on
                    __builtin_amdgcn_s_barrier();
                    __builtin_amdgcn_sched_barrier(0);
                }
                acc[i][j] = TRANS ? __builtin_amdgcn_mfma_f32_16x16x32_bf16(fa[half][i], fb[half][j], acc[i][j], 0, 0, 0)
                                  : __builtin_amdgcn_mfma_f32_16x16x32_bf16(fb[half][j], fa[half][i], acc[i][j], 0, 0, 0);
                __builtin_amdgcn_sched_barrier(0);
                if constexpr (m % RS == 0 && m / RS < NR) read1(m / RS, half ^ 1, half ? sn : s, half ^ 1);
                if constexpr (NR > NM && m == NM - 1) {
#pragma unroll
                    for (int r = NM; r < NR; ++r) read1(r, half ^ 1, half ? sn : s, half ^ 1);
                }
#pragma unroll
                for (int l = 0; l < L_NOW; ++l)
                    if (BAR + l * SPAN / L == q) load1(l, kt + NS, off, s);
#pragma unroll
                for (int l = L_NOW; l < L; ++l)
                    if (BAR + l * SPAN / L == q + 2 * NM) load1(l, kt + NS - 1, off_prev, sp);
                __builtin_amdgcn_sched_barrier(0);
            };
            for_constants(slot, std::make_integer_sequence<int, 2 * NM>());
            // keep the accumulators in the accumulation registers across the back edge
#pragma unroll
            for (int i = 0; i < TM; ++i)
#pragma unroll
                for (int j = 0; j < TN; ++j) asm volatile("" : "+a"(acc[i][j]));
        }
    }
    wait_vmcnt<0>();                                     // no load into LDS outlives the workgroup

    if (g.partial) {
        // lane: row l%16 of tile i, columns 4*(l/16) .. +3 of tile j
        const int c = col0 + wn * TN * 16 + 4 * (lane >> 4);
#pragma unroll
        for (int i = 0; i < TM; ++i) {
            const uint32_t r = row0 + wm * TM * 16 + i * 16 + (lane & 15);
            float* p = g.partial + (int64_t(split) * g.rows_pad + r) * g.ld + c;
            if (r < a.total_rows) {
#pragma unroll
                for (int j = 0; j < TN; ++j)
                    if (c + j * 16 < a.C) *reinterpret_cast<floatx4*>(p + j * 16) = acc[i][j];
            }
        }
        return;
    }
    // Offsets in bytes from the tile's first token (checked by the host to fit 31 bits); ~0 is out of bounds: not stored.
    const uint32_t t_first = a.R == 1 ? row0 : row0 / a.R;
    const __amdgpu_buffer_rsrc_t ro = __builtin_amdgcn_make_buffer_rsrc(
        static_cast<bf16_t*>(a.Out) + int64_t(t_first) * a.c_tok_stride, 0, 0x7fffffff, 0x00020000);
    constexpr uint32_t OUT = 0x80000000u;
    const int32_t* tr = reinterpret_cast<const int32_t*>(tab);
    const int32_t* tc = tr + S::TAB_ROWS;
    const uint32_t ctok = uint32_t(a.c_tok_stride);
    auto row_offset = [&](uint32_t lr) -> uint32_t {
        const uint32_t r = row0 + lr, t = a.R == 1 ? r : r / a.R;
        return r < a.total_rows ? ((t - t_first) * ctok + uint32_t(tr[lr])) * 2u : OUT;
    };
    auto col_offset = [&](int lc) -> uint32_t { return col0 + lc < a.C ? uint32_t(tc[lc]) * 2u : OUT; };
    // x, y: two neighbouring 16 x 16 tiles along the direction in which a lane holds 4 consecutive values. Afterwards it
    // holds 8: of x in lanes 0-31, of y in lanes 32-63, values 8*((l/16)%2) ..
    auto merge = [&](const floatx4& x, const floatx4& y) -> uintx4 {
        typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
        auto pack = [](float u, float v) {
            bf16x2 h;
            h[0] = bf16_t(u);
            h[1] = bf16_t(v);
            return __builtin_bit_cast(unsigned, h);
        };
        const auto s0 = __builtin_amdgcn_permlane32_swap(pack(x[0], x[1]), pack(y[0], y[1]), false, false);
        const auto s1 = __builtin_amdgcn_permlane32_swap(pack(x[2], x[3]), pack(y[2], y[3]), false, false);
        const auto t0 = __builtin_amdgcn_permlane16_swap(s0[0], s0[1], false, false);
        const auto t1 = __builtin_amdgcn_permlane16_swap(s1[0], s1[1], false, false);
        uintx4 o;
        o[0] = t0[0];
        o[1] = t1[0];
        o[2] = t0[1];
        o[3] = t1[1];
        return o;
    };
    const int piece = 16 * (lane >> 5) + 8 * ((lane >> 4) & 1);
    const __amdgpu_buffer_rsrc_t rlo = __builtin_amdgcn_make_buffer_rsrc(
        static_cast<bf16_t*>(a.Out) + int64_t(t_first) * a.c_tok_stride + (FORM == GEMM_PARTS ? g.out_lo : 0), 0, 0x7fffffff, 0x00020000);
    auto low = [](const floatx4& v) -> floatx4 {
        floatx4 r;
#pragma unroll
        for (int e = 0; e < 4; ++e) r[e] = low_part(v[e]);
        return r;
    };
    if (FORM == GEMM_ANY && TRANS && g.scalar_out) {
        // lane: column l%16 of tile j, rows 4*(l/16) .. +3 of tile i
        uint32_t co[TN];
#pragma unroll
        for (int j = 0; j < TN; ++j) co[j] = col_offset(wn * TN * 16 + j * 16 + (lane & 15));
#pragma unroll
        for (int i = 0; i < TM; ++i) {
            uint32_t base[4];
#pragma unroll
            for (int v = 0; v < 4; ++v) base[v] = row_offset(wm * TM * 16 + i * 16 + 4 * (lane >> 4) + v);
#pragma unroll
            for (int j = 0; j < TN; ++j) {
                asm volatile("" : "+a"(acc[i][j]));
                __builtin_amdgcn_sched_barrier(0);
#pragma unroll
                for (int v = 0; v < 4; ++v)
                    __builtin_amdgcn_raw_buffer_store_b16(__builtin_bit_cast(unsigned short, bf16_t(acc[i][j][v])), ro,
                                                          int(((base[v] | co[j]) & OUT) ? ~0u : base[v] + co[j]), 0, 0);
            }
        }
    } else if (TRANS) {
        uint32_t base[TM / 2];
#pragma unroll
        for (int i = 0; i < TM / 2; ++i) base[i] = row_offset(wm * TM * 16 + i * 32 + piece);
#pragma unroll
        for (int j = 0; j < TN; ++j) {
            const uint32_t co = col_offset(wn * TN * 16 + j * 16 + (lane & 15));
            // (one column of tiles at a time: the scheduler otherwise converts all of them first, and spills)
#pragma unroll
            for (int i = 0; i < TM; ++i) asm volatile("" : "+a"(acc[i][j]));
            __builtin_amdgcn_sched_barrier(0);
#pragma unroll
            for (int i = 0; i < TM / 2; ++i)
                __builtin_amdgcn_raw_buffer_store_b128(merge(acc[2 * i][j], acc[2 * i + 1][j]), ro,
                                                       int(((base[i] | co) & OUT) ? ~0u : base[i] + co), 0, 0);
        }
    } else {
        uint32_t co[TN / 2];
#pragma unroll
        for (int j = 0; j < TN / 2; ++j) co[j] = col_offset(wn * TN * 16 + j * 32 + piece);
#pragma unroll
        for (int i = 0; i < TM; ++i) {
            const uint32_t base = row_offset(wm * TM * 16 + i * 16 + (lane & 15));
#pragma unroll
            for (int j = 0; j < TN; ++j) asm volatile("" : "+a"(acc[i][j]));
            __builtin_amdgcn_sched_barrier(0);
#pragma unroll
            for (int j = 0; j < TN / 2; ++j)
                __builtin_amdgcn_raw_buffer_store_b128(merge(acc[i][2 * j], acc[i][2 * j + 1]), ro,
                                                       int(((base | co[j]) & OUT) ? ~0u : base + co[j]), 0, 0);
            if (FORM == GEMM_PARTS && g.out_lo) {
#pragma unroll
                for (int j = 0; j < TN / 2; ++j)
                    __builtin_amdgcn_raw_buffer_store_b128(merge(low(acc[i][2 * j]), low(acc[i][2 * j + 1])), rlo,
                                                           int(((base | co[j]) & OUT) ? ~0u : base + co[j]), 0, 0);
            }
        }
    }
}
#endif

template <int TM, int TN, int NS, int TRANS, int FORM = GEMM_PLAIN>
__global__ void __launch_bounds__(256, FORM == GEMM_SHORT ? 3 : 1) step_gemm_kernel(StepArgs a, GemmArgs g) {
#ifdef __HIP_DEVICE_COMPILE__
    gemm_tile<TM, TN, NS, TRANS, FORM>(a, g);
#endif
}

// Products that do not wait for each other, in one launch: blockIdx.y says which. The two halves of a train are a few tiles each, and
// so are the four products that give its cores' gradients: a launch of one of them takes 4.6 us on an idle chip, whatever it does.
constexpr int kGemmMany = 4;
struct GemmMany {
    StepArgs a[kGemmMany];
    GemmArgs g[kGemmMany];
};

template <int TM, int TN, int NS, int FORM>
__global__ void __launch_bounds__(256, 1) step_gemm_many_kernel(GemmMany m) {
#ifdef __HIP_DEVICE_COMPILE__
    gemm_tile<TM, TN, NS, 0, FORM>(m.a[blockIdx.y], m.g[blockIdx.y]);
#endif
}
