// tn_linear: C-ABI library and gfx950 kernels for the forward pass of
// tensor-network linear layers (Section 3.5 of the paper: TN matmuls applied
// to token activations by sequential core contractions).
//
// Every contraction step of a plan (see tn_plan.hpp) is one launch of a
// "scatter GEMM":
//     Out[t, crow[r] + ccol[c]] = sum_k A[t, r, k] * Bp[c][k]
// A is the step's input (plain row-major [tokens*R, K] except possibly for the
// first step, which may gather from x through two tables), Bp is the packed
// parameter tensor [Cp][Kp] (K contiguous, zero padded), and the output is
// written directly in the layout the next step wants to read, so no separate
// permutation kernel ever runs.
#include <hip/hip_runtime.h>

#include <cmath>
#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <mutex>
#include <new>
#include <type_traits>
#include <utility>
#include <vector>

#include "../../include/tn_linear.h"
#include "tn_plan.hpp"
#include "tn_matrix.hpp"

// Scratch memory of tn_linear_forward_scratch: one array per GPU the library is loaded on, held until the
// process ends. Host code never uses this name as an address; it asks the runtime for the device address once
// per device (scratch_address) and passes that pointer on.
constexpr int64_t kScratchBytes = int64_t(32) << 20;
static __device__ __align__(256) unsigned char scratch[kScratchBytes];

namespace {

#include "kernels/common.hpp"
#include "kernels/pack.hpp"
#include "kernels/transpose.hpp"
#include "kernels/quant.hpp"
#include "kernels/tiled.hpp"
#include "kernels/gemm.hpp"
#include "kernels/stream.hpp"
#include "kernels/chained.hpp"
#include "kernels/factorpair.hpp"
#include "kernels/kronsum.hpp"
#include "kernels/krondirect.hpp"
#include "kernels/grad.hpp"

// ---------------------------------------------------------------------------------------------
// host side
// ---------------------------------------------------------------------------------------------
enum Variant : int {
    VAR_SCALAR = 0,
    VAR_MFMA_256x32 = 2,      // narrow outputs (<= 32 columns)
    VAR_PIPE_128x256 = 3,     // register-prefetch tiles, 4 waves, 2 workgroups per CU, one LDS stage
    VAR_PIPE_256x128 = 8,     // same, 4 waves stacked along rows
    VAR_SHORTK = 9,           // K <= 64, store-bound: registers-only operands, barrier-free
    VAR_GEMM = 12,            // plain A with K % 32 == 0, more than 64 rows: tiles chosen per launch (gemm_choice)
    VAR_KRONSUM = 20,         // (as a forced id only, read by tn::kron_shape) the Kronecker-sum kernel wherever
                              // the plan's layout allows it
};

struct DevStep {
    tn::Step plan;
    void* packed = nullptr;       // [Cp][Kp]
    const int32_t *arow = nullptr, *acol = nullptr, *crow = nullptr, *ccol = nullptr;
    int Kp = 0, Cp = 0;
    int variant = VAR_SCALAR;
    int amode = 0, cmode = 0;
    int bn = 64, bm = 64;
    bool fuse_next = false;       // this step and the next run as one launch
    void* chain_bbf = nullptr;    // chain2: the next step's packed tensor in the chained layout
    int chain_cfg = 0;            // chain2 instantiation: 0 <3,6,5>, 1 <2,8,2>, 2 <2,5,2>; 3: none, only pair_cfg
    int pair_cfg = -1;            // instantiation of the kernels with a workgroup to a token (factor_pair_configs), -1: none
    int64_t pair_gap[2] = {0, 0}; // calls of more tokens than the first and fewer than the second are left to step_chain2_kernel
    int chain_run_c1 = 0;         // chain2: output pieces run along c1 (else along c2)
    void* q4_codes = nullptr;     // 4-bit stream of the tensor for decode-size launches (codes, then block scales)
    void* q4_scales = nullptr;
    bool no_skinny = false;       // TN_FLAG_NO_SKINNY
    // gradient of the step's tensor as one product over the tokens: the row of c and the column of k in the caller's tensor
    const int32_t *grad_row = nullptr, *grad_col = nullptr;
    // operands and output in two parts (see step_gemm_kernel): how far the low ones are, in elements, 0: one part
    int64_t a_lo = 0, b_lo = 0, out_lo = 0;
    int segments() const { return 1 + (a_lo != 0) + (b_lo != 0); }
};

// One product of the matrix plan (tn_matrix.hpp) as a launch of the matrix-product kernel. What it reads is either kept by
// the layer or written by an earlier product of the same call.
struct DevProduct {
    DevStep s;                    // packed: the B operand
    const void* a = nullptr;      // the A operand
    void* out = nullptr;
};

}  // namespace

// A call on the kernel that makes the slices on chip: blocks of res_per x str_per values of the bond, a workgroup each.
struct DirectGeom {
    int res_per = 1, str_per = 1, str_blocks = 1, n_splits = 1;
    int64_t partial_bytes = 0;
    float us = 0.f;
    bool taken = false;       // the price is below that of the slices in memory
};
// Prices are kept for calls of up to this many tokens. Below it they decide: of a decoder's projections, rings of rank 96 are taken at one token in a
// workspace of their own and up to 2 to 4 in a shared one, of rank 32 up to 2 to 8 and 8 to 16; trains of rank 32 all the way.
constexpr int64_t kDirectMaxTokens = 16;

struct tn_linear_s {
    tn::Plan plan;
    std::vector<DevStep> steps;
    int elt = 4;
    int64_t max_tokens = 0, chunk_tokens = 0;
    int64_t packed_bytes = 0, workspace_bytes = 0;
    int32_t* tables = nullptr;        // arow | acol | crow | ccol of every step, one allocation
    void* ws[2] = {nullptr, nullptr};
    void* partial = nullptr;          // fp32 partial sums of the split-K kernel
    int64_t partial_bytes = 0;
    std::vector<tn::LaunchIO> schedule;   // launches of one pass over the chain and the buffers they use
    int flags = 0;
    bool owns_workspace = true;
    int device = 0;
    int num_cus = 256;
    bool profiling = false;
    // whole chain in one launch with everything in LDS (small layers)
    bool small_chain = false;
    void* small_chain_image = nullptr;    // descriptions, tensors (fp32, padded rows) and tables of all steps, as they sit in LDS
    int small_chain_image_words = 0;
    SmallChainDesc small_chain_desc[kSmallChainMaxSteps] = {};
    int small_chain_buf_words[2] = {0, 0};      // of a per-token buffer: an output per thread, tiles
    bool small_chain_tiles[2] = {false, false}; // the form on tiles: calls of up to a token per compute unit, larger ones
    // chained pair kernel (two-step plans of the train shape): second packed tensor in its layout
    bool pair = false;
    void* pair_b1f = nullptr;
    int64_t pair_min_tokens = 0;
    // Kronecker-sum kernel (two-step plans over a shared bond): both packed tensors in per-bond slices
    bool kron = false;
    tn::KronDims kron_dims;
    void* kron_h0f = nullptr;
    void* kron_h1f = nullptr;
    int64_t kron_min_tokens = 0;
    // the same kernel on a plan that exists only for large calls: the layer keeps its compact tensors and
    // steps, and calls of at least lazy_min_tokens tokens rebuild the merged plan's slices in the workspace
    bool lazy = false;
    bool lazy_slices_kept = false;    // the slices sit in memory only this handle writes (its own workspace): built once, at create
    tn::Plan lazy_plan;
    tn::KronDims lazy_dims;
    int64_t lazy_min_tokens = 0;
    int64_t lazy_kept_bytes = 0;              // what the lazy plan added to packed_bytes (sources and tables)
    int64_t lazy_slice_bytes = 0;             // both slice arrays
    int64_t lazy_h1_offset = 0;               // byte offset of the second array inside the slice buffer
    void* lazy_slices = nullptr;              // in the workspace (owned or caller's)
    std::vector<void*> lazy_sources;          // per half: the two tensors it is made of, as matrices [free][shared]
    int32_t* lazy_tables = nullptr;           // xrow | xcol | yrow | ycol of the merged plan
    const int32_t *lazy_xrow = nullptr, *lazy_xcol = nullptr, *lazy_yrow = nullptr, *lazy_ycol = nullptr;
    KronGenArgs lazy_gen[2];
    // the slices as two products of the matrix-product kernel, where the modes' digits allow it (tn::SlicePlan)
    bool lazy_products = false;
    DevProduct lazy_half[2];
    // the same slices by MFMA (one workgroup per value of the bond), where the half's shape allows it
    bool lazy_mfma[2] = {false, false};
    KronGenMfmaArgs lazy_gen_mfma[2];
    size_t lazy_gen_smem[2] = {0, 0};
    void* lazy_gen_tables[2] = {nullptr, nullptr};
    // calls of a few tokens of such a layer: the slices made on chip (tn::DirectPlan); what it keeps is in lazy_sources
    bool direct = false;
    int direct_cfg = 0, direct_steps = 1;
    KronDirectArgs direct_args;               // what does not depend on the call
    DirectGeom direct_geom[kDirectMaxTokens + 1];
    // calls whose token count lies in one of mat_ranges: the tensors contracted with each other into W, in the workspace and per
    // call, and then Y = X W^T (tn_matrix.hpp)
    bool matrix = false;
    std::vector<std::pair<int64_t, int64_t>> mat_ranges;      // [first, end), ascending
    int64_t mat_flops = 0;                    // of building W
    int64_t mat_bytes = 0;                    // W and the halves that are built per call
    int64_t mat_half_off[2] = {0, 0};         // byte offsets of the halves; W comes first
    void* mat_mem = nullptr;                  // in the workspace (owned or caller's)
    bool mat_build[2] = {false, false};       // the half is made of two tensors: built per call
    DevProduct mat_half[2], mat_w;
    DevStep mat_y;
    size_t mat_kept_count = 0;                // of mat_kept: those of the forward order, which come first
    int64_t mat_kept_bytes = 0;
    std::vector<void*> mat_kept;              // operands made from the caller's tensors, and the tables
    std::vector<SourceArgs> create_sources;   // operands that are still to be written (create time)
    std::vector<std::vector<int32_t>> create_tables;     // host copies of tables on their way to the GPU, until create's last wait
    // the plan of that order, made once and used by the two prepare functions; cleared when create ends
    struct MatrixPlans {
        bool tried = false, ok = false;
        tn::Plan net;
        tn::MatrixPlan m;
    } matrix_plans;
    // 4-bit form of the caller's tensors (TN_FLAG_QUANT_MXFP4): packed codes and block exponents per tensor
    std::vector<void*> quant_codes, quant_exps;
    std::vector<int64_t> quant_elems;
    int64_t quant_bytes = 0;
    int64_t q4_stream_bytes = 0;              // 4-bit streams of the steps whose decode-size launches read them
    std::vector<void*> create_temps;          // device buffers that only live until create returns
    // gradients with respect to the parameter tensors (TN_FLAG_TRAINABLE)
    bool trainable = false;
    std::vector<DevStep> bwd;                 // per step s >= 1: the step with its tensor transposed (gives dIn_s from dOut_s)
    int32_t* bwd_tables = nullptr;            // plain output tables of those steps
    void* bwd_ws = nullptr;                   // saved step inputs | two gradient buffers, for bwd_chunk tokens
    std::vector<int64_t> bwd_saved_off;       // element offset (per token block) of the saved input of step s
    int64_t bwd_saved_elems = 0;              // per token
    int64_t bwd_chunk = 0, bwd_ws_bytes = 0;
    float* bwd_partial = nullptr;
    int64_t bwd_partial_bytes = 0;
    void* grad_product_mem = nullptr;         // in bwd_ws: transposed operands of launch_grad_product
    // gradients of many tokens: dW = dY^T X, and from it those of the tensors on the cut of tn_matrix.hpp (a dense layer's
    // tensor is W)
    bool mgrad = false;
    int64_t mgrad_min_tokens = 0, mgrad_chunk = 0;
    int64_t mgrad_flops = 0;                  // of a pass, beside dW
    int64_t mgrad_f[2] = {0, 0};              // modes of the halves
    int64_t mgrad_off[10] = {};               // byte offsets in bwd_ws: X, dY; in two parts each: dW, dW transposed, the two
                                              // operands, and of either half dH, dH transposed
    bool mgrad_together = false;              // the halves' cores in shared launches (else they share the room for dH)
    DevStep mgrad_dw;                         // rows m, columns n; K, A and B are the call's
    struct GradHalf {
        bool pair = false;
        DevProduct op;                        // this half as the operand of the other one's gradient
        DevStep dh;                           // its gradient: rows its modes, columns the bond
        int64_t F1 = 0, F2 = 0, S = 0;
        void *a = nullptr, *b = nullptr;      // packed [S][F1 padded], [S][F2]
        tn::GradOut out_a, out_b;
    } mgrad_half[2];
    // both halves' gradients in one pass over dW (bond_grad_kernel), where the bond is narrow
    bool mgrad_bond = false;
    int32_t bond_ranges = 0, bond_tiles_per_range = 0;
    int64_t bond_sums_bytes[2] = {0, 0};      // at the start of bwd_partial
    struct ProfRec { int step; hipEvent_t start, stop; };
    std::vector<ProfRec> prof;
};

namespace {

constexpr int64_t kDefaultWorkspaceBytes = int64_t(4) << 30;

// The scratch memory a forward call works in: the two intermediate buffers (each holds chunk_tokens tokens
// of the largest intermediate) and the fp32 partial sums of the split kernels. Normally the handle's own
// workspace; tn_linear_forward_scratch carves it out of the library's static device array instead.
struct Workspace {
    void* ws[2] = {nullptr, nullptr};
    void* partial = nullptr;
    int64_t partial_bytes = 0;
    int64_t chunk_tokens = 0;
};

inline int round_up(int v, int m) { return (v + m - 1) / m * m; }

void clear_profile(tn_linear_s* h) {
    for (auto& r : h->prof) {
        (void)hipEventDestroy(r.start);
        (void)hipEventDestroy(r.stop);
    }
    h->prof.clear();
}

void free_handle(tn_linear_s* h) {
    if (!h) return;
    clear_profile(h);
    for (auto& s : h->steps) {
        if (s.packed) (void)hipFree(s.packed);
        if (s.chain_bbf) (void)hipFree(s.chain_bbf);
        if (s.q4_codes) (void)hipFree(s.q4_codes);       // one allocation: the scales follow the codes
    }
    if (h->tables) (void)hipFree(h->tables);
    for (void* v : h->quant_codes)
        if (v) (void)hipFree(v);
    for (void* v : h->quant_exps)
        if (v) (void)hipFree(v);
    for (void* v : h->create_temps)
        if (v) (void)hipFree(v);
    for (auto& b : h->bwd)
        if (b.packed) (void)hipFree(b.packed);
    if (h->bwd_tables) (void)hipFree(h->bwd_tables);
    if (h->bwd_ws) (void)hipFree(h->bwd_ws);
    if (h->bwd_partial) (void)hipFree(h->bwd_partial);
    if (h->pair_b1f) (void)hipFree(h->pair_b1f);
    if (h->kron_h0f) (void)hipFree(h->kron_h0f);
    if (h->kron_h1f) (void)hipFree(h->kron_h1f);
    for (void* v : h->lazy_sources)
        if (v) (void)hipFree(v);
    if (h->lazy_tables) (void)hipFree(h->lazy_tables);
    for (void* v : h->lazy_gen_tables)
        if (v) (void)hipFree(v);
    if (h->lazy_slices && h->owns_workspace) (void)hipFree(h->lazy_slices);
    for (void* v : h->mat_kept)
        if (v) (void)hipFree(v);
    if (h->mat_mem && h->owns_workspace) (void)hipFree(h->mat_mem);
    if (h->small_chain_image) (void)hipFree(h->small_chain_image);
    if (h->owns_workspace) {
        for (void* w : h->ws)
            if (w) (void)hipFree(w);
        if (h->partial) (void)hipFree(h->partial);
    }
    delete h;
}

void choose_variant(const tn_linear_s* h, DevStep* s, int flags) {
    const tn::Step& p = s->plan;
    if (h->plan.dtype != TN_DTYPE_BF16 || (flags & TN_FLAG_SCALAR_KERNELS)) {
        s->variant = VAR_SCALAR;
        s->bm = 64;
        s->bn = 64;
    } else if (p.C <= 32) {
        s->variant = VAR_MFMA_256x32;
        s->bm = 256;
        s->bn = 32;
    } else {
        int forced = (flags >> TN_FLAG_VARIANT_SHIFT) & 0xff;
        // default: the tile width that wastes the fewest padded columns (256 on a tie); the
        // register-only kernel for short-K, wide steps
        const bool shortk_ok = p.K <= 64 && p.c_vec == 8;
        int v = round_up(int(p.C), 128) < round_up(int(p.C), 256) ? VAR_PIPE_256x128 : VAR_PIPE_128x256;
        // the matrix-product kernel wherever A is a plain matrix, K a multiple of 32 and the output comes in aligned
        // pieces of 8: it has the tile sizes for any number of rows (777 rows x 5120 x 25600: 208 us, 506 us on 256x256
        // tiles of one size; 777 x 2304 x 5120: 28 us, 119 us on the split-K kernel that too few tiles led to)
        // Outputs in no such pieces (an odd number of columns) are stored one by one: from 256 columns on, where that does not pad
        // them further, it is still the faster kernel.
        const bool gemm_ok = p.a_plain && p.K % 32 == 0 && p.K >= 64 && p.K < (int64_t(1) << 21) &&
                             (p.c_vec == 8 || p.r_vec == 8 || (p.C >= 256 && round_up(int(p.C), 128) == round_up(int(p.C), 256)));
        if (gemm_ok) v = VAR_GEMM;
        if (shortk_ok && p.C >= 256) v = VAR_SHORTK;
        if (forced == VAR_PIPE_128x256 || forced == VAR_PIPE_256x128 || (forced == VAR_SHORTK && shortk_ok) ||
            (forced == VAR_GEMM && gemm_ok))
            v = forced;
        s->variant = v;
        switch (v) {
            case VAR_SHORTK: s->bm = 128; s->bn = 128; break;
            case VAR_PIPE_128x256: s->bm = 128; s->bn = 256; break;
            case VAR_PIPE_256x128: s->bm = 256; s->bn = 128; break;
            default: s->bm = 256; s->bn = p.C > 128 ? 256 : 128; break;      // VAR_GEMM
        }
    }
    // 0: plain rows of 16-byte pieces; 2: gathered rows of 16-byte pieces (the tiled pipeline kernel; every other kernel
    // reads such a step element by element, like 1); 1: element-wise gather; 3: 16-byte pieces along the rows (prepare_backward)
    s->amode = (p.a_plain && p.K % 8 == 0) ? 0 : (p.a_vec == 8 ? 2 : 1);
    s->cmode = p.c_vec == 8 ? 1 : (p.r_vec == 8 ? 2 : 0);
    s->Kp = round_up(int(p.K), 64);
    s->Cp = round_up(int(p.C), s->bn);
}

struct SplitCfg {
    bool use = false;
    int tm = 1, nw = 4, row_tiles = 0, col_blocks = 0, nsplit = 1, ksteps_per_split = 0;
    bool lds_rows = false;        // one row tile: the kernel that keeps the rows of A in LDS
    bool skinny = false;          // one row tile against 256 columns per workgroup (step_skinny_kernel)
    int64_t partial_bytes = 0;
};

constexpr int64_t kMaxPartialBytes = int64_t(64) << 20;
constexpr size_t kSplitLdsRowBytes = 144 * 1024;  // rows of A a split-K workgroup may keep in LDS (the reduction reuses it)
// Measured (dense 5120->8192 and 25600->5120, us per call, rows in LDS against rows gathered from memory): bf16 stream
// 1 row 17.5 / 19.3 and 56.3 / 60.0 (captured graph over 16 copies), 8 rows 18.6 / 15.8 (same layer back to back), 64
// rows (two row tiles, five splits to fit) 62.8 / 31.2; 4-bit stream 1 row 8.6 / 13.0, 8 rows 8.4 / 11.2, 64 rows
// 56.7 / 26.1. Hence: one row tile only; a bf16 stream up to 4 rows, a 4-bit stream up to 32.
constexpr int64_t kSplitLdsMaxBf16Rows = 4;
constexpr int64_t kSplitOneSplitBlocks = 128;
constexpr int kSkinnyFillWorkgroups = 256;       // compute units the skinny kernel's grid is planned for
constexpr int64_t kSkinnyLdsPerCu = 160 * 1024;  // LDS of a compute unit: bounds the workgroups it holds at a time
constexpr int64_t kSplitLdsMaxQ4Rows = 12;
constexpr int64_t kSkinnyMinRows = 8, kSkinnyMinRowsTimesK = 100000;

// Decide whether a launch of `rows` rows runs on the split-K kernel: when the tiled kernel would
// start fewer workgroups than there are compute units and K is long enough to share out.
SplitCfg split_config(const DevStep& s, int64_t rows) {
    SplitCfg c;
    if (s.variant == VAR_SCALAR || rows <= 0) return c;
    int64_t tiles = ((rows + s.bm - 1) / s.bm) * (s.Cp / s.bn);
    int nks = s.Kp / 16;
    // the narrow tile keeps 4 waves of a CU busy at best: it needs twice as many tiles to fill the chip
    if (tiles >= (s.variant == VAR_MFMA_256x32 ? 512 : 128) || nks < 8) return c;
    c.tm = rows > 32 ? 2 : 1;
    c.row_tiles = int((rows + 32 * c.tm - 1) / (32 * c.tm));
    c.col_blocks = int((s.plan.C + 31) / 32);
    int64_t base = int64_t(c.row_tiles) * c.col_blocks;
    // long K: wide workgroups (16 waves for up to 32 rows, 8 for up to 64), so that one split per
    // tile is enough to keep the weight stream busy and no reduction pass is needed
    c.nw = nks >= 64 ? 8 : 4;
    int64_t target_wgs = 3072 / c.nw;
    int want = int(std::max<int64_t>(1, target_wgs / base));
    int max_split = std::max(1, nks / (2 * c.nw));      // at least 2 k-steps per wave
    c.nsplit = std::min(want, max_split);
    if (c.row_tiles == 1 && base >= kSplitOneSplitBlocks) c.nsplit = 1;      // enough column blocks: no second pass over partial sums
    const bool rows_fit_as_planned =
        size_t(rows) * size_t(round_up((nks + c.nsplit - 1) / c.nsplit, 4) * 16 + 8) * 2 <= kSplitLdsRowBytes;
    const bool skinny_possible = c.row_tiles == 1 && nks % 4 == 0 && c.col_blocks >= 8 && !s.no_skinny;
    // a 4-bit stream whose rows would need extra splits to fit, or with many rows x K to copy per column block, goes
    // to the 256-column kernel instead
    if (c.row_tiles == 1 && c.tm == 1 && nks % 4 == 0 && rows <= (s.q4_codes ? kSplitLdsMaxQ4Rows : kSplitLdsMaxBf16Rows) &&
        !(s.q4_codes && skinny_possible && (!rows_fit_as_planned || rows * int64_t(s.plan.K) >= kSkinnyMinRowsTimesK))) {
        // the kernel that keeps the rows of A in LDS: enough splits that the rows' share of A fits (at least two
        // pieces of 64 k per wave stay in a split), and whole pieces of 64 k per split
        c.lds_rows = true;
        const int min_ksteps = 8 * c.nw;
        while (size_t(rows) * size_t(round_up((nks + c.nsplit - 1) / c.nsplit, 4) * 16 + 8) * 2 > kSplitLdsRowBytes &&
               (nks + c.nsplit) / (c.nsplit + 1) >= min_ksteps)
            ++c.nsplit;
    }
    if (!c.lds_rows && skinny_possible &&
        (rows > 32 || s.q4_codes || (rows >= kSkinnyMinRows && rows * int64_t(s.plan.K) >= kSkinnyMinRowsTimesK))) {
        // up to 64 rows against 256 columns per workgroup (step_skinny_kernel), every wave a column block of its own.
        // The number of splits (equal, whole pieces of 64 k, the rows' share of A within the LDS budget) is the one
        // with the least bytes on the critical path: the busiest CU runs ceil(grid / CUs) workgroups, each of which
        // moves its pieces of the stream and its rows of A (a quarter more when LDS leaves room for only one
        // workgroup per CU: nothing overlaps its start and end), and every split adds fp32 partial sums that are
        // written and read back.
        const int n_chunks = nks / 4, col_tiles = (c.col_blocks + 7) / 8;
        auto cps_of = [&](int ns) { return (n_chunks + ns - 1) / ns; };
        auto lds_bytes = [&](int ns) { return int64_t(rows) * (int64_t(cps_of(ns)) * 64 + 8) * 2; };
        const double stream_bytes_per_k = s.q4_codes ? 256 * 17.0 / 32.0 : 256 * 2.0;
        int best = 0;
        double best_cost = 0;
        for (int ns = 1; ns <= std::max(1, n_chunks / 2); ++ns) {
            if (ns > 1 && cps_of(ns) == cps_of(ns - 1)) continue;              // same pieces per split: more empty tail
            if (lds_bytes(ns) > int64_t(kSplitLdsRowBytes)) continue;
            const int n_real = (n_chunks + cps_of(ns) - 1) / cps_of(ns);
            const int64_t pb = n_real > 1 ? int64_t(n_real) * 32 * c.tm * s.Cp * 4 : 0;
            if (pb > kMaxPartialBytes) break;
            const int per_cu = int(std::max<int64_t>(1, std::min<int64_t>(4, kSkinnyLdsPerCu / std::max<int64_t>(1, lds_bytes(ns)))));
            const int64_t grid = int64_t(col_tiles) * n_real;
            const int64_t serial = (grid + kSkinnyFillWorkgroups - 1) / kSkinnyFillWorkgroups;      // workgroups the busiest CU runs
            const double wg_bytes = cps_of(ns) * 64.0 * (stream_bytes_per_k + 2.0 * double(rows));
            const double cost = double(serial) * wg_bytes * kSkinnyFillWorkgroups * (per_cu == 1 ? 1.25 : 1.0) + 2.0 * double(pb);
            if (!best || cost < best_cost) {
                best = ns;
                best_cost = cost;
            }
        }
        if (best) {
            const int cps = cps_of(best);
            c.skinny = true;
            c.nsplit = (n_chunks + cps - 1) / cps;
            c.ksteps_per_split = cps * 4;
            c.partial_bytes = c.nsplit > 1 ? int64_t(c.nsplit) * 32 * c.tm * s.Cp * 4 : 0;
            c.use = true;
            return c;
        }
    }
    for (;;) {
        c.ksteps_per_split = (nks + c.nsplit - 1) / c.nsplit;
        if (s.q4_codes || c.lds_rows) c.ksteps_per_split = round_up(c.ksteps_per_split, 4);    // pieces of 64 k
        c.nsplit = (nks + c.ksteps_per_split - 1) / c.ksteps_per_split;      // no empty split
        c.partial_bytes = c.nsplit > 1 ? int64_t(c.nsplit) * c.row_tiles * 32 * c.tm * s.Cp * 4 : 0;
        if (c.partial_bytes <= kMaxPartialBytes || c.nsplit == 1) break;
        c.nsplit = std::max(1, c.nsplit / 2);
    }
    c.use = true;
    return c;
}

template <int WM, int WN, int TM, int TN>
void launch_mfma(const DevStep& s, const StepArgs& a, dim3 grid, hipStream_t st) {
    if (s.amode == 0)
        hipLaunchKernelGGL((step_mfma_kernel<WM, WN, TM, TN, 0>), grid, dim3(256), 0, st, a, s.cmode);
    else
        hipLaunchKernelGGL((step_mfma_kernel<WM, WN, TM, TN, 1>), grid, dim3(256), 0, st, a, s.cmode);
}

template <int WM, int WN, int TM, int TN, int STAGES, int MINB>
int launch_pipe(const DevStep& s, const StepArgs& a, int64_t rows, hipStream_t st) {
    constexpr int BM = WM * TM * 32, BN = WN * TN * 32;
    constexpr size_t smem = pipe_smem_bytes<WM, WN, TM, TN, STAGES>();
    int nrow = int((rows + BM - 1) / BM), ncol = s.Cp / BN;
    int nrow_pad = (nrow + 7) / 8 * 8;
    dim3 grid(uint32_t(nrow_pad) * uint32_t(ncol));
    using kern_t = void (*)(StepArgs, int, int, int);
    constexpr int ROWS = BM == 256 ? 3 : 1;            // the mode of row runs where a thread has a block of 8 x 8 of the tile
    static const kern_t kerns[8] = {
        step_mfma_pipe_kernel<WM, WN, TM, TN, 0, STAGES, MINB, 0>, step_mfma_pipe_kernel<WM, WN, TM, TN, 1, STAGES, MINB, 0>,
        step_mfma_pipe_kernel<WM, WN, TM, TN, 2, STAGES, MINB, 0>, step_mfma_pipe_kernel<WM, WN, TM, TN, ROWS, STAGES, MINB, 0>,
        step_mfma_pipe_kernel<WM, WN, TM, TN, 0, STAGES, MINB, 1>, step_mfma_pipe_kernel<WM, WN, TM, TN, 1, STAGES, MINB, 1>,
        step_mfma_pipe_kernel<WM, WN, TM, TN, 2, STAGES, MINB, 1>, step_mfma_pipe_kernel<WM, WN, TM, TN, ROWS, STAGES, MINB, 1>};
    if (!s.packed) {                       // configuration call (create time): raise the kernels' LDS limit
        for (kern_t k : kerns)
            if (hipFuncSetAttribute(reinterpret_cast<const void*>(k), hipFuncAttributeMaxDynamicSharedMemorySize,
                                    int(smem)) != hipSuccess)
                return TN_ERR_HIP;
        return TN_OK;
    }
    kern_t k = kerns[(s.cmode == 2 ? 4 : 0) + s.amode];
    hipLaunchKernelGGL(k, grid, dim3(WM * WN * 64), smem, st, a, s.cmode, nrow, ncol);
    return TN_OK;
}

// Tile sizes of step_gemm_kernel, their LDS stages, and what they cost, in us: `t1` per K tile of 64 with one workgroup on every CU and
// `o1` per round of workgroups (start, first loads, stores); t2, o2 likewise with two on every CU, where they fit: there the
// start and the stores of one run under the products of the other, and short K or many rounds favour them (10240 x 4096 x 64: 160 x 128
// tiles 22.4 us, 224 x 256 24.1, 192 x 128 29). Fitted to 212 products of 70 to 15360 rows, 32 to 25600 columns and K of 64 to
// 40960, every tile and number of K ranges of each: the choice is 1.4 % above the best on average, 5 % at the 90th percentile, 20 %
// at most. 64 x 64 is for outputs of up to 64 columns, the gradients towards a bond, which read A once and are
// bound by the loads in flight. Larger tiles do more per us, smaller ones leave less of the last round of workgroups empty and
// pad fewer rows.
// As times, which is how the orders of contraction are compared, they are 6 % low on average with the column operand in the caches, as W is
// (0.92 to 1.19 of the price; 70 to 8192 rows of six products of up to 84 MB), and 13 % with it in memory (0.91 to 1.53, most at few rows); of
// the two products with 262 MB of it 10 % high (0.71 to 1.04).
struct GemmTile {
    int tm, tn, stages;
    float t1, o1, t2, o2;
};
constexpr int kGemmTiles = 14;
constexpr GemmTile kGemmTile[kGemmTiles] = {
    {8, 8, 2, 1.25f, 7.1f, 0.f, 0.f}, {7, 8, 2, 1.14f, 6.4f, 0.f, 0.f}, {6, 8, 2, 0.95f, 6.7f, 0.f, 0.f}, {5, 8, 3, 0.79f, 6.3f, 0.f, 0.f},
    {4, 8, 3, 0.69f, 5.3f, 0.f, 0.f}, {3, 8, 3, 0.59f, 4.4f, 0.f, 0.f}, {2, 8, 3, 0.43f, 4.6f, 0.f, 0.f}, {8, 4, 3, 0.71f, 4.8f, 0.f, 0.f},
    {6, 4, 3, 0.59f, 4.0f, 0.f, 0.f}, {5, 4, 2, 0.67f, 3.4f, 0.96f, 4.6f}, {4, 4, 2, 0.61f, 3.2f, 0.84f, 3.7f},
    {3, 4, 2, 0.54f, 3.2f, 0.71f, 2.9f}, {2, 4, 3, 0.27f, 3.4f, 0.60f, 2.4f},
    {2, 2, 4, 0.18f, 3.0f, 0.34f, 3.2f}};

// A K tile takes at least a load's time divided by the tiles in flight; a column operand above kGemmColdBytes comes from
// memory. Without this, 600 x 5120 x 8192 takes 64-row tiles (92 us instead of 65).
constexpr float kGemmColdUs = 1.0f, kGemmColdBytes = 60e6f;

struct GemmChoice {
    int tile = -1, n_split = 1, ktiles_per_split = 1;
    int64_t partial_bytes = 0;
    float us = 0.f;               // what it is expected to take
};

constexpr float kGemmLaunchUs = 3.f;
constexpr int64_t kGemmMinRows = 65;        // up to 64 rows the launch is a stream of the packed tensor: the kernels of stream.hpp
constexpr float kGemmPartialBytesPerUs = 5e6f;    // partial sums, written and read back, and the launch that adds them:
constexpr float kGemmReduceUs = 3.f;

// Tile of the form for K of one or two tiles (GEMM_SHORT), us per tile and the least it takes: 10240 x 4096 x 64 22.2 us (27.3 on the tiles
// above), 4096 x 23040 x 128 70 (74), 5120 x 25600 x 128 76 (84), 7168 x 5120 x 128 24.5 (31.6). 128 x 128 tiles take 21.6, 68, 77 and 25.5, 64 x 128 24.6, 74,
// 84 and 28.
constexpr int kGemmShortTm = 5, kGemmShortTn = 4;
constexpr float kGemmShortUs[2] = {0.009f, 0.0115f}, kGemmShortLeastUs[2] = {4.4f, 5.2f};

// A column operand above this passes through the caches once per band of four row tiles: 33 us for 262 MB, which tiles of 256 x 256
// hide and smaller ones less (4000 x 25600 x 5120: tiles of 256 rows 808 us, of 224 865, of 192 887, of 160 934; their K tiles alone
// 817, 805, 779, 764). One band and its remainder overlap (600 x 25600 x 5120: five tiles of 128 rows 157 us, four of 160 181).
constexpr float kGemmCachedBytes = 128e6f;

// The tile size and the number of K ranges with the least time for `rows` rows; partial sums within `cap` bytes.
// `brief`: the form for K of one or two tiles may be taken (tile = kGemmTiles).
// `only`: of this tile.
GemmChoice gemm_choice(const tn_linear_s* h, const DevStep& s, int64_t rows, int64_t cap, bool brief = false, int only = -1) {
    GemmChoice best;
    const int nk = s.Kp / 64 * s.segments();
    const bool trans = s.cmode != 1;
    const uint32_t cus = uint32_t(h->num_cus);
    const float b_bytes = 2.f * float(s.plan.C) * float(s.Kp);
    for (int t = only < 0 ? 0 : only; t < (only < 0 ? kGemmTiles : only + 1); ++t) {
        const GemmTile& g = kGemmTile[t];
        if (uint32_t(s.Cp) % uint32_t(32 * g.tn) || (trans && (g.tm & 1))) continue;
        const int64_t all_tiles = int64_t((uint32_t(rows) + 32 * g.tm - 1) / uint32_t(32 * g.tm)) *
                                  ((uint32_t(s.plan.C) + 32 * g.tn - 1) / uint32_t(32 * g.tn));      // rows and columns below 2^31
        if (all_tiles > (int64_t(1) << 26)) continue;
        const uint32_t tiles = uint32_t(all_tiles);
        // (an output of a few tiles: a core's gradient from that of its half, 128 x 64 with K of 2 x 5120, is a chain of K tiles that
        // wait for memory: 8 ranges 16 us, 32 ranges 7)
        const int most = tiles <= 16 ? 32 : 8;
        for (int ns = 1; ns <= most; ++ns) {
            // more ranges only while they fill an idle chip, at least 4 K tiles each
            if (ns > 1 && (trans || tiles * uint32_t(ns - 1) >= 2 * cus || nk < 4 * ns)) break;
            const int per = (nk + ns - 1) / ns, n_real = (nk + per - 1) / per;
            if (n_real != ns) continue;
            const int64_t pb = ns > 1 ? int64_t(ns) * rows * s.Cp * 4 : 0;
            if (pb > cap) break;
            const uint32_t items = tiles * uint32_t(ns);
            const uint32_t slots = g.t2 > 0.f ? 2 * cus : cus;
            const uint32_t full = items / slots, rest = items - full * slots;
            const bool half = g.t2 > 0.f && rest > 0 && rest <= cus;            // a last round with one workgroup per CU
            const float least = b_bytes > kGemmColdBytes ? kGemmColdUs / float(g.stages - 1) : 0.f;
            const float per_tile = std::max(g.t2 > 0.f ? g.t2 : g.t1, least), per_round = g.t2 > 0.f ? g.o2 : g.o1;
            const float rounds = float(full + (rest > 0 && !half ? 1 : 0));
            float us = rounds * per_round + (half ? g.o1 : 0.f) + float(per) * (rounds * per_tile + (half ? std::max(g.t1, least) : 0.f));
            if (b_bytes > kGemmCachedBytes) {
                const float bands = 0.25f * float((uint32_t(rows) + 32 * g.tm - 1) / uint32_t(32 * g.tm));
                const float shown = std::min(1.f, float(64 - g.tm * g.tn) / 24.f);       // the largest tiles hide the passes
                us += (1.25f + std::max(0.f, bands - 1.25f) * shown) * b_bytes / 8e6f;
            }
            if (ns > 1) us += kGemmReduceUs + 2.f * float(ns) * float(rows) * float(s.plan.C) * 4.f / kGemmPartialBytesPerUs;
            if (best.tile < 0 || us < best.us) {
                best.us = us;
                best.tile = t;
                best.n_split = ns;
                best.ktiles_per_split = per;
                best.partial_bytes = pb;
            }
        }
    }
    if (brief && !trans && nk <= 2 && uint32_t(s.Cp) % uint32_t(32 * kGemmShortTn) == 0) {
        const int64_t tiles = ((rows + 32 * kGemmShortTm - 1) / (32 * kGemmShortTm)) * ((s.plan.C + 32 * kGemmShortTn - 1) / (32 * kGemmShortTn));
        const float us = std::max(float(tiles) * kGemmShortUs[nk - 1] * 256.f / float(h->num_cus), kGemmShortLeastUs[nk - 1]);
        if (tiles <= (int64_t(1) << 26) && (best.tile < 0 || us < best.us)) {
            best = GemmChoice();
            best.us = us;
            best.tile = kGemmTiles;
            best.ktiles_per_split = nk;
        }
    }
    return best;
}

using gemm_kern_t = void (*)(StepArgs, GemmArgs);

template <int I, int TRANS, int FORM>
constexpr gemm_kern_t gemm_kernel_of() {
    if constexpr (TRANS && (kGemmTile[I].tm & 1)) return nullptr;
    else return step_gemm_kernel<kGemmTile[I].tm, kGemmTile[I].tn, kGemmTile[I].stages, TRANS, FORM>;
}

template <int TRANS, int FORM, int... I>
gemm_kern_t gemm_kernel_at(int tile, std::integer_sequence<int, I...>) {
    static const gemm_kern_t k[kGemmTiles] = {gemm_kernel_of<I, TRANS, FORM>()...};
    return k[tile];
}

template <int... I>
size_t gemm_smem_at(int tile, std::integer_sequence<int, I...>) {
    constexpr size_t b[kGemmTiles] = {GemmShape<kGemmTile[I].tm, kGemmTile[I].tn, kGemmTile[I].stages>::SMEM...};
    return b[tile];
}

gemm_kern_t gemm_kernel(int tile, bool trans, int form) {
    using seq = std::make_integer_sequence<int, kGemmTiles>;
    if (form == GEMM_PARTS) return trans ? nullptr : gemm_kernel_at<0, GEMM_PARTS>(tile, seq());
    if (form == GEMM_ANY) return trans ? gemm_kernel_at<1, GEMM_ANY>(tile, seq()) : gemm_kernel_at<0, GEMM_ANY>(tile, seq());
    return trans ? gemm_kernel_at<1, GEMM_PLAIN>(tile, seq()) : gemm_kernel_at<0, GEMM_PLAIN>(tile, seq());
}
gemm_kern_t gemm_short_kernel(int nk) {
    return nk == 1 ? step_gemm_kernel<kGemmShortTm, kGemmShortTn, 1, 0, GEMM_SHORT> : step_gemm_kernel<kGemmShortTm, kGemmShortTn, 2, 0, GEMM_SHORT>;
}
size_t gemm_short_smem(int nk) { return nk == 1 ? GemmShape<kGemmShortTm, kGemmShortTn, 1>::SMEM : GemmShape<kGemmShortTm, kGemmShortTn, 2>::SMEM; }

size_t gemm_smem(int tile) { return gemm_smem_at(tile, std::make_integer_sequence<int, kGemmTiles>()); }

// The tile of the launches of several products.
constexpr int kGemmManyTile = kGemmTiles - 1;
static_assert(kGemmTile[kGemmManyTile].tm == 2 && kGemmTile[kGemmManyTile].tn == 2, "64 x 64");
using gemm_many_t = void (*)(GemmMany);
gemm_many_t gemm_many_kernel(int form) {
    constexpr GemmTile t = kGemmTile[kGemmManyTile];
    return form == GEMM_PARTS ? step_gemm_many_kernel<t.tm, t.tn, t.stages, GEMM_PARTS> : step_gemm_many_kernel<t.tm, t.tn, t.stages, GEMM_PLAIN>;
}

int configure_gemm() {
    for (int form : {GEMM_PLAIN, GEMM_PARTS})
        if (hipFuncSetAttribute(reinterpret_cast<const void*>(gemm_many_kernel(form)), hipFuncAttributeMaxDynamicSharedMemorySize,
                                int(gemm_smem(kGemmManyTile))) != hipSuccess)
            return TN_ERR_HIP;
    for (int t = 0; t < kGemmTiles; ++t)
        for (int form = 0; form < 6; ++form) {
            const gemm_kern_t k = gemm_kernel(t, (form & 1) != 0, GEMM_PLAIN + form / 2);
            if (k && hipFuncSetAttribute(reinterpret_cast<const void*>(k), hipFuncAttributeMaxDynamicSharedMemorySize,
                                         int(gemm_smem(t))) != hipSuccess)
                return TN_ERR_HIP;
        }
    for (int nk = 1; nk <= 2; ++nk)
        if (hipFuncSetAttribute(reinterpret_cast<const void*>(gemm_short_kernel(nk)), hipFuncAttributeMaxDynamicSharedMemorySize,
                                int(gemm_short_smem(nk))) != hipSuccess)
            return TN_ERR_HIP;
    return TN_OK;
}

// Output offsets inside one tile are 31-bit byte offsets from its first token.
bool gemm_fits(const DevStep& s) {
    return s.variant == VAR_GEMM && (256 / s.plan.R + 2) * s.plan.c_tok_stride * 2 < (int64_t(1) << 31);
}

// fp32 sums instead of the output: where they went.
struct GemmSums {
    float* sums = nullptr;         // [n_split][rows][ld]
    int64_t ld = 0;
    int n_split = 1;
};

int gemm_form(const DevStep& s, const StepArgs& a) {
    return s.a_lo || s.b_lo || s.out_lo ? GEMM_PARTS : (a.K % 64 || s.cmode == 0 ? GEMM_ANY : GEMM_PLAIN);
}

GemmArgs gemm_args(const DevStep& s, const GemmTile& t, const GemmChoice& c, int64_t rows) {
    GemmArgs g;
    g.n_row = int32_t((rows + 32 * t.tm - 1) / (32 * t.tm));
    g.n_col = int32_t((s.plan.C + 32 * t.tn - 1) / (32 * t.tn));
    g.n_split = c.n_split;
    g.ktiles_per_split = c.ktiles_per_split;
    g.rows_pad = rows;
    g.ld = s.Cp;
    g.scalar_out = s.cmode == 0;
    g.a_lo = s.a_lo;
    g.b_lo = s.b_lo;
    g.out_lo = s.out_lo;
    g.partial = nullptr;
    return g;
}

// With `f32` the launch leaves its fp32 sums in `partial` (or at f32->sums, as one range with rows of f32->ld).
int launch_gemm(const tn_linear_s* h, const DevStep& s, const StepArgs& a, int64_t rows, void* partial, int64_t partial_bytes,
                hipStream_t st, GemmSums* f32 = nullptr) {
    const bool trans = s.cmode != 1;
    const bool one_range = (h->flags & TN_FLAG_NO_SPLIT_K) || !partial || (f32 && f32->sums);
    const int form = gemm_form(s, a);
    const GemmChoice c = gemm_choice(h, s, rows, one_range ? 0 : partial_bytes, form == GEMM_PLAIN && !f32);
    if (c.tile < 0 || (trans && (s.a_lo || s.b_lo || s.out_lo))) return TN_ERR_UNSUPPORTED;
    if (f32 && !f32->sums && (!partial || int64_t(c.n_split) * rows * s.Cp * 4 > partial_bytes)) return TN_ERR_UNSUPPORTED;
    const GemmTile t = c.tile == kGemmTiles ? GemmTile{kGemmShortTm, kGemmShortTn, 0} : kGemmTile[c.tile];
    GemmArgs g = gemm_args(s, t, c, rows);
    g.partial = c.n_split > 1 || f32 ? static_cast<float*>(partial) : nullptr;
    if (f32) {
        if (f32->sums) {
            g.partial = f32->sums;
            g.ld = f32->ld;
        }
        *f32 = GemmSums{g.partial, g.ld, c.n_split};
    }
    const int64_t items = int64_t(g.n_row) * g.n_col * g.n_split;
    const bool brief = c.tile == kGemmTiles;
    hipLaunchKernelGGL(brief ? gemm_short_kernel(s.Kp / 64) : gemm_kernel(c.tile, trans, form), dim3(uint32_t((items + 7) / 8 * 8)), dim3(256),
                       brief ? gemm_short_smem(s.Kp / 64) : gemm_smem(c.tile), st, a, g);
    if (c.n_split > 1 && !f32) {
        const int64_t total = rows * s.plan.C;
        const dim3 blocks(uint32_t(std::min<int64_t>((total + 255) / 256, 2048)));
        if (s.out_lo)
            hipLaunchKernelGGL(step_split_reduce_parts_kernel, blocks, dim3(256), 0, st, a, g.partial, c.n_split, uint32_t(rows), s.out_lo);
        else
            hipLaunchKernelGGL(step_split_reduce_kernel, blocks, dim3(256), 0, st, a, g.partial, c.n_split, uint32_t(rows));
    }
    return TN_OK;
}

// A launch for the matrix-product kernel: more than a row tile of rows; a step stored one by one only where the split-K kernel has no
// use for its ranges. (Short K whose output blocks are at most one round of the split-K kernel in one range is faster here too: K = 128,
// 66 to 1000 rows of 64 to 2048 columns 3.1 to 3.4 us, 5.7 to 6.2 there; K = 1024, 460 x 1024 5.6 and 8.4; of 350 calls of random
// layers with such steps none took longer, 11 took 0.76 to 0.95 of the time.)
bool gemm_rows(const DevStep& s, int64_t rows) {
    if (rows < kGemmMinRows || !gemm_fits(s)) return false;
    return s.cmode != 0 || !split_config(s, rows).use;
}

StepArgs product_args(const DevStep& s, const void* A, const void* B, void* out) {
    StepArgs a{};
    a.A = A;
    a.B = B;
    a.Out = out;
    a.crow = s.crow;
    a.ccol = s.ccol;
    a.total_rows = uint32_t(s.plan.R);
    a.R = uint32_t(s.plan.R);
    a.K = s.Kp;
    a.Kp = s.Kp;
    a.C = int32_t(s.plan.C);
    a.Cp = s.Cp;
    return a;
}

// One product of the matrix plan: out[crow[r] + ccol[c]] = sum_k A[r][k] B[c][k], or its fp32 sums.
int launch_product_of(const tn_linear_s* h, const DevStep& s, const void* A, const void* B, void* out, void* partial,
                      int64_t partial_bytes, hipStream_t st, GemmSums* f32 = nullptr) {
    const int rc = launch_gemm(h, s, product_args(s, A, B, out), s.plan.R, partial, partial_bytes, st, f32);
    if (rc != TN_OK) return rc;
    return hipGetLastError() == hipSuccess ? TN_OK : TN_ERR_HIP;
}

// Products that do not wait for each other: in one launch where none would take longer by more than that launch saves (halves of a
// rank-64 train 5120 -> 8192: 5.0 us, one after the other 9.4) and all of them fit the chip at once, else one by one. With `f32`
// they leave their sums, each in its own part of `partial`; otherwise they are outputs, in one range of K.
struct ProductJob {
    const DevStep* s;
    const void *A, *B;
    void* out;
    GemmSums f32;
};

int64_t one_range_bytes(const DevStep& s) { return (s.plan.R * s.Cp * 4 + 255) & ~int64_t(255); }

int launch_products(const tn_linear_s* h, ProductJob* jobs, int n, bool f32, void* partial, int64_t partial_bytes, hipStream_t st) {
    // the sums: a range's for each, and an equal share of what is left
    int64_t spare = partial_bytes, at[kGemmMany + 1] = {};
    for (int i = 0; i < n && f32; ++i) spare -= one_range_bytes(*jobs[i].s);
    if (n > kGemmMany || (f32 && spare < 0)) return TN_ERR_UNSUPPORTED;
    for (int i = 0; i < n && f32; ++i) at[i + 1] = at[i] + one_range_bytes(*jobs[i].s) + (spare / n & ~int64_t(255));
    GemmMany m;
    memset(&m, 0, sizeof(m));
    int64_t all = 0, most = 0;
    bool one = n > 1;
    int form = 0;
    for (int i = 0; i < n && one; ++i) {
        const DevStep& s = *jobs[i].s;
        m.a[i] = product_args(s, jobs[i].A, jobs[i].B, jobs[i].out);
        const int f = gemm_form(s, m.a[i]);
        one = s.cmode == 1 && f != GEMM_ANY && (i == 0 || f == form);
        form = f;
        if (!one) break;
        const bool ranges = !(h->flags & TN_FLAG_NO_SPLIT_K);
        const int64_t room = f32 ? at[i + 1] - at[i] : partial_bytes;
        const GemmChoice best = gemm_choice(h, s, s.plan.R, ranges ? room : 0, form == GEMM_PLAIN && !f32);
        const GemmChoice c = gemm_choice(h, s, s.plan.R, ranges && f32 ? room : 0, false, kGemmManyTile);
        one = c.tile >= 0 && c.us <= best.us + kGemmLaunchUs;
        if (!one) break;
        m.g[i] = gemm_args(s, kGemmTile[kGemmManyTile], c, s.plan.R);
        if (f32) {
            m.g[i].partial = reinterpret_cast<float*>(static_cast<char*>(partial) + at[i]);
            jobs[i].f32 = GemmSums{m.g[i].partial, m.g[i].ld, c.n_split};
        }
        const int64_t items = int64_t(m.g[i].n_row) * m.g[i].n_col * m.g[i].n_split;
        all += items;
        most = std::max(most, items);
    }
    if (one && all <= 2 * int64_t(h->num_cus)) {
        hipLaunchKernelGGL(gemm_many_kernel(form), dim3(uint32_t((most + 7) / 8 * 8), uint32_t(n)), dim3(256), gemm_smem(kGemmManyTile), st, m);
        return hipGetLastError() == hipSuccess ? TN_OK : TN_ERR_HIP;
    }
    for (int i = 0; i < n; ++i) {
        jobs[i].f32 = GemmSums{};
        const int rc = launch_product_of(h, *jobs[i].s, jobs[i].A, jobs[i].B, jobs[i].out, f32 ? static_cast<char*>(partial) + at[i] : partial,
                                         f32 ? at[i + 1] - at[i] : partial_bytes, st, f32 ? &jobs[i].f32 : nullptr);
        if (rc != TN_OK) return rc;
    }
    return TN_OK;
}

int launch_product(const tn_linear_s* h, const DevProduct& p, void* partial, int64_t partial_bytes, hipStream_t st) {
    return launch_product_of(h, p.s, p.a, p.s.packed, p.out, partial, partial_bytes, st);
}

// W from the layer's tensors, then Y = X W^T.
int launch_matrix_build(const tn_linear_s* h, void* partial, int64_t partial_bytes, hipStream_t st) {
    ProductJob jobs[2];
    int n = 0;
    for (int i = 0; i < 2; ++i)
        if (h->mat_build[i]) jobs[n++] = ProductJob{&h->mat_half[i].s, h->mat_half[i].a, h->mat_half[i].s.packed, h->mat_half[i].out, {}};
    const int rc = launch_products(h, jobs, n, false, partial, partial_bytes, st);
    if (rc != TN_OK) return rc;
    return launch_product(h, h->mat_w, partial, partial_bytes, st);
}

int launch_matrix_y(const tn_linear_s* h, const void* x, void* y, int64_t tokens, void* partial, int64_t partial_bytes, hipStream_t st) {
    const DevStep& s = h->mat_y;
    StepArgs a{};
    a.A = x;
    a.B = s.packed;
    a.Out = y;
    a.crow = s.crow;
    a.ccol = s.ccol;
    a.a_tok_stride = s.plan.a_tok_stride;
    a.c_tok_stride = s.plan.c_tok_stride;
    a.total_rows = uint32_t(tokens);
    a.R = 1;
    a.K = s.Kp;
    a.Kp = s.Kp;
    a.C = int32_t(s.plan.C);
    a.Cp = s.Cp;
    const int rc = launch_gemm(h, s, a, tokens, partial, partial_bytes, st);
    if (rc != TN_OK) return rc;
    return hipGetLastError() == hipSuccess ? TN_OK : TN_ERR_HIP;
}

// Instantiations of the split-K kernel that keeps the rows of A in LDS (one row tile of up to 32 rows): index
// (8 waves ? 4 : 0) + (gathered A ? 2 : 0) + (4-bit stream ? 1 : 0).
using split_lds_t = void (*)(StepArgs, float*, int, int);
constexpr int kSplitLdsKernels = 8;
const split_lds_t* split_lds_kernels() {
    static const split_lds_t lds[kSplitLdsKernels] = {
        step_split_lds_kernel<1, 0, 4, 0>, step_split_lds_kernel<1, 0, 4, 1>, step_split_lds_kernel<1, 1, 4, 0>,
        step_split_lds_kernel<1, 1, 4, 1>, step_split_lds_kernel<1, 0, 8, 0>, step_split_lds_kernel<1, 0, 8, 1>,
        step_split_lds_kernel<1, 1, 8, 0>, step_split_lds_kernel<1, 1, 8, 1>};
    return lds;
}

// step_skinny_kernel: index (tm - 1) * 4 + (gathered A ? 2 : 0) + (4-bit stream ? 1 : 0).
constexpr int kSkinnyKernels = 8;
using skinny_t = void (*)(StepArgs, float*, int, int, int);
const skinny_t* skinny_kernels() {
    static const skinny_t k[kSkinnyKernels] = {step_skinny_kernel<1, 0, 0>, step_skinny_kernel<1, 0, 1>, step_skinny_kernel<1, 1, 0>,
                                                  step_skinny_kernel<1, 1, 1>, step_skinny_kernel<2, 0, 0>, step_skinny_kernel<2, 0, 1>,
                                                  step_skinny_kernel<2, 1, 0>, step_skinny_kernel<2, 1, 1>};
    return k;
}

int launch_step(const tn_linear_s* h, const Workspace& w, const DevStep& s, const void* A, void* Out, int64_t tokens,
                hipStream_t st) {
    StepArgs a;
    a.A = A;
    a.B = s.packed;
    a.Out = Out;
    a.arow = s.arow;
    a.acol = s.acol;
    a.crow = s.crow;
    a.ccol = s.ccol;
    a.a_tok_stride = s.plan.a_tok_stride;
    a.c_tok_stride = s.plan.c_tok_stride;
    int64_t rows = tokens * s.plan.R;
    a.total_rows = uint32_t(rows);
    a.R = uint32_t(s.plan.R);
    a.K = int32_t(s.plan.K);
    a.Kp = s.Kp;
    a.C = int32_t(s.plan.C);
    a.Cp = s.Cp;
    if (gemm_rows(s, rows)) {
        const int rc = launch_gemm(h, s, a, rows, w.partial, w.partial_bytes, st);
        if (rc != TN_OK) return rc;
        return hipGetLastError() == hipSuccess ? TN_OK : TN_ERR_HIP;
    }
    SplitCfg sc = (h->flags & TN_FLAG_NO_SPLIT_K) ? SplitCfg() : split_config(s, rows);
    if (sc.use && (sc.partial_bytes == 0 || (w.partial && sc.partial_bytes <= w.partial_bytes))) {
        dim3 sgrid(uint32_t(sc.row_tiles), uint32_t(sc.col_blocks), uint32_t(sc.nsplit));
        float* part = static_cast<float*>(w.partial);
        using split_t = void (*)(StepArgs, float*, int);
        split_t k = nullptr;
        const int q4 = s.q4_codes ? 1 : 0;
        if (q4) {
            // the launch is a stream of the packed tensor: read its 4-bit form
            a.B = s.q4_codes;
            a.Bs = s.q4_scales;
        }
        const int x_ld = sc.ksteps_per_split * 16 + 8;
        const size_t x_bytes = size_t(rows) * size_t(x_ld) * sizeof(bf16_t);
        if (sc.skinny) {
            if (x_bytes > kSplitLdsRowBytes) return TN_ERR_UNSUPPORTED;       // split_config sized it to fit
            const dim3 kgrid(1, uint32_t((sc.col_blocks + 7) / 8), uint32_t(sc.nsplit));
            hipLaunchKernelGGL(skinny_kernels()[(sc.tm - 1) * 4 + (s.amode == 0 ? 0 : 2) + q4], kgrid, dim3(512), x_bytes, st, a,
                               part, sc.ksteps_per_split, x_ld, s.plan.c_vec >= 4 ? 1 : 0);
        } else if (sc.lds_rows && sc.tm == 1 && sc.row_tiles == 1 && sc.ksteps_per_split % 4 == 0 && x_bytes <= kSplitLdsRowBytes) {
            // one row tile whose share of A fits in LDS
            const size_t red_bytes = size_t(sc.nw) * sc.tm * 4096;
            hipLaunchKernelGGL(split_lds_kernels()[(sc.nw == 8 ? 4 : 0) + (s.amode == 0 ? 0 : 2) + q4], sgrid,
                               dim3(uint32_t(sc.nw * 64)), std::max(red_bytes, x_bytes), st, a, part, sc.ksteps_per_split, x_ld);
        } else if (q4) {
            if (sc.tm == 1)
                k = sc.nw == 8 ? (s.amode == 0 ? step_split_q4_kernel<1, 0, 8> : step_split_q4_kernel<1, 1, 8>)
                               : (s.amode == 0 ? step_split_q4_kernel<1, 0, 4> : step_split_q4_kernel<1, 1, 4>);
            else
                k = sc.nw == 8 ? (s.amode == 0 ? step_split_q4_kernel<2, 0, 8> : step_split_q4_kernel<2, 1, 8>)
                               : (s.amode == 0 ? step_split_q4_kernel<2, 0, 4> : step_split_q4_kernel<2, 1, 4>);
        } else if (sc.tm == 1)
            k = sc.nw == 8 ? (s.amode == 0 ? step_split_kernel<1, 0, 8> : step_split_kernel<1, 1, 8>)
                           : (s.amode == 0 ? step_split_kernel<1, 0, 4> : step_split_kernel<1, 1, 4>);
        else
            k = sc.nw == 8 ? (s.amode == 0 ? step_split_kernel<2, 0, 8> : step_split_kernel<2, 1, 8>)
                           : (s.amode == 0 ? step_split_kernel<2, 0, 4> : step_split_kernel<2, 1, 4>);
        if (k) hipLaunchKernelGGL(k, sgrid, dim3(uint32_t(sc.nw * 64)), 0, st, a, part, sc.ksteps_per_split);
        if (sc.nsplit > 1) {
            int64_t total = rows * s.plan.C;
            uint32_t blocks = uint32_t(std::min<int64_t>((total + 255) / 256, 2048));
            hipLaunchKernelGGL(step_split_reduce_kernel, dim3(blocks), dim3(256), 0, st, a, part, sc.nsplit,
                               uint32_t(sc.row_tiles * 32 * sc.tm));
        }
        return hipGetLastError() == hipSuccess ? TN_OK : TN_ERR_HIP;
    }
    dim3 grid(uint32_t((rows + s.bm - 1) / s.bm), uint32_t(s.Cp / s.bn));
    switch (s.variant) {
        case VAR_SCALAR:
            if (h->plan.dtype == TN_DTYPE_BF16)
                hipLaunchKernelGGL(step_scalar_kernel<bf16_t>, grid, dim3(256), 0, st, a);
            else
                hipLaunchKernelGGL(step_scalar_kernel<float>, grid, dim3(256), 0, st, a);
            break;
        case VAR_MFMA_256x32:
            launch_mfma<4, 1, 2, 1>(s, a, grid, st);
            break;
        case VAR_PIPE_128x256: {
            int rc = launch_pipe<2, 2, 2, 4, 1, 2>(s, a, rows, st);
            if (rc != TN_OK) return rc;
            break;
        }
        case VAR_GEMM: {
            // few rows without the split-K kernels; offsets that do not fit take the register-prefetch tiles
            int rc = gemm_fits(s) ? launch_gemm(h, s, a, rows, w.partial, w.partial_bytes, st) : launch_pipe<4, 1, 2, 4, 1, 2>(s, a, rows, st);
            if (rc != TN_OK) return rc;
            break;
        }
        case VAR_SHORTK: {
            // forms (tuning override in flag bits 16..19, value = form + 1): 0 = 64 rows per wave with
            // double-buffered packed fragments, 1 = 64 rows single-buffered, 2 = 32 rows single-buffered
            if (tokens * s.plan.c_tok_stride >= (int64_t(1) << 35)) {
                // output offsets would not fit the kernel's 32-bit (x8) row bases: use the tiled kernel
                int rc = launch_pipe<4, 1, 2, 4, 1, 2>(s, a, rows, st);
                if (rc != TN_OK) return rc;
                break;
            }
            // measured: 32 rows per wave at 4 workgroups per CU streams best when A is a plain matrix
            // (4.7 TB/s stored); with a gathered A the 64-row double-buffered form is slightly ahead
            int mode = (h->flags >> 16) & 0xf;
            mode = mode ? mode - 1 : (s.amode == 0 ? 2 : 0);
            const int wrows = mode == 2 ? 32 : 64;
            int64_t row_tiles = (rows + 2 * wrows - 1) / (2 * wrows);
            int col_iters = s.Cp / 128;
            int groups = int(std::min<int64_t>(col_iters, std::max<int64_t>(1, 1024 / row_tiles)));
            dim3 g{uint32_t(row_tiles), uint32_t(groups)};
            using k_t = void (*)(StepArgs);
            k_t k;
            if (mode == 2)
                k = s.amode == 0 ? step_shortk_kernel<0, 1, 0, 4> : step_shortk_kernel<1, 1, 0, 4>;
            else if (mode == 1)
                k = s.amode == 0 ? step_shortk_kernel<0, 2, 0, 3> : step_shortk_kernel<1, 2, 0, 3>;
            else
                k = s.amode == 0 ? step_shortk_kernel<0, 2, 1, 2> : step_shortk_kernel<1, 2, 1, 2>;
            hipLaunchKernelGGL(k, g, dim3(256), 0, st, a);
            break;
        }
        case VAR_PIPE_256x128: {
            int rc = launch_pipe<4, 1, 2, 4, 1, 2>(s, a, rows, st);
            if (rc != TN_OK) return rc;
            break;
        }
        default:
            return TN_ERR_UNSUPPORTED;
    }
    return hipGetLastError() == hipSuccess ? TN_OK : TN_ERR_HIP;
}

// Small layers: all steps in one launch when the packed tensors (as fp32, rows padded by one) and two
// per-token buffers fit in 96 KB of LDS. Used for fp32 layers at any token count (their other path is
// the plain FMA kernel, one launch per step) and for bf16 layers up to 32 tokens.
constexpr size_t kSmallChainMaxSmem = 96 * 1024;
// what they take with the buffers' banks padded (small_chain_word) and the steps' descriptions
constexpr size_t kSmallChainMaxLds = kSmallChainMaxSmem + kSmallChainMaxSmem / 16 + 1024;
constexpr int64_t kSmallChainMaxBf16Tokens = 32;

using small_chain_t = void (*)(SmallChainArgs);
small_chain_t small_chain_kernel_of(bool bf16, bool tiles) {
    if (bf16) return tiles ? small_chain_kernel<bf16_t, true> : small_chain_kernel<bf16_t, false>;
    return tiles ? small_chain_kernel<float, true> : small_chain_kernel<float, false>;
}

// Which form of the whole-chain kernel: what a token takes in each, in us, beside what both take. Fitted to 195 random layers
// (dense, trains, rings, Tucker; 1 to 5 steps) at 16 and 256 tokens, where a compute unit has one workgroup, and at 512 and 16384
// (`many`), where it has two. Of the layers one in three is faster on tiles, by up to 2.4 times, the others by up to 5 times with an output
// per thread (dense 256 x 64 at 16384 tokens 41 us, on tiles 215; the four steps 54 x 90 x 70 and smaller ones of a train 44 us at 16 tokens, on tiles
// 23). The choice is 0.2 % above the better one on average, 10 % at most (29 % at 16384 tokens), and no more than 3 % slower
// than an output per thread at any.
bool small_chain_on_tiles(const SmallChainImageArgs& im, bool many) {
    float threads = many ? -0.04f : -0.12f, tiles = 0.f;
    for (int s = 0; s < im.nsteps; ++s) {
        const SmallChainDesc& d = im.d[s];
        const float turns = float((int64_t(d.R) * d.C + small_chain_threads(false) - 1) / small_chain_threads(false));
        // an output per thread: per k one word of the tensor, whose rows fall on the same banks where their length has powers of two
        // in it, or with 16-byte reads a quarter of that; gathered, a table's word too
        float per_k = many ? 0.006f : 0.005f;
        if (d.gathered || (d.K & 3)) {
            const float rows = float(std::min(d.C, 64)) * float(std::min(d.ldb & -d.ldb, 64)) / 64.f;
            per_k = (d.gathered ? (many ? 0.0235f : 0.0177f) : (many ? 0.012f : 0.0102f)) + (many ? 0.0053f : 0.0029f) * (std::max(1.f, rows) - 1.f);
        }
        threads += (many ? 0.12f : 0.2f) + turns * ((many ? 0.42f : 0.327f) + per_k * float(d.K));
        // tiles: a wave's, one after another, and what all of them read from LDS
        const int n = (d.R + 15) / 16 * ((d.C + 15) / 16), waves = small_chain_threads(true) / 64, k16 = (d.K + 15) / 16;
        tiles += (many ? 0.084f : 0.226f) + float((n + waves - 1) / waves) * ((many ? 0.715f : 0.478f) + (many ? 0.286f : 0.305f) * float(k16)) +
                 (many ? 0.049f : 0.018f) * float(n) * float(k16);
    }
    return (many ? 1.1f : 1.05f) * tiles < threads;
}

int plan_small_chain(tn_linear_s* h, hipStream_t st) {
    if (h->flags & (TN_FLAG_SCALAR_KERNELS | TN_FLAG_NO_SMALL_CHAIN)) return TN_OK;
    const size_t ns = h->steps.size();
    if (ns == 0 || ns > size_t(kSmallChainMaxSteps)) return TN_OK;
    SmallChainImageArgs im;
    memset(&im, 0, sizeof(im));
    im.nsteps = int32_t(ns);
    const int64_t head = int64_t(ns) * kSmallChainDescWords;
    int64_t off = 0;                               // behind the descriptions
    for (size_t s = 0; s < ns; ++s) {
        const DevStep& d = h->steps[s];
        const tn::Step& p = d.plan;
        if (p.R * p.C > (int64_t(1) << 20)) return TN_OK;
        im.d[s].b_off = int32_t(head + off);
        im.d[s].R = int32_t(p.R);
        im.d[s].K = int32_t(p.K);
        im.d[s].C = int32_t(p.C);
        im.d[s].ldb = int32_t((p.K & 3) ? p.K + 1 : p.K + 4);
        im.d[s].gathered = p.a_plain ? 0 : 1;
        im.B[s] = d.packed;
        im.nks[s] = d.Kp >> 4;
        im.arow[s] = d.arow;
        im.acol[s] = d.acol;
        im.crow[s] = d.crow;
        im.ccol[s] = d.ccol;
        off += (p.C * ((p.K & 3) ? p.K + 1 : p.K + 4) + 3) & ~int64_t(3);      // every tensor starts 16-byte aligned
        if (off > int64_t(kSmallChainMaxSmem / 4)) return TN_OK;
    }
    for (size_t s = 0; s < ns; ++s) {              // the offset tables
        const tn::Step& p = h->steps[s].plan;
        im.d[s].t_off = int32_t(head + off);
        off += p.R + p.C + (p.a_plain ? 0 : p.R + p.K);
        if (off > int64_t(kSmallChainMaxSmem / 4)) return TN_OK;
    }
    off = (off + 3) & ~int64_t(3);
    const int64_t buf = (std::max(h->plan.N, h->plan.max_intermediate) + 3) & ~int64_t(3);
    if ((off + 2 * buf) * 4 > int64_t(kSmallChainMaxSmem)) return TN_OK;
    im.image_words = int32_t(head + off);
    memcpy(h->small_chain_desc, im.d, sizeof(im.d));
    for (int many = 0; many < 2; ++many) h->small_chain_tiles[many] = small_chain_on_tiles(im, many != 0);
    h->small_chain_buf_words[0] = int(buf);
    h->small_chain_buf_words[1] = small_chain_word(int(buf)) + 4;
    h->small_chain_image_words = im.image_words;
    if (hipMalloc(&h->small_chain_image, size_t(im.image_words) * 4) != hipSuccess) return TN_ERR_ALLOC;
    h->packed_bytes += int64_t(im.image_words) * 4;
    if (h->elt == 2)
        hipLaunchKernelGGL(small_chain_image_kernel<bf16_t>, dim3(1), dim3(256), 0, st, im, static_cast<float*>(h->small_chain_image));
    else
        hipLaunchKernelGGL(small_chain_image_kernel<float>, dim3(1), dim3(256), 0, st, im, static_cast<float*>(h->small_chain_image));
    if (hipGetLastError() != hipSuccess) return TN_ERR_HIP;
    h->small_chain = true;
    return TN_OK;
}

int launch_small_chain(const tn_linear_s* h, const void* x, void* y, int64_t tokens, hipStream_t st) {
    SmallChainArgs a;
    a.X = x;
    a.Y = y;
    a.image = static_cast<const float*>(h->small_chain_image);
    a.N = h->plan.N;
    a.M = h->plan.M;
    a.tokens = int32_t(tokens);
    a.nsteps = int32_t(h->steps.size());
    a.image_words = h->small_chain_image_words;
    const bool tiles = h->small_chain_tiles[tokens > h->num_cus ? 1 : 0];
    const int buf_words = h->small_chain_buf_words[tiles ? 1 : 0];
    a.buf_off[0] = a.image_words;
    a.buf_off[1] = a.image_words + buf_words;
    memcpy(a.d, h->small_chain_desc, sizeof(a.d));
    const size_t smem = size_t(a.image_words + 2 * buf_words) * 4;
    const dim3 block{uint32_t(small_chain_threads(tiles))};
    dim3 grid(uint32_t(std::min<int64_t>(tokens, int64_t(h->num_cus) * 2)));
    hipLaunchKernelGGL(small_chain_kernel_of(h->elt == 2, tiles), grid, block, smem, st, a);
    return hipGetLastError() == hipSuccess ? TN_OK : TN_ERR_HIP;
}

// The chained pair kernel runs every call of a layer it fits. With few token tiles (8 workgroups per 32 tokens) the
// range of a is split over workgroups, fp32 partial sums are written to the partial buffer and kron_reduce_kernel
// adds them in split order.
constexpr int64_t kPairMinTokens = 1;
#ifndef TN_PAIR_STAGES
#define TN_PAIR_STAGES 4
#define TN_PAIR_BAR 1
#endif
constexpr int kPairStages = TN_PAIR_STAGES, kPairBar = TN_PAIR_BAR;
constexpr size_t kPairSmemBytes = kPairStages * 20 * 1024;

struct PairGeom {
    int n_tok_tiles = 1, n_jsets = 1, n_splits = 1, a_per_split = 1;
    int64_t partial_bytes = 0;
};

PairGeom pair_geometry(const tn_linear_s* h, int64_t tokens, int64_t partial_cap) {
    PairGeom g;
    const int64_t A = h->steps[0].plan.R, J = h->steps[1].plan.R;
    g.n_tok_tiles = int((tokens + 31) / 32);
    g.n_jsets = int(J / 8);
    const int64_t base = int64_t(g.n_tok_tiles) * g.n_jsets;
    // one round of workgroups (a CU holds one): as many splits as keep the grid within the number of CUs
    int64_t want = std::max<int64_t>(1, int64_t(h->num_cus) / base);
    want = std::min<int64_t>(want, std::max<int64_t>(1, A / 2));                      // at least two values of a each
    // every split writes tokens * M floats that the reduction reads back: within one token tile the number of splits
    // that balances the two (measured at 8, 16 and 32 tokens: 16-20, 16, 13) grows as tokens^-1/2; with several
    // token tiles filling the chip matters more
    if (want > 1 && tokens <= 32) {
        const double per_split_mb = double(tokens) * double(h->plan.M) * 8.0 / 1e6;      // written and read
        const double best = std::sqrt(double(A) * 4.8 / per_split_mb);
        want = std::min<int64_t>(want, std::max<int64_t>(1, int64_t(best + 0.5)));
    }
    want = std::min<int64_t>(want, std::max<int64_t>(1, partial_cap / (tokens * h->plan.M * 4)));       // stays the last word
    g.a_per_split = int((A + want - 1) / want);
    g.n_splits = int((A + g.a_per_split - 1) / g.a_per_split);                        // no empty split
    g.partial_bytes = g.n_splits > 1 ? int64_t(g.n_splits) * tokens * h->plan.M * 4 : 0;
    return g;
}

int prepare_pair(tn_linear_s* h, hipStream_t st) {
    if ((h->flags & (TN_FLAG_NO_PAIR_CHAIN | TN_FLAG_SCALAR_KERNELS)) || !tn::pair_chainable(h->plan)) return TN_OK;
    const DevStep& s0 = h->steps[0];
    const DevStep& s1 = h->steps[1];
    if (s0.Kp != 64 || s0.Cp < s0.plan.C || s1.Kp != s1.plan.K) return TN_OK;
    const int A = int(s0.plan.R);
    if (hipMalloc(&h->pair_b1f, size_t(A) * 8192 * sizeof(bf16_t)) != hipSuccess) return TN_ERR_ALLOC;
    h->packed_bytes += int64_t(A) * 8192 * int64_t(sizeof(bf16_t));
    uint32_t blocks = uint32_t(std::min<int64_t>((int64_t(A) * 8192 + 255) / 256, 4096));
    hipLaunchKernelGGL(pair_repack_kernel, dim3(blocks), dim3(256), 0, st, static_cast<const bf16_t*>(s1.packed),
                       static_cast<bf16_t*>(h->pair_b1f), A, s1.Kp >> 4, s1.Cp);
    if (hipGetLastError() != hipSuccess) return TN_ERR_HIP;
    h->pair = true;
    h->pair_min_tokens = kPairMinTokens;
    return TN_OK;
}

int launch_pair(const tn_linear_s* h, const Workspace& w, const void* x, void* y, int64_t tokens, hipStream_t st) {
    const DevStep& s0 = h->steps[0];
    const DevStep& s1 = h->steps[1];
    const PairGeom g = pair_geometry(h, tokens, w.partial ? w.partial_bytes : 0);
    if (g.partial_bytes > (w.partial ? w.partial_bytes : 0)) return TN_ERR_UNSUPPORTED;      // never write past the buffer
    PairArgs p;
    p.X = x;
    p.Y = y;
    p.B0 = s0.packed;
    p.B1f = h->pair_b1f;
    p.yrow = s1.crow;
    p.ycol = s1.ccol;
    p.N = h->plan.N;
    p.M = h->plan.M;
    p.tokens = int32_t(tokens);
    p.A = int32_t(s0.plan.R);
    p.J = int32_t(s1.plan.R);
    p.C1 = int32_t(s1.plan.C);
    p.n_tok_tiles = g.n_tok_tiles;
    p.n_jsets = g.n_jsets;
    p.n_splits = g.n_splits;
    p.a_per_split = g.a_per_split;
    p.partial = static_cast<float*>(w.partial);
    const int64_t grid = p.n_splits > 1 ? int64_t(p.n_tok_tiles) * p.n_jsets * p.n_splits
                                        : int64_t((p.n_tok_tiles + 7) / 8 * 8) * p.n_jsets;
    hipLaunchKernelGGL((step_pair_kernel<kPairStages, kPairBar>), dim3(uint32_t(grid)), dim3(256), kPairSmemBytes, st, p);
    if (g.n_splits > 1) {
        const int64_t n = tokens * h->plan.M;
        hipLaunchKernelGGL(kron_reduce_kernel, dim3(uint32_t((n + 63) / 64)), dim3(256), 0, st,
                           static_cast<const float*>(w.partial), static_cast<bf16_t*>(y), n, g.n_splits);
    }
    return hipGetLastError() == hipSuccess ? TN_OK : TN_ERR_HIP;
}

// Kronecker-sum kernel: instantiations (see tn::kron_shape for the order) and launch geometry.
// From kKronMinTokens tokens on it replaces the two launches. A workgroup holds 4 tokens; when there are
// fewer workgroups than compute units the shared bond is split over several of them (fp32 partial sums,
// added by kron_reduce_kernel).
constexpr int64_t kKronMinTokens = 1;

struct KronTiles {
    int at = 0, ks0 = 0, o2t = 0, o1t = 0;
    size_t smem = 0;
    bool two_tokens = false;      // the instantiation with two tokens per wave exists
};

// Two tokens per wave where the registers allow it: at most 12 accumulation tiles (192 registers) for the two tokens'
// sums and at most 32 fragments of their inputs (<3,4,4,2> with 16 tiles spills).
template <int AT, int KS0, int O2T, int O1T>
constexpr bool kron_two_tokens_fit() { return 2 * O2T * O1T <= 12 && 2 * AT * KS0 <= 32; }

template <int AT, int KS0, int O2T, int O1T>
int kron_entry(const KronArgs* p, uint32_t grid, hipStream_t st, KronTiles* tiles) {
    using S = KronShape<AT, KS0, O2T, O1T>;
    constexpr bool two = kron_two_tokens_fit<AT, KS0, O2T, O1T>();
    if (tiles) {
        *tiles = KronTiles{AT, KS0, O2T, O1T, S::SMEM, two};
        return TN_OK;
    }
    if (!p) {       // configuration call (create time)
        bool ok = hipFuncSetAttribute(reinterpret_cast<const void*>(step_kronsum_kernel<AT, KS0, O2T, O1T, 0, 1>),
                                      hipFuncAttributeMaxDynamicSharedMemorySize, int(S::SMEM)) == hipSuccess &&
                  hipFuncSetAttribute(reinterpret_cast<const void*>(step_kronsum_kernel<AT, KS0, O2T, O1T, 1, 1>),
                                      hipFuncAttributeMaxDynamicSharedMemorySize, int(S::SMEM)) == hipSuccess;
        if constexpr (two)
            ok = ok && hipFuncSetAttribute(reinterpret_cast<const void*>(step_kronsum_kernel<AT, KS0, O2T, O1T, 0, 2>),
                                           hipFuncAttributeMaxDynamicSharedMemorySize, int(S::SMEM)) == hipSuccess;
        return ok ? TN_OK : TN_ERR_HIP;
    }
    if (p->share) {
        hipLaunchKernelGGL((step_kronsum_kernel<AT, KS0, O2T, O1T, 1, 1>), dim3(grid), dim3(256), S::SMEM, st, *p);
    } else if (p->tpw == 2) {
        if constexpr (two) hipLaunchKernelGGL((step_kronsum_kernel<AT, KS0, O2T, O1T, 0, 2>), dim3(grid), dim3(256), S::SMEM, st, *p);
        else return TN_ERR_UNSUPPORTED;
    } else {
        hipLaunchKernelGGL((step_kronsum_kernel<AT, KS0, O2T, O1T, 0, 1>), dim3(grid), dim3(256), S::SMEM, st, *p);
    }
    return TN_OK;
}

#define TN_KRON_CASE(i)                                                                                        \
    case i:                                                                                                   \
        return kron_entry<tn::kKronConfig[i][0], tn::kKronConfig[i][1], tn::kKronConfig[i][2], tn::kKronConfig[i][3]>( \
            p, grid, st, tiles);

int kron_dispatch(int cfg, const KronArgs* p, uint32_t grid, hipStream_t st, KronTiles* tiles = nullptr) {
    static_assert(tn::kKronConfigs == 8, "one case per instantiation");
    switch (cfg) {
        TN_KRON_CASE(0)
        TN_KRON_CASE(1)
        TN_KRON_CASE(2)
        TN_KRON_CASE(3)
        TN_KRON_CASE(4)
        TN_KRON_CASE(5)
        TN_KRON_CASE(6)
        TN_KRON_CASE(7)
        default: return TN_ERR_INVALID_ARG;
    }
}
#undef TN_KRON_CASE

struct KronGeom {
    int n_chunks = 1, n_splits = 1, rho_per_split = 1;
    int64_t quads = 1, partial_bytes = 0;
    bool share = false;       // the four waves of a workgroup share one token (quads then counts tokens)
    int tpw = 1;              // tokens per wave (quads then counts groups of 4 * tpw tokens)
};

// measured on seven ring classes with stored half rings (us per call, shared / a wave per token): one token 30/44,
// 110/214, 146/206, 79/119, 51/65, 31/35, 16/16; two tokens 34/44, 165/195, 214/204, 109/111, 65/63, 41/36, 18/17
constexpr int64_t kKronShareMaxTokens = 1;
// calls from which a wave takes two tokens, where that instantiation exists (8192->5120 at rank 64, ms per call, two / one:
// 64 tokens 0.63 / 0.67, 128 1.15 / 1.23, 300 2.46 / 2.74, 8192 58.4 / 65.6)
constexpr int64_t kKronTwoTokensMin = 64;

// workgroups a CU holds at a time: one when the three LDS stages take more than half of its 160 KB
int kron_per_cu(const tn::KronDims& d) {
    const int* c = tn::kKronConfig[d.cfg];
    return 3 * 4096 * ((c[3] * c[1] + c[2] * 2 * c[0] + 3) / 4) > 80 * 1024 ? 1 : 2;
}

constexpr float kKronPartialBytesPerUs = 3.5e6f;      // partial sums, written and read back

// What a launch of the Kronecker-sum kernel is expected to take: per value of the bond 21 ns per MFMA of a wave and 0.25 us (half of
// that where two workgroups on a CU share its matrix cores), values one after another, in rounds of workgroups; per round the start, longer
// with the fragments and stores of two tokens per wave; and the partial sums. Expected / measured, us: trains 5120 -> 25600 of rank
// 96 at 600 tokens 384 / 395, of rank 64 at 4000 1396 / 1499; 8192 -> 5120 of rank 32 at 600 99 / 108, of rank 96 at 4000 722 /
// 764; 25600 -> 5120 of rank 96 at 4000 1434 / 1492; 5120 -> 8192 of rank 96 at 600 189 / 191.
float kron_us(const tn_linear_s* h, const tn::KronDims& d, const KronGeom& g) {
    const int* c = tn::kKronConfig[d.cfg];
    const int per_cu = kron_per_cu(d);
    const int64_t slots = int64_t(h->num_cus) * per_cu;
    const int64_t wgs = g.quads * g.n_chunks * g.n_splits;
    const int64_t rounds = (wgs + slots - 1) / slots, turns = (wgs + h->num_cus - 1) / h->num_cus;
    const float per_rho = float(c[3] * c[0] * (c[1] + 2 * c[2]) * g.tpw) * 0.021f + 0.25f / float(per_cu);
    return 10.f + float(rounds) * (g.tpw == 2 && per_cu == 1 ? 42.f : 10.f) + float(turns) * float(g.rho_per_split) * per_rho +
           float(g.partial_bytes) / kKronPartialBytesPerUs;
}

KronGeom kron_geometry(const tn_linear_s* h, const tn::KronDims& d, int64_t tokens, int64_t partial_cap) {
    KronGeom g;
    const int o1_chunk = 32 * tn::kKronConfig[d.cfg][3];
    g.n_chunks = int((d.O1 + o1_chunk - 1) / o1_chunk);
    g.share = tokens <= kKronShareMaxTokens && !(h->flags & TN_FLAG_NO_DECODE_FUSION);
    {
        KronTiles kt;
        const bool two = kron_dispatch(d.cfg, nullptr, 0, nullptr, &kt) == TN_OK && kt.two_tokens;
        g.tpw = (two && tokens >= kKronTwoTokensMin) ? 2 : 1;
    }
    g.quads = g.share ? tokens : (tokens + 4 * g.tpw - 1) / (4 * g.tpw);
    int64_t base = g.quads * g.n_chunks;
    // As many splits as keep the grid within one round of workgroups (rounding up instead left a second round with a handful of
    // workgroups: 300 tokens took as long as 512), at least 4 values of the bond each, partial sums within their buffer. Where
    // the chunks of o1 are several and a CU holds one workgroup, also two rounds; and 2 values each where 4 leave CUs without a
    // workgroup: whichever is priced lowest, the partial sums counted twice (at 24 tokens the rank-64 train 8192 ->
    // 5120 gains less from 2 values each than they cost: 33.8 / 34.5 us). Two rounds pay the start and the partial sums twice, but
    // divide the bond more evenly. us per call of rings 5120 -> 25600 in two rounds / one: rank 32 84 / 65 at one token, 133 / 100 at 8, 334 / 343 at 56;
    // rank 64 284 / 248 at 8, 536 / 500 at 24, 1138 / 1247 at 56. Trains of rank 96 and 64 at 4 values / at 2: 25600 -> 5120 37.5 / 34.9 at one
    // token, 48.5 / 45.4 at 16; 5120 -> 25600 at 4 tokens 35.0 / 36.9 (rank 64), 41.6 / 44.6.
    const int64_t cap = std::max<int64_t>(1, partial_cap / (tokens * h->plan.M * 4));
    auto with = [&](int64_t want) {
        KronGeom c = g;
        want = std::min(want, cap);
        c.rho_per_split = int((d.P + want - 1) / want);
        c.n_splits = int((d.P + c.rho_per_split - 1) / c.rho_per_split);      // no empty split
        c.partial_bytes = c.n_splits > 1 ? int64_t(c.n_splits) * tokens * h->plan.M * 4 : 0;
        return c;
    };
    if (base >= h->num_cus) return with(1);
    const bool one_per_cu = kron_per_cu(d) == 1;
    KronGeom best;
    float best_us = 0.f;
    bool any = false;
    for (int rounds = one_per_cu ? 1 : 2; rounds <= (one_per_cu && g.n_chunks == 1 ? 1 : 2); ++rounds)
        for (int least = 4; least >= 2; least -= 2) {
            const int64_t fit = std::max<int64_t>(1, rounds * int64_t(h->num_cus) / base), most = std::max<int64_t>(1, d.P / least);
            if (least == 2 && (fit <= std::max<int64_t>(1, d.P / 4) || base * std::max<int64_t>(1, d.P / 4) >= h->num_cus)) continue;
            const KronGeom c = with(std::min(fit, most));
            const float us = kron_us(h, d, c) + float(c.partial_bytes) / kKronPartialBytesPerUs;
            if (!any || us < best_us) {
                best = c;
                best_us = us;
                any = true;
            }
        }
    return best;
}

int prepare_kron(tn_linear_s* h, hipStream_t st) {
    if ((h->flags & (TN_FLAG_NO_PAIR_CHAIN | TN_FLAG_SCALAR_KERNELS)) || h->pair || h->small_chain) return TN_OK;
    tn::KronDims d;
    if (!tn::kron_shape(h->plan, &d)) return TN_OK;
    const DevStep& s0 = h->steps[0];
    const DevStep& s1 = h->steps[1];
    if (s0.variant == VAR_SCALAR || s1.variant == VAR_SCALAR) return TN_OK;
    KronTiles kt;
    if (kron_dispatch(d.cfg, nullptr, 0, nullptr, &kt) != TN_OK) return TN_OK;
    const int at = kt.at, ks0 = kt.ks0, o2t = kt.o2t, o1t = kt.o1t;
    const int n_chunks = int((d.O1 + 32 * o1t - 1) / (32 * o1t));
    const int64_t e0 = int64_t(n_chunks) * d.P * o1t * ks0 * 512;
    const int64_t e1 = d.P * int64_t(o2t) * 2 * at * 512;
    if (hipMalloc(&h->kron_h0f, size_t(e0) * sizeof(bf16_t)) != hipSuccess) return TN_ERR_ALLOC;
    if (hipMalloc(&h->kron_h1f, size_t(e1) * sizeof(bf16_t)) != hipSuccess) return TN_ERR_ALLOC;
    h->packed_bytes += (e0 + e1) * int64_t(sizeof(bf16_t));
    hipLaunchKernelGGL(kron_repack0_kernel, dim3(uint32_t(std::min<int64_t>((e0 + 255) / 256, 8192))), dim3(256), 0, st,
                       static_cast<const bf16_t*>(s0.packed), static_cast<bf16_t*>(h->kron_h0f), n_chunks, int(d.P), ks0,
                       o1t, int(d.O1), int(d.K0), s0.Kp >> 4);
    hipLaunchKernelGGL(kron_repack1_kernel, dim3(uint32_t(std::min<int64_t>((e1 + 255) / 256, 8192))), dim3(256), 0, st,
                       static_cast<const bf16_t*>(s1.packed), static_cast<bf16_t*>(h->kron_h1f), int(d.P), o2t, at,
                       int(d.C1), int(d.A), s1.Kp >> 4);
    if (hipGetLastError() != hipSuccess) return TN_ERR_HIP;
    h->kron = true;
    h->kron_dims = d;
    h->kron_min_tokens = kKronMinTokens;
    if (h->kron_min_tokens <= 1) {
        // every call runs the one-launch kernel: the per-step packed tensors are not needed any more
        if (hipStreamSynchronize(st) != hipSuccess) return TN_ERR_HIP;
        for (DevStep& s : h->steps) {
            h->packed_bytes -= int64_t(s.Cp) * s.Kp * h->elt;
            (void)hipFree(s.packed);
            s.packed = nullptr;
        }
    }
    return TN_OK;
}

struct KronSetup {
    const tn::KronDims* dims;
    const void *h0f, *h1f;
    const int32_t *xrow, *xcol, *yrow, *ycol;
};

int launch_kron(const tn_linear_s* h, const Workspace& w, const KronSetup& k, const void* x, void* y, int64_t tokens,
                hipStream_t st) {
    const tn::KronDims& d = *k.dims;
    const KronGeom g = kron_geometry(h, d, tokens, w.partial ? w.partial_bytes : 0);
    if (g.partial_bytes > (w.partial ? w.partial_bytes : 0)) return TN_ERR_UNSUPPORTED;      // never write past the buffer
    KronArgs p;
    p.X = x;
    p.Y = g.n_splits > 1 ? w.partial : y;
    p.H0f = k.h0f;
    p.H1f = k.h1f;
    p.xrow = k.xrow;
    p.xcol = k.xcol;
    p.yrow = k.yrow;
    p.ycol = k.ycol;
    p.N = h->plan.N;
    p.M = h->plan.M;
    p.tokens = int32_t(tokens);
    p.A = int32_t(d.A);
    p.K0 = int32_t(d.K0);
    p.O1 = int32_t(d.O1);
    p.C1 = int32_t(d.C1);
    p.P = int32_t(d.P);
    p.n_chunks = g.n_chunks;
    p.n_splits = g.n_splits;
    p.rho_per_split = g.rho_per_split;
    p.x_vec8 = d.x_vec8 ? 1 : 0;
    p.share = g.share ? 1 : 0;
    p.tpw = g.tpw;
    const int64_t grid = g.quads * g.n_chunks * g.n_splits;
    int rc = kron_dispatch(d.cfg, &p, uint32_t(grid), st);
    if (rc != TN_OK) return rc;
    if (g.n_splits > 1) {
        const int64_t n = tokens * h->plan.M;
        hipLaunchKernelGGL(kron_reduce_kernel, dim3(uint32_t((n + 63) / 64)), dim3(256), 0, st,
                           static_cast<const float*>(w.partial), static_cast<bf16_t*>(y), n, g.n_splits);
    }
    return hipGetLastError() == hipSuccess ? TN_OK : TN_ERR_HIP;
}

int launch_kron_eager(const tn_linear_s* h, const Workspace& w, const void* x, void* y, int64_t tokens, hipStream_t st) {
    const DevStep& s0 = h->steps[0];
    const DevStep& s1 = h->steps[1];
    KronSetup k{&h->kron_dims, h->kron_h0f, h->kron_h1f, s0.plan.a_plain ? nullptr : s0.arow,
                s0.plan.a_plain ? nullptr : s0.acol, s1.crow, s1.ccol};
    return launch_kron(h, w, k, x, y, tokens, st);
}

// Large calls of a layer with a lazily merged plan: rebuild the two slice arrays in the workspace from the
// library's copies of the caller's tensors (once per call), then run the Kronecker-sum kernel on them.
constexpr size_t kGenMfmaMaxSmem = 160 * 168 * 2;

int gen_mfma_dispatch(const KronGenMfmaArgs* a, size_t smem, hipStream_t st) {
    using kern_t = void (*)(KronGenMfmaArgs);
    static const kern_t kerns[4] = {kron_generate_mfma_kernel<2>, kron_generate_mfma_kernel<4>, kron_generate_mfma_kernel<6>,
                                    kron_generate_mfma_kernel<8>};
    if (!a) {               // configuration call (create time)
        for (kern_t k : kerns)
            if (hipFuncSetAttribute(reinterpret_cast<const void*>(k), hipFuncAttributeMaxDynamicSharedMemorySize,
                                    int(kGenMfmaMaxSmem)) != hipSuccess)
                return TN_ERR_HIP;
        return TN_OK;
    }
    const int idx = (a->Sp + 31) / 32 - 1;
    if (idx < 0 || idx > 3) return TN_ERR_INVALID_ARG;
    hipLaunchKernelGGL(kerns[idx], dim3(uint32_t(a->P)), dim3(256), smem, st, *a);
    return TN_OK;
}

int gen_mfma_both_dispatch(const KronGenMfmaArgs* a0, const KronGenMfmaArgs* a1, size_t smem, hipStream_t st) {
    using kern_t = void (*)(KronGenMfmaArgs, KronGenMfmaArgs);
    static const kern_t kerns[4] = {kron_generate_mfma_both_kernel<2>, kron_generate_mfma_both_kernel<4>,
                                    kron_generate_mfma_both_kernel<6>, kron_generate_mfma_both_kernel<8>};
    if (!a0) {              // configuration call (create time)
        for (kern_t k : kerns)
            if (hipFuncSetAttribute(reinterpret_cast<const void*>(k), hipFuncAttributeMaxDynamicSharedMemorySize,
                                    int(kGenMfmaMaxSmem)) != hipSuccess)
                return TN_ERR_HIP;
        return TN_OK;
    }
    const int idx = (std::max(a0->Sp, a1->Sp) + 31) / 32 - 1;
    if (idx < 0 || idx > 3) return TN_ERR_INVALID_ARG;
    hipLaunchKernelGGL(kerns[idx], dim3(uint32_t(a0->P + a1->P)), dim3(256), smem, st, *a0, *a1);
    return TN_OK;
}

int launch_lazy_generate(const tn_linear_s* h, hipStream_t st) {
    if (h->lazy_products) {
        int rc = launch_product(h, h->lazy_half[0], nullptr, 0, st);
        return rc != TN_OK ? rc : launch_product(h, h->lazy_half[1], nullptr, 0, st);
    }
    if (h->lazy_mfma[0] && h->lazy_mfma[1]) {
        int rc = gen_mfma_both_dispatch(&h->lazy_gen_mfma[0], &h->lazy_gen_mfma[1],
                                        std::max(h->lazy_gen_smem[0], h->lazy_gen_smem[1]), st);
        if (rc != TN_OK) return rc;
        return hipGetLastError() == hipSuccess ? TN_OK : TN_ERR_HIP;
    }
    for (int w = 0; w < 2; ++w) {
        if (h->lazy_mfma[w]) {
            int rc = gen_mfma_dispatch(&h->lazy_gen_mfma[w], h->lazy_gen_smem[w], st);
            if (rc != TN_OK) return rc;
            continue;
        }
        const KronGenArgs& g = h->lazy_gen[w];
        const int64_t pieces = w == 0 ? int64_t(g.n_chunks) * g.P * g.O1T * g.KS0 * 64 : int64_t(g.P) * g.O2T * 2 * g.AT * 64;
        hipLaunchKernelGGL(kron_generate_kernel, dim3(uint32_t(std::min<int64_t>((pieces + 255) / 256, 1 << 20))), dim3(256),
                           0, st, g);
    }
    return hipGetLastError() == hipSuccess ? TN_OK : TN_ERR_HIP;
}

// Tables of the MFMA form of the slice generation for half w (see kron_generate_mfma_kernel): which rows of the
// two source matrices a value of the bond uses, and where each element of a slice sits in their product.
// perm maps the kernels' numbering of k (w = 0) or a (w = 1) to the plan's. Returns false (and leaves the scalar
// kernel in charge) when the half does not fit: more than 160 distinct rows on a side or a shared bond longer
// than 128.
bool prepare_gen_mfma(tn_linear_s* h, int w, const KronGenArgs& g, const tn::KronDims& d, int64_t merged_C,
                      const std::vector<int32_t>& perm, hipStream_t st) {
    if (g.Sp > 128 || g.Sp % 16) return false;
    const int64_t P = d.P;
    struct Elem { int64_t rP, rQ; };
    const int64_t pieces = w == 0 ? int64_t(g.n_chunks) * g.O1T * g.KS0 * 64 : int64_t(g.O2T) * 2 * g.AT * 64;
    std::vector<Elem> elems(size_t(pieces) * 8, Elem{-1, -1});
    for (int64_t lp = 0; lp < pieces; ++lp) {
        const int l = int(lp & 63);
        int64_t blk = lp >> 6;
        for (int e = 0; e < 8; ++e) {
            int64_t cB, kB;
            bool inside;
            if (w == 0) {
                int64_t b2 = blk;
                const int ks = int(b2 % g.KS0);
                b2 /= g.KS0;
                const int o1t = int(b2 % g.O1T);
                const int chunk = int(b2 / g.O1T);
                const int64_t o1 = int64_t(32) * g.O1T * chunk + 32 * o1t + (l & 31);
                const int64_t k = 16 * ks + 8 * (l >> 5) + e;
                inside = o1 < d.O1 && k < d.K0;
                cB = o1 * P;
                kB = inside ? perm[size_t(k)] : 0;
            } else {
                const int is = int(blk % (2 * g.AT));
                const int j = int(blk / (2 * g.AT));
                const int64_t c = 32 * j + (l & 31);
                const int64_t a = 16 * is + 8 * (e >> 2) + 4 * (l >> 5) + (e & 3);
                inside = c < d.C1 && a < d.A;
                cB = c;
                kB = inside ? int64_t(perm[size_t(a)]) * P : 0;
            }
            if (!inside) continue;
            const int64_t m = gen_offset(g.sc, cB) + gen_offset(g.sk, kB);
            elems[size_t(lp) * 8 + e] = Elem{m / merged_C, m % merged_C};
        }
    }
    // the column side of the product is the tensor whose row changes from one element of a piece to the next
    bool cols_from_q = true;
    for (size_t i = 0; i + 1 < elems.size(); i += 8)
        if (elems[i].rP >= 0 && elems[i + 1].rP >= 0) {
            cols_from_q = elems[i].rQ != elems[i + 1].rQ;
            break;
        }
    std::vector<int64_t> rows_r, rows_c;
    for (const Elem& el : elems)
        if (el.rP >= 0) {
            rows_r.push_back(cols_from_q ? el.rP : el.rQ);
            rows_c.push_back(cols_from_q ? el.rQ : el.rP);
        }
    auto uniq = [](std::vector<int64_t>* v) {
        std::sort(v->begin(), v->end());
        v->erase(std::unique(v->begin(), v->end()), v->end());
    };
    uniq(&rows_r);
    uniq(&rows_c);
    const int64_t NR = int64_t(rows_r.size()), NC = int64_t(rows_c.size());
    if (NR < 1 || NC < 1 || NR > 160 || NC > 160) return false;
    const int LDC = round_up(int(NC), 32) + 8;
    // one allocation: rowR | rowC | rhoR | rhoC (int32), then the piece table (8 x uint16 per piece, 16-byte aligned)
    const size_t n_int = size_t(NR + NC + 2 * P);
    const size_t tab_off = (n_int * 4 + 15) & ~size_t(15);
    std::vector<unsigned char> host(tab_off + size_t(pieces) * 16);
    int32_t* ints = reinterpret_cast<int32_t*>(host.data());
    for (int64_t r = 0; r < NR; ++r) ints[r] = int32_t(rows_r[size_t(r)]);
    for (int64_t c = 0; c < NC; ++c) ints[NR + c] = int32_t(rows_c[size_t(c)]);
    for (int64_t rho = 0; rho < P; ++rho) {
        const int64_t m = w == 0 ? gen_offset(g.sc, rho) : gen_offset(g.sk, rho);
        ints[NR + NC + rho] = int32_t(cols_from_q ? m / merged_C : m % merged_C);
        ints[NR + NC + P + rho] = int32_t(cols_from_q ? m % merged_C : m / merged_C);
    }
    uint16_t* tab = reinterpret_cast<uint16_t*>(host.data() + tab_off);
    for (size_t i = 0; i < elems.size(); ++i) {
        if (elems[i].rP < 0) {
            tab[i] = 0xFFFF;
            continue;
        }
        const int64_t vr = cols_from_q ? elems[i].rP : elems[i].rQ, vc = cols_from_q ? elems[i].rQ : elems[i].rP;
        const int64_t r = std::lower_bound(rows_r.begin(), rows_r.end(), vr) - rows_r.begin();
        const int64_t c = std::lower_bound(rows_c.begin(), rows_c.end(), vc) - rows_c.begin();
        tab[i] = uint16_t(r * LDC + c);
    }
    // are the pieces runs of consecutive columns? (first slice: 8 in a row; second: two runs of 4); a run is
    // either wholly inside the tensor or wholly outside, and starts at a multiple of its length
    const int run = w == 0 ? 8 : 4;
    bool contig = true;
    for (size_t i = 0; i < elems.size() && contig; i += size_t(run)) {
        const bool out0 = tab[i] == 0xFFFF;
        for (int e = 0; e < run && contig; ++e) {
            if ((tab[i + e] == 0xFFFF) != out0) contig = false;
            else if (!out0 && (tab[i + e] != tab[i] + e || tab[i] % run)) contig = false;
        }
    }
    if (hipMalloc(&h->lazy_gen_tables[w], host.size()) != hipSuccess) return false;
    if (hipMemcpyAsync(h->lazy_gen_tables[w], host.data(), host.size(), hipMemcpyHostToDevice, st) != hipSuccess ||
        hipStreamSynchronize(st) != hipSuccess)
        return false;
    h->packed_bytes += int64_t(host.size());
    KronGenMfmaArgs& a = h->lazy_gen_mfma[w];
    memset(&a, 0, sizeof(a));
    a.Rc = cols_from_q ? g.Pc : g.Qc;
    a.Cc = cols_from_q ? g.Qc : g.Pc;
    const int32_t* dints = static_cast<const int32_t*>(h->lazy_gen_tables[w]);
    a.rowR = dints;
    a.rowC = dints + NR;
    a.rhoR = dints + NR + NC;
    a.rhoC = dints + NR + NC + P;
    a.tab = static_cast<const unsigned char*>(h->lazy_gen_tables[w]) + tab_off;
    a.NR = int32_t(NR);
    a.NC = int32_t(NC);
    a.LDC = LDC;
    a.Sp = g.Sp;
    a.pieces_per_rho = int32_t(pieces);
    a.pieces_per_chunk = int32_t(pieces / (w == 0 ? g.n_chunks : 1));
    a.P = int32_t(P);
    a.contig = contig ? (w == 0 ? 1 : 2) : 0;
    h->lazy_gen_smem[w] = size_t(NR) * LDC * 2;
    h->lazy_mfma[w] = true;
    return true;
}

// The kernels may number k and a in any order as long as x is gathered through the same numbering. Pick the one that
// makes an index of extent % unit == 0 the fastest-running digit (it is then a run of consecutive columns of the
// product matrix the slices are assembled from): returns new number -> the plan's number.
std::vector<int32_t> minor_digit_permutation(const std::vector<int64_t>& extents, int unit) {
    int64_t total = 1;
    for (int64_t e : extents) total *= e;
    std::vector<int32_t> perm(static_cast<size_t>(total));
    for (int64_t i = 0; i < total; ++i) perm[size_t(i)] = int32_t(i);
    const int n = int(extents.size());
    if (n < 2 || extents[size_t(n - 1)] % unit == 0) return perm;      // already so (or nothing to choose)
    int pick = -1;
    for (int j = 0; j < n; ++j)
        if (extents[size_t(j)] % unit == 0 && (pick < 0 || extents[size_t(j)] > extents[size_t(pick)])) pick = j;
    if (pick < 0) return perm;
    std::vector<int> order;                 // digits of the new number, outer -> inner
    for (int j = 0; j < n; ++j)
        if (j != pick) order.push_back(j);
    order.push_back(pick);
    std::vector<int64_t> weight(size_t(n), 1);      // of each digit in the plan's number
    for (int j = n - 2; j >= 0; --j) weight[size_t(j)] = weight[size_t(j + 1)] * extents[size_t(j + 1)];
    for (int64_t i = 0; i < total; ++i) {
        int64_t rem = i, orig = 0;
        for (int q = n - 1; q >= 0; --q) {
            const int j = order[size_t(q)];
            orig += (rem % extents[size_t(j)]) * weight[size_t(j)];
            rem /= extents[size_t(j)];
        }
        perm[size_t(i)] = int32_t(orig);
    }
    return perm;
}

int launch_kron_lazy(const tn_linear_s* h, const Workspace& w, const void* x, void* y, int64_t tokens, hipStream_t st) {
    KronSetup k{&h->lazy_dims, h->lazy_slices, static_cast<const char*>(h->lazy_slices) + h->lazy_h1_offset,
                h->lazy_xrow, h->lazy_xcol, h->lazy_yrow, h->lazy_ycol};
    return launch_kron(h, w, k, x, y, tokens, st);
}

template <int CFG, int SS>
int direct_entry(const KronDirectArgs* p, uint32_t grid, hipStream_t st) {
    constexpr size_t smem = KronDirectShape<CFG, SS>::SMEM;
    if (!p)         // configuration call (create time)
        return hipFuncSetAttribute(reinterpret_cast<const void*>(step_krondirect_kernel<CFG, SS>), hipFuncAttributeMaxDynamicSharedMemorySize,
                                   int(smem)) == hipSuccess
                   ? TN_OK
                   : TN_ERR_HIP;
    hipLaunchKernelGGL((step_krondirect_kernel<CFG, SS>), dim3(grid), dim3(256), smem, st, *p);
    return TN_OK;
}

template <int CFG>
int direct_of(int steps, const KronDirectArgs* p, uint32_t grid, hipStream_t st) {
    static_assert(tn::kDirectMaxSteps == 3, "one case per number of steps");
    switch (steps) {
        case 1: return direct_entry<CFG, 1>(p, grid, st);
        case 2: return direct_entry<CFG, 2>(p, grid, st);
        case 3: return direct_entry<CFG, 3>(p, grid, st);
        default: return TN_ERR_INVALID_ARG;
    }
}

int direct_dispatch(int cfg, int steps, const KronDirectArgs* p, uint32_t grid, hipStream_t st) {
    static_assert(tn::kDirectConfigs == 5, "one case per instantiation");
    switch (cfg) {
        case 0: return direct_of<0>(steps, p, grid, st);
        case 1: return direct_of<1>(steps, p, grid, st);
        case 2: return direct_of<2>(steps, p, grid, st);
        case 3: return direct_of<3>(steps, p, grid, st);
        case 4: return direct_of<4>(steps, p, grid, st);
        default: return TN_ERR_INVALID_ARG;
    }
}

// Sums a split of a token leaves: whole tiles of the output.
int64_t direct_sums(const tn_linear_s* h) {
    return int64_t((h->direct_args.O1 + 15) / 16) * ((h->direct_args.C1 + 15) / 16) * 256;
}

// Blocks of the bond for the workgroups of a call, one to a compute unit, of the least time: the launches, a value of the bond
// (0.2 us, 0.5 with the resident cores in LDS, and 12 ns per MFMA of a wave), a turn of the resident cores (in LDS, longer the more steps
// they have, the first of them above all), and the partial sums written and read. Expected / measured, us: rings of one token 5120 -> 8192
// rank 96 57 / 56, rank 32 17 / 16; 5120 -> 25600 rank 96 108 / 104 to 116, rank 32 30 / 31; 25600 -> 5120 rank 96 104 / 110 to 116;
// 5120 -> 1024 rank 96 32 / 28; of two tokens 5120 -> 8192 rank 96 98 / 90; trains 25600 -> 5120 rank 96 at 1, 6, 12 and 16 tokens 17.5 / 17.4,
// 26.7 / 26.4, 35.4 / 35.1, 39.6 / 39.7 (28.2 and 31.7 for the last two, were a turn the same everywhere), rank 64 at 12 26.3 / 25.9.
DirectGeom direct_geometry(const tn_linear_s* h, int64_t tokens, int64_t partial_cap) {
    const KronDirectArgs& a = h->direct_args;
    const int* g = tn::kDirectConfig[h->direct_cfg];
    const int mfmas = h->direct_steps * (g[6] * g[7] + g[9] * g[10]) + g[2] * (g[0] * g[1] + g[3] * ((g[0] + 1) / 2));
    const float per_value = (g[12] ? 0.5f : 0.2f) + float(mfmas) * 0.0123f;
    const float more = g[12] ? float(h->direct_steps - 1) : 0.f, first = 9.f + 1.7f * more, per_turn = 1.f + 0.375f * more;
    const int64_t slots = std::max<int64_t>(1, h->num_cus / tokens);
    DirectGeom best;
    best.us = std::numeric_limits<float>::max();
    for (int str_per = 1; str_per <= a.n_str; ++str_per) {
        const int str_blocks = (a.n_str + str_per - 1) / str_per;
        if ((a.n_str + str_blocks - 1) / str_blocks != str_per) continue;        // as many blocks with fewer values each
        for (int64_t want = std::max<int64_t>(1, slots / str_blocks); want >= 1; want /= 2) {
            const int64_t blocks = std::min<int64_t>(want, a.n_res);
            DirectGeom c;
            c.str_per = str_per;
            c.str_blocks = str_blocks;
            c.res_per = int((a.n_res + blocks - 1) / blocks);
            c.n_splits = (a.n_res + c.res_per - 1) / c.res_per * str_blocks;
            c.partial_bytes = c.n_splits > 1 ? int64_t(c.n_splits) * tokens * direct_sums(h) * 4 : 0;
            const int64_t rounds = (tokens * c.n_splits + h->num_cus - 1) / h->num_cus;
            c.us = first + float(rounds) * float(c.res_per) * (per_turn + float(str_per) * per_value) + float(c.partial_bytes) / 2e6f;
            if (c.partial_bytes <= partial_cap && c.us < best.us) best = c;
        }
    }
    return best;
}

// The calls that take it, against the slices in memory (of a layer that shares its workspace: written by every call: two launches, 3.4 TB/s). us per
// call, made on chip / in memory, shared workspace, then a workspace of its own: rings 5120 -> 8192 of rank 96 at one token 56 / 179, 50 / 95, at 2
// 86 / 180, 86 / 97, at 4 157 / 185, 157 / 100; of rank 32 16 / 50, 16 / 30, at 4 25 / 50, 25 / 36; 5120 -> 25600 of rank 64 at one 56 / 144,
// 52 / 102; 25600 -> 5120 of rank 96 109 / 294, 102 / 177; 5120 -> 1024 of rank 96 29 / 61, 26 / 32, at 2 43 / 61, 43 / 32; trains 25600 ->
// 5120 of rank 96 at one 18 / 33, 17 / 24, at 4 23 / 35, 22 / 26.
void price_direct(tn_linear_s* h) {
    for (int64_t t = 1; h->direct && t <= std::min(h->max_tokens, kDirectMaxTokens); ++t) {
        DirectGeom g = direct_geometry(h, t, h->partial ? h->partial_bytes : 0);
        const float slices = h->lazy_slices_kept ? 0.f : 8.f + float(h->lazy_slice_bytes) / 3.4e6f;
        const KronGeom k = kron_geometry(h, h->lazy_dims, t, h->partial ? h->partial_bytes : 0);
        // one workgroup walks the bond, one token: its four waves share a value there (rank-96 ring 25600 -> 5120 on chip 19.9 ms, from memory
        // 16.0, from 2 tokens on 20.0 and 31.7; rank-96 train 562 us and 167)
        g.taken = g.us < kron_us(h, h->lazy_dims, k) * (k.share && k.n_splits == 1 ? 0.5f : 1.f) + slices;
        h->direct_geom[t] = g;
    }
}

int launch_direct(const tn_linear_s* h, const Workspace& w, const DirectGeom& g, const void* x, void* y, int64_t tokens, hipStream_t st) {
    KronDirectArgs p = h->direct_args;
    p.X = x;
    p.Y = g.n_splits > 1 ? w.partial : y;
    p.tokens = int32_t(tokens);
    p.res_per = g.res_per;
    p.str_per = g.str_per;
    p.str_blocks = g.str_blocks;
    p.n_splits = g.n_splits;
    if (g.partial_bytes > (w.partial ? w.partial_bytes : 0)) return TN_ERR_UNSUPPORTED;      // never write past the buffer
    const int rc = direct_dispatch(h->direct_cfg, h->direct_steps, &p, uint32_t(tokens * g.n_splits), st);
    if (rc != TN_OK) return rc;
    if (g.n_splits > 1) {
        p.Y = y;
        hipLaunchKernelGGL(krondirect_reduce_kernel, dim3(uint32_t(tokens * direct_sums(h) / 64)), dim3(256), 0, st, p,
                           static_cast<const float*>(w.partial));
    }
    return hipGetLastError() == hipSuccess ? TN_OK : TN_ERR_HIP;
}

// Token count from which a lazily merged plan replaces the compact steps: every call. With the one-token form of
// the Kronecker-sum kernel (four waves share the token) rebuilding the slices and streaming them once is as fast as
// the compact steps or faster on every ring class of the 64-layer stack (us per one-token call, rebuilt / compact:
// 25600->5120 r32 49/69, r96 326/527; 5120->25600 r64 246/246; 5120->8192 r96 253/262; 8192->5120 r64 118/130;
// 5120->1024 r96 97/163, r32 24/46).
constexpr int64_t kLazyMinTokens = 1;

void fill_gen_dims(GenDims* g, const std::vector<tn::GatherDim>& d) {
    g->n = int32_t(d.size());
    for (size_t j = 0; j < d.size(); ++j) {
        g->ext[j] = int32_t(d[j].extent);
        g->str[j] = d[j].stride;
    }
}

// Tables to the GPU without waiting for them: the host copy stays with the handle until create's last wait.
int upload_tables(tn_linear_s* h, std::vector<int32_t>&& tab, void* dst, hipStream_t st) {
    h->create_tables.push_back(std::move(tab));
    const std::vector<int32_t>& t = h->create_tables.back();
    return hipMemcpyAsync(dst, t.data(), t.size() * sizeof(int32_t), hipMemcpyHostToDevice, st) == hipSuccess ? TN_OK : TN_ERR_HIP;
}

bool matrix_plan_of(tn_linear_s* h, const tn_linear_desc* desc) {
    tn_linear_s::MatrixPlans& p = h->matrix_plans;
    if (!p.tried) p.ok = tn::make_matrix_plan(desc, &p.net, &p.m);
    p.tried = true;
    return p.ok;
}

// An operand kept for the products: allocated, freed with the handle, written by the next write_operands.
int keep_operand(tn_linear_s* h, const tn_linear_desc* desc, const tn::SourceOp& o, int64_t Kp, bool packed, void** out,
                 std::vector<void*>* owner = nullptr) {
    SourceArgs a;
    memset(&a, 0, sizeof(a));
    a.R = o.R;
    a.K = o.K;
    a.Rp = packed ? (o.R + tn::kMatrixColPad - 1) / tn::kMatrixColPad * tn::kMatrixColPad : o.R;
    a.Kp = Kp;
    a.packed = packed ? 1 : 0;
    a.nr = int32_t(o.rows.size());
    a.nk = int32_t(o.ks.size());
    for (size_t j = 0; j < o.rows.size(); ++j) {
        a.rext[j] = int32_t(o.rows[j].extent);
        a.rlim[j] = int32_t(o.rows[j].limit);
        a.rstr[j] = o.rows[j].stride;
    }
    for (size_t j = 0; j < o.ks.size(); ++j) {
        a.kext[j] = int32_t(o.ks[j].extent);
        a.klim[j] = int32_t(o.ks[j].limit);
        a.kstr[j] = o.ks[j].stride;
    }
    const int64_t n = a.Rp * a.Kp;
    void* dst = nullptr;
    if (hipMalloc(&dst, size_t(n) * sizeof(bf16_t)) != hipSuccess) return TN_ERR_ALLOC;
    (owner ? owner : &h->mat_kept)->push_back(dst);
    h->packed_bytes += n * int64_t(sizeof(bf16_t));
    a.src = static_cast<const bf16_t*>(desc->tensors[o.slot]);
    a.dst = static_cast<bf16_t*>(dst);
    h->create_sources.push_back(a);
    *out = dst;
    return TN_OK;
}

// The operands asked for since the last time, on `st`.
int write_operands(tn_linear_s* h, hipStream_t st) {
    for (size_t i = 0; i < h->create_sources.size(); i += kSourceMany) {
        const size_t n = std::min<size_t>(kSourceMany, h->create_sources.size() - i);
        SourceMany m;
        memset(&m, 0, sizeof(m));
        int64_t most = 0;
        for (size_t j = 0; j < n; ++j) {
            m.s[j] = h->create_sources[i + j];
            most = std::max(most, m.s[j].Rp * m.s[j].Kp);
        }
        hipLaunchKernelGGL(operand_source_kernel, dim3(uint32_t(std::min<int64_t>((most + 255) / 256, 65536)), uint32_t(n)), dim3(256), 0, st, m);
    }
    h->create_sources.clear();
    return hipGetLastError() == hipSuccess ? TN_OK : TN_ERR_HIP;
}

void fill_product_step(DevStep* s, const tn::Product& p) {
    s->plan.R = p.R;
    s->plan.K = p.Kp;
    s->plan.C = p.C;
    s->plan.c_tok_stride = p.out_elems;
    s->variant = VAR_GEMM;
    s->cmode = 1;
    s->Kp = int(p.Kp);
    s->Cp = round_up(int(p.C), tn::kMatrixColPad);
}

// Decide whether the layer gets a lazily merged plan, and prepare it: the plan TN_FLAG_MERGE_GROW would give
// must be two steps the Kronecker-sum kernel takes (large intermediate, little padding), each absorbing a
// tensor merged from two of the caller's, and cheaper than the compact plan. Nothing of that plan is stored
// except copies of the caller's tensors involved and four offset tables.
int prepare_lazy(tn_linear_s* h, const tn_linear_desc* desc, hipStream_t st) {
    if (h->plan.dtype != TN_DTYPE_BF16 || h->pair || h->kron || h->small_chain) return TN_OK;
    if (desc->flags & (TN_FLAG_NO_PAIR_CHAIN | TN_FLAG_SCALAR_KERNELS | TN_FLAG_NO_MERGE | TN_FLAG_MERGE_GROW |
                       TN_FLAG_MERGE_HALVES | TN_FLAG_NO_LAZY_MERGE | TN_FLAG_TRAINABLE))
        return TN_OK;
    if (((desc->flags >> TN_FLAG_VARIANT_SHIFT) & 0xff) != 0) return TN_OK;      // tuning overrides: keep what they ask
    if (desc->max_tokens < kLazyMinTokens) return TN_OK;
    tn_linear_desc grow = *desc;
    grow.flags |= TN_FLAG_MERGE_HALVES;
    tn::Plan& q = h->lazy_plan;
    if (tn::make_plan(&grow, &q) != TN_OK || q.steps.size() != 2 || q.merges.size() != 2 || q.flops >= h->plan.flops)
        return TN_OK;
    tn::KronDims d;
    if (!tn::kron_shape(q, &d)) return TN_OK;
    const tn::MergeOp* mo[2];
    for (int w = 0; w < 2; ++w) {
        int mi = q.steps[size_t(w)].slot - q.n_caller_tensors;
        if (mi < 0 || mi >= 2) return TN_OK;
        mo[w] = &q.merges[size_t(mi)];
        if (mo[w]->p_slot >= q.n_caller_tensors || mo[w]->q_slot >= q.n_caller_tensors) return TN_OK;
        if (mo[w]->kp.empty() || q.steps[size_t(w)].trace_extent != 1) return TN_OK;
    }
    KronTiles kt;
    if (kron_dispatch(d.cfg, nullptr, 0, nullptr, &kt) != TN_OK) return TN_OK;
    const int at = kt.at, ks0 = kt.ks0, o2t = kt.o2t, o1t = kt.o1t;
    tn::Plan net;
    tn::SlicePlan sp;
    if (!(desc->flags & TN_FLAG_SCALAR_GENERATE) && tn::build_network(desc, &net) == TN_OK && tn::make_slice_plan(net, q, d, &sp)) {
        std::vector<int32_t> tab;
        size_t at[8];
        const std::vector<int32_t>* all[8] = {&sp.xrow, &sp.xcol, &sp.yrow, &sp.ycol, &sp.half[0].row_off, &sp.half[0].col_off,
                                              &sp.half[1].row_off, &sp.half[1].col_off};
        for (int i = 0; i < 8; ++i) {
            at[i] = tab.size();
            tab.insert(tab.end(), all[i]->begin(), all[i]->end());
        }
        if (hipMalloc(reinterpret_cast<void**>(&h->lazy_tables), tab.size() * sizeof(int32_t)) != hipSuccess) return TN_ERR_ALLOC;
        if (hipMemcpyAsync(h->lazy_tables, tab.data(), tab.size() * sizeof(int32_t), hipMemcpyHostToDevice, st) != hipSuccess ||
            hipStreamSynchronize(st) != hipSuccess)
            return TN_ERR_HIP;
        h->lazy_xrow = h->lazy_tables + at[0];
        h->lazy_xcol = h->lazy_tables + at[1];
        h->lazy_yrow = h->lazy_tables + at[2];
        h->lazy_ycol = h->lazy_tables + at[3];
        for (int w = 0; w < 2; ++w) {
            DevProduct& p = h->lazy_half[w];
            fill_product_step(&p.s, sp.half[w]);
            p.s.crow = h->lazy_tables + at[4 + 2 * w];
            p.s.ccol = h->lazy_tables + at[5 + 2 * w];
            void* a = nullptr;
            int rc = keep_operand(h, desc, sp.half[w].a, sp.half[w].Kp, false, &a, &h->lazy_sources);
            p.a = a;
            if (rc == TN_OK) rc = keep_operand(h, desc, sp.half[w].b, sp.half[w].Kp, true, &p.s.packed, &h->lazy_sources);
            if (rc != TN_OK) return rc;
        }
        d.x_vec8 = sp.x_vec8;
        h->lazy_h1_offset = sp.h1_offset;
        h->lazy_slice_bytes = sp.bytes;
        h->lazy_products = true;
        h->lazy = true;
        h->lazy_dims = d;
        h->lazy_min_tokens = kLazyMinTokens;
        return TN_OK;
    }
    // the four source matrices (shared indices innermost), written from the caller's tensors
    const int32_t sp_len[2] = {round_up(int(mo[0]->K), 16), round_up(int(mo[1]->K), 16)};
    for (int w = 0; w < 2; ++w)
        for (int side = 0; side < 2; ++side) {
            const int64_t rows = side == 0 ? mo[w]->R : mo[w]->C;
            const int64_t n = rows * sp_len[w];
            void* buf = nullptr;
            if (hipMalloc(&buf, size_t(n) * sizeof(bf16_t)) != hipSuccess) return TN_ERR_ALLOC;
            h->lazy_sources.push_back(buf);
            h->packed_bytes += n * int64_t(sizeof(bf16_t));
            GenDims fd, sd;
            memset(&fd, 0, sizeof(fd));
            memset(&sd, 0, sizeof(sd));
            fill_gen_dims(&fd, side == 0 ? mo[w]->rdims : mo[w]->cdims);
            fill_gen_dims(&sd, side == 0 ? mo[w]->kp : mo[w]->kq);
            hipLaunchKernelGGL(kron_source_kernel, dim3(uint32_t(std::min<int64_t>((n + 255) / 256, 65536))), dim3(256), 0, st,
                               static_cast<const bf16_t*>(desc->tensors[side == 0 ? mo[w]->p_slot : mo[w]->q_slot]),
                               static_cast<bf16_t*>(buf), fd, sd, rows, int32_t(mo[w]->K), sp_len[w]);
        }
    if (hipGetLastError() != hipSuccess) return TN_ERR_HIP;
    const tn::Step& s0 = q.steps[0];
    const tn::Step& s1 = q.steps[1];
    const int n_chunks = int((d.O1 + 32 * o1t - 1) / (32 * o1t));
    const int64_t e0 = int64_t(n_chunks) * d.P * o1t * ks0 * 512;
    const int64_t e1 = d.P * int64_t(o2t) * 2 * at * 512;
    h->lazy_h1_offset = (e0 * 2 + 255) & ~int64_t(255);
    h->lazy_slice_bytes = h->lazy_h1_offset + ((e1 * 2 + 255) & ~int64_t(255));
    for (int w = 0; w < 2; ++w) {
        KronGenArgs& g = h->lazy_gen[w];
        memset(&g, 0, sizeof(g));
        const tn::Step& sp = q.steps[size_t(w)];
        g.Pc = h->lazy_sources[size_t(2 * w)];
        g.Qc = h->lazy_sources[size_t(2 * w + 1)];
        fill_gen_dims(&g.sc, sp.cdims);
        fill_gen_dims(&g.sk, sp.kdims);
        g.merged_C = mo[w]->C;
        g.Sp = sp_len[w];
        g.which = w;
        g.n_chunks = n_chunks;
        g.P = int32_t(d.P);
        g.KS0 = ks0;
        g.O1T = o1t;
        g.O1 = int32_t(d.O1);
        g.K0 = int32_t(d.K0);
        g.O2T = o2t;
        g.AT = at;
        g.C1 = int32_t(d.C1);
        g.A = int32_t(d.A);
    }
    // The MFMA form of the rebuild, with k and a numbered so that the pieces of the slices are runs of columns of
    // the products; if a half does not fit that form, both keep the plan's numbering (the plain-FMA kernel knows no
    // other) and the halves that fit still use MFMA.
    std::vector<int32_t> perm_k(size_t(d.K0)), perm_a(size_t(d.A));
    for (int64_t i = 0; i < d.K0; ++i) perm_k[size_t(i)] = int32_t(i);
    for (int64_t i = 0; i < d.A; ++i) perm_a[size_t(i)] = int32_t(i);
    if (!(desc->flags & TN_FLAG_SCALAR_GENERATE)) {
        std::vector<int64_t> kext;
        for (const tn::GatherDim& gd : s0.kdims) kext.push_back(gd.extent);
        const std::vector<int32_t> pk = minor_digit_permutation(kext, 8), pa = minor_digit_permutation(s0.rext, 4);
        const bool ok = int64_t(pk.size()) == d.K0 && int64_t(pa.size()) == d.A &&
                        prepare_gen_mfma(h, 0, h->lazy_gen[0], d, mo[0]->C, pk, st) &&
                        prepare_gen_mfma(h, 1, h->lazy_gen[1], d, mo[1]->C, pa, st);
        if (ok) {
            perm_k = pk;
            perm_a = pa;
        } else {
            for (int w = 0; w < 2; ++w) {
                if (h->lazy_gen_tables[w]) (void)hipFree(h->lazy_gen_tables[w]);
                h->lazy_gen_tables[w] = nullptr;
                h->lazy_mfma[w] = false;
            }
            (void)prepare_gen_mfma(h, 0, h->lazy_gen[0], d, mo[0]->C, perm_k, st);
            (void)prepare_gen_mfma(h, 1, h->lazy_gen[1], d, mo[1]->C, perm_a, st);
        }
    }
    // tables of the merged plan: where a and k (in the kernels' numbering) sit in a token of x, where o1 and o2 go
    std::vector<int32_t> tab;
    bool identity = s0.a_plain;
    for (int64_t i = 0; i < d.K0 && identity; ++i) identity = perm_k[size_t(i)] == i;
    for (int64_t i = 0; i < d.A && identity; ++i) identity = perm_a[size_t(i)] == i;
    const size_t n_xrow = identity ? 0 : size_t(d.A), n_xcol = identity ? 0 : size_t(d.K0);
    if (!identity) {
        for (int64_t a = 0; a < d.A; ++a)
            tab.push_back(s0.a_plain ? int32_t(perm_a[size_t(a)] * d.K0) : s0.arow[size_t(perm_a[size_t(a)])]);
        for (int64_t k = 0; k < d.K0; ++k)
            tab.push_back(s0.a_plain ? perm_k[size_t(k)] : s0.acol[size_t(perm_k[size_t(k)])]);
        // 8 consecutive k of one a as one aligned 16-byte piece of x?
        d.x_vec8 = true;
        for (int64_t a = 0; a < d.A; ++a)
            if (tab[size_t(a)] % 8) d.x_vec8 = false;
        for (int64_t k = 0; k < d.K0; ++k) {
            const int32_t v = tab[size_t(d.A + k)], v0 = tab[size_t(d.A + (k & ~int64_t(7)))];
            if (v != v0 + (k & 7) || (!(k & 7) && v % 8)) d.x_vec8 = false;
        }
    }
    tab.insert(tab.end(), s1.crow.begin(), s1.crow.end());
    tab.insert(tab.end(), s1.ccol.begin(), s1.ccol.end());
    if (hipMalloc(reinterpret_cast<void**>(&h->lazy_tables), tab.size() * sizeof(int32_t)) != hipSuccess) return TN_ERR_ALLOC;
    if (hipMemcpyAsync(h->lazy_tables, tab.data(), tab.size() * sizeof(int32_t), hipMemcpyHostToDevice, st) != hipSuccess ||
        hipStreamSynchronize(st) != hipSuccess)
        return TN_ERR_HIP;
    if (!identity) {
        h->lazy_xrow = h->lazy_tables;
        h->lazy_xcol = h->lazy_tables + n_xrow;
    }
    h->lazy_yrow = h->lazy_tables + n_xrow + n_xcol;
    h->lazy_ycol = h->lazy_yrow + s1.crow.size();
    h->lazy = true;
    h->lazy_dims = d;
    h->lazy_min_tokens = kLazyMinTokens;
    return TN_OK;
}

// A lazily merged layer: the plan with the slices made on chip, where an instantiation holds its shape.
int prepare_direct(tn_linear_s* h, const tn_linear_desc* desc, hipStream_t st) {
    if (!h->lazy || (desc->flags & (TN_FLAG_NO_DECODE_FUSION | TN_FLAG_SCALAR_GENERATE))) return TN_OK;
    tn::Plan net;
    tn::DirectPlan d;
    int tensors[2][2];
    if (tn::build_network(desc, &net) != TN_OK || !tn::merged_tensors(net, h->lazy_plan, tensors) || !tn::make_direct_plan(net, tensors, &d)) return TN_OK;
    KronDirectArgs& a = h->direct_args;
    memset(&a, 0, sizeof(a));
    for (int w = 0; w < 2; ++w)
        for (int side = 0; side < 2; ++side) {
            void* p = nullptr;
            const int rc = keep_operand(h, desc, d.src[w][side], 32 * d.steps, true, &p, &h->lazy_sources);
            if (rc != TN_OK) return rc;
            a.src[w][side] = p;
            a.tiles[w][side] = int32_t(d.tiles[w][side]);
        }
    std::vector<int32_t> tab;
    size_t at[6];
    const std::vector<int32_t>* all[4] = {&d.xrow, &d.xcol, &d.yrow, &d.ycol};
    for (int i = 0; i < 4; ++i) {
        at[i] = tab.size();
        tab.insert(tab.end(), all[i]->begin(), all[i]->end());
    }
    for (int w = 0; w < 2; ++w) {
        at[4 + w] = tab.size();
        tab.resize(tab.size() + (d.unit[w].size() + 1) / 2);
        memcpy(&tab[at[4 + w]], d.unit[w].data(), d.unit[w].size() * sizeof(uint16_t));
    }
    void* mem = nullptr;
    if (hipMalloc(&mem, tab.size() * sizeof(int32_t)) != hipSuccess) return TN_ERR_ALLOC;
    h->lazy_sources.push_back(mem);
    h->packed_bytes += int64_t(tab.size() * sizeof(int32_t));
    const int32_t* dev = static_cast<const int32_t*>(mem);
    a.xrow = dev + at[0];
    a.xcol = dev + at[1];
    a.yrow = dev + at[2];
    a.ycol = dev + at[3];
    a.unit[0] = reinterpret_cast<const uint16_t*>(dev + at[4]);
    a.unit[1] = reinterpret_cast<const uint16_t*>(dev + at[5]);
    a.N = h->plan.N;
    a.M = h->plan.M;
    a.A = int32_t(d.A);
    a.K0 = int32_t(d.K0);
    a.O1 = int32_t(d.O1);
    a.C1 = int32_t(d.C1);
    a.n_res = int32_t(d.n_res);
    a.n_str = int32_t(d.n_str);
    a.x_vec8 = d.x_vec8 ? 1 : 0;
    h->direct_cfg = d.cfg;
    h->direct_steps = d.steps;
    h->direct = true;
    return upload_tables(h, std::move(tab), mem, st);
}

// What one launch of a product takes, in us: its tiles, or the stores of its output (W of 10240 x 4096 in 22 us, 84 MB; in two parts 3.5 TB/s).
// Without the form for short K, which W's product of a narrow bond runs on, W was priced 7 us too high. The price of a tile has 3 us of a
// launch in it, 3 more are what a launch costs a program that does not replay a graph. With 5, two products of 3.2 and 4.4 us of a train of two
// cores (40 x 8, 32 x 16, rank 24) were left for steps that take 12.6 to 15.2 at 33 to 500 tokens, 8.7 to 8.9 so.
constexpr float kGemmStoreBytesPerUs = 4e6f;
float product_us(const tn_linear_s* h, const DevStep& s) {
    const bool plain = !s.a_lo && !s.b_lo && !s.out_lo;
    return kGemmLaunchUs + std::max(gemm_choice(h, s, s.plan.R, 0, plain).us, float(s.plan.R) * float(s.plan.C) * (plain ? 2.f / kGemmStoreBytesPerUs : 4.f / 3.5e6f));
}

constexpr int64_t kMatrixNoEnd = std::numeric_limits<int64_t>::max();

// Does a call of so many tokens contract the tensors with each other first?
bool takes_matrix(const tn_linear_s* h, int64_t tokens) {
    if (!h->matrix) return false;
    for (const auto& r : h->mat_ranges)
        if (tokens >= r.first && tokens < r.second) return true;
    return false;
}

// Decide whether calls of many tokens contract the tensors with each other first, from how many tokens on, and prepare it.
// The other orders are priced at the rates their kernels reach at many tokens (FLOP per us: chained pair kernel 1.3e9, one
// launch per step 0.45e9; the Kronecker-sum kernel by kron_us). Measured, us per call in this order / in the other: ring
// 25600 -> 5120 of rank 32 343 / 410 at 96 tokens, 767 / 8109 at 2048, 1955 / 30730 at 8192; ring 5120 -> 8192 of rank 96 776 /
// 911 at 48 tokens, 885 / 35579 at 2048; train 5120 -> 25600 of rank 96 226 / 207 at 387 tokens, 226 / 391 at 420; train 5120 -> 8192 of rank 64 106 / 184 at 1138 tokens, 143 / 199 at
// 2048, 488 / 792 at 8192; of rank 32, whose chain has little more than 2 M N, 100 / 81 at 1000, 99 / 145 at 1025, 145 / 154 at 2048.
// Of 500 such pairs (trains and rings of ranks 32 to 96, five projections, 16 to 8192 tokens) this order is never taken where it is more than 6 %
// slower; it is left where it is up to 1.8 times as fast (train 5120 -> 8192 of rank 64, 103 / 181 at 1060 tokens): the chained pair kernel is priced
// by the token, while it takes rounds of workgroups.
int prepare_matrix(tn_linear_s* h, const tn_linear_desc* desc, hipStream_t st) {
    if (h->plan.dtype != TN_DTYPE_BF16 ||
        (desc->flags & (TN_FLAG_NO_PAIR_CHAIN | TN_FLAG_SCALAR_KERNELS | TN_FLAG_NO_MERGE | TN_FLAG_NO_LAZY_MERGE)) ||
        ((desc->flags >> TN_FLAG_VARIANT_SHIFT) & 0xff) != 0)
        return TN_OK;
    // W takes at least the time to write it: where the product alone is no faster than what there is, no plan is made
    DevStep& y = h->mat_y;
    y.plan.R = 1;
    y.plan.K = h->plan.N;
    y.plan.C = h->plan.M;
    y.plan.a_tok_stride = h->plan.N;
    y.plan.c_tok_stride = h->plan.M;
    y.variant = VAR_GEMM;
    y.cmode = 1;
    y.Kp = int(h->plan.N);
    y.Cp = round_up(int(h->plan.M), tn::kMatrixColPad);
    if (h->plan.N % 64 || h->plan.format == TN_FORMAT_DENSE || h->plan.format == TN_FORMAT_TUCKER || !gemm_fits(y)) return TN_OK;
    auto other_us = [&](int64_t t) {
        if (h->pair) return std::max(12.f, float(t) * float(h->plan.flops) / 1.3e9f);
        if (h->kron) return kron_us(h, h->kron_dims, kron_geometry(h, h->kron_dims, t, kMaxPartialBytes));
        if (h->lazy) return kron_us(h, h->lazy_dims, kron_geometry(h, h->lazy_dims, t, kMaxPartialBytes)) + (desc->workspace ? float(h->lazy_slice_bytes) / 1.6e6f : 0.f);
        return 6.f * float(h->steps.size()) + float(t) * float(h->plan.flops) / 0.45e9f;
    };
    // Token counts [first, end) for which this order is taken: from where it is clearly the cheaper one to where it no longer is.
    // There may be several such ranges: the prices are staircases, in row tiles here and in rounds of workgroups of the Kronecker-sum kernel.
    // They are looked for on a grid of counts and their ends between its points: with the ends on the grid, a train 5120 -> 8192 of rank 64
    // took this order at 1260 tokens and not at 1259 or 1261.
    auto ranges = [&](float build_us, bool any = false) {      // any: whether there are, the first point is enough
        std::vector<std::pair<int64_t, int64_t>> r;
        auto changes = [&](int64_t t, bool in) {
            const float us = build_us + gemm_choice(h, y, t, kMaxPartialBytes).us, other = other_us(t);
            return in ? us >= other : 1.04f * us < other;
        };
        bool in = false;
        int64_t last = 7;
        for (int64_t t = 8; t <= desc->max_tokens; last = t, t += t < 64 ? 8 : t / 16) {
            if (!changes(t, in)) continue;
            if (any) return std::vector<std::pair<int64_t, int64_t>>{{t, kMatrixNoEnd}};
            int64_t at = t;                        // the first count of this interval that does, not the grid's
            for (int64_t lo = last; at - lo > 1;) {
                const int64_t mid = lo + (at - lo) / 2;
                (changes(mid, in) ? at : lo) = mid;
            }
            if (in) r.back().second = at;
            else r.push_back({at, kMatrixNoEnd});
            in = !in;
        }
        return r;
    };
    if (ranges(kGemmLaunchUs + float(h->plan.M) * float(h->plan.N) * 2.f / kGemmStoreBytesPerUs, true).empty()) return TN_OK;
    if (!matrix_plan_of(h, desc)) return TN_OK;
    const tn::MatrixPlan& m = h->matrix_plans.m;
    h->mat_bytes = m.w_elems * 2;
    float us = 0.f;
    for (int i = 0; i < 2; ++i) {
        h->mat_build[i] = m.half[i].tensors.size() == 2;
        if (!h->mat_build[i]) continue;
        h->mat_half_off[i] = h->mat_bytes;
        h->mat_bytes += (m.half[i].build.out_elems * 2 + 255) & ~int64_t(255);
        fill_product_step(&h->mat_half[i].s, m.half[i].build);
        us += product_us(h, h->mat_half[i].s);
    }
    fill_product_step(&h->mat_w.s, m.w);
    us += product_us(h, h->mat_w.s);
    h->mat_flops = 2 * m.w.R * m.w.C * m.w.K;
    for (int i = 0; i < 2; ++i)
        if (h->mat_build[i]) h->mat_flops += 2 * m.half[i].build.R * m.half[i].build.C * m.half[i].build.K;
    const std::vector<std::pair<int64_t, int64_t>> taken = ranges(us);
    if (taken.empty()) return TN_OK;
    // room in the workspace: beside what else is kept there, or sharing a caller's block with it
    const int64_t room = desc->workspace
                             ? desc->workspace_bytes - (desc->flags & TN_FLAG_NO_SPLIT_K ? 0 : std::min<int64_t>(kMaxPartialBytes, desc->workspace_bytes / 4)) - 512
                             : (desc->workspace_limit_bytes > 0 ? desc->workspace_limit_bytes : kDefaultWorkspaceBytes) -
                                   (h->lazy ? h->lazy_slice_bytes : 0) - 2 * h->plan.max_intermediate * h->elt;
    if (h->mat_bytes > room) return TN_OK;
    // tables: rows and columns of the three products, then of Y
    std::vector<int32_t> tab;
    size_t at[8];
    auto put = [&](int i, const std::vector<int32_t>& v) {
        at[i] = tab.size();
        tab.insert(tab.end(), v.begin(), v.end());
    };
    for (int i = 0; i < 2; ++i) {
        put(2 * i, m.half[i].build.row_off);
        put(2 * i + 1, m.half[i].build.col_off);
    }
    put(4, m.w.row_off);
    put(5, m.w.col_off);
    put(6, {0});
    std::vector<int32_t> cols(size_t(m.M));
    for (int64_t c = 0; c < m.M; ++c) cols[size_t(c)] = int32_t(c);
    put(7, cols);
    void* tables = nullptr;
    if (hipMalloc(&tables, tab.size() * sizeof(int32_t)) != hipSuccess) return TN_ERR_ALLOC;
    h->mat_kept.push_back(tables);
    if (upload_tables(h, std::move(tab), tables, st) != TN_OK) return TN_ERR_HIP;
    auto set_tables = [&](DevStep* s, int i) {
        s->crow = static_cast<const int32_t*>(tables) + at[i];
        s->ccol = static_cast<const int32_t*>(tables) + at[i + 1];
    };
    for (int i = 0; i < 2; ++i) {
        const tn::MatrixHalf& H = m.half[i];
        int rc;
        void* p = nullptr;
        if (!h->mat_build[i]) {
            rc = keep_operand(h, desc, H.keep, m.Krp, i == 1, &p);
            if (i == 0) h->mat_w.a = p;
            else h->mat_w.s.packed = p;
        } else {
            set_tables(&h->mat_half[i].s, 2 * i);
            rc = keep_operand(h, desc, H.build.a, H.build.Kp, false, &p);
            h->mat_half[i].a = p;
            if (rc == TN_OK) rc = keep_operand(h, desc, H.build.b, H.build.Kp, true, &h->mat_half[i].s.packed);
        }
        if (rc != TN_OK) return rc;
    }
    set_tables(&h->mat_w.s, 4);
    set_tables(&y, 6);
    h->matrix = true;
    h->mat_ranges = taken;
    return TN_OK;
}

// The plan and what it kept go away: every call runs the other orders.
int drop_matrix(tn_linear_s* h, hipStream_t st) {
    (void)hipGetLastError();                                        // of the allocation that was refused
    if (hipStreamSynchronize(st) != hipSuccess) return TN_ERR_HIP;  // the kernels that write the operands may still be running
    for (size_t i = 0; i < h->mat_kept_count; ++i) (void)hipFree(h->mat_kept[i]);
    h->mat_kept.erase(h->mat_kept.begin(), h->mat_kept.begin() + std::ptrdiff_t(h->mat_kept_count));
    h->packed_bytes -= h->mat_kept_bytes;
    h->mat_kept_count = 0;
    h->mat_kept_bytes = 0;
    h->matrix = false;
    return TN_OK;
}

// Where W and the halves are.
void place_matrix(tn_linear_s* h, void* mem) {
    char* base = static_cast<char*>(mem);
    h->mat_mem = mem;
    h->mat_w.out = base;
    h->mat_y.packed = base;
    for (int i = 0; i < 2; ++i)
        if (h->mat_build[i]) {
            void* half = base + h->mat_half_off[i];
            h->mat_half[i].out = half;
            if (i == 0) h->mat_w.a = half;
            else h->mat_w.s.packed = half;
        }
}

// ---- both factors on a side of a Tucker core, a workgroup to a token ----
using factor_pair_t = void (*)(FactorPairArgs, FactorPairArgs);
struct FactorPairConfig {
    bool in;                               // the side of the modes comes in
    int A, B, P, Q;                        // largest extents
    int per_cu;                            // workgroups on a compute unit
    factor_pair_t kern;
    size_t smem;
    // multiply-adds of a token, padding included, for each workgroup that a compute unit holds
    int64_t work() const { return int64_t(A) * Q * (in ? B + P : P + B) / per_cu; }
};

template <int A32, int B32, int P32, int Q32>
constexpr FactorPairConfig factor_in_config() {
    return {true, 32 * A32, 32 * B32, 32 * P32, 32 * Q32, A32 < 5 ? 3 : 2, factor_in_kernel<A32, B32, P32, Q32>, factor_in_smem<A32, B32, P32, Q32>()};
}
template <int A32, int B32, int P32, int Q32>
constexpr FactorPairConfig factor_out_config() {
    return {false, 32 * A32, 32 * B32, 32 * P32, 32 * Q32, A32 < 5 ? 3 : 2, factor_out_kernel<A32, B32, P32, Q32>, factor_out_smem<A32, B32, P32, Q32>()};
}

// Modes of up to 64 x 96, 64 x 128 and 160 x 160.
constexpr int kFactorPairConfigs = 12;
const FactorPairConfig* factor_pair_configs() {
    static const FactorPairConfig c[kFactorPairConfigs] = {
        factor_in_config<2, 3, 2, 2>(),  factor_in_config<2, 4, 2, 2>(),  factor_in_config<2, 4, 2, 3>(),  factor_in_config<5, 5, 1, 1>(),
        factor_in_config<5, 5, 2, 2>(),  factor_in_config<5, 5, 3, 3>(),  factor_out_config<2, 3, 2, 2>(), factor_out_config<2, 3, 2, 3>(),
        factor_out_config<2, 4, 2, 3>(), factor_out_config<5, 5, 1, 1>(), factor_out_config<5, 5, 2, 2>(), factor_out_config<5, 5, 3, 3>()};
    return c;
}

// Two steps that are such a pair: a token's plain matrix [R][K] in, [C1][R] between them, a plain matrix [C1][C2] out, extents of whole
// tiles of the matrix cores.
bool is_factor_pair(const tn::Step& s, const tn::Step& u) {
    auto strides = [](const std::vector<int32_t>& t, int64_t stride) {
        for (size_t i = 0; i < t.size(); ++i)
            if (t[i] != int64_t(i) * stride) return false;
        return true;
    };
    if (!s.a_plain || !u.a_plain || s.trace_extent != 1 || u.trace_extent != 1 || u.R != s.C || u.K != s.R) return false;
    if (s.R % 16 || s.K % 16 || s.C % 16 || u.C % 16) return false;
    if (s.a_tok_stride != s.R * s.K || s.c_tok_stride != s.R * s.C || u.a_tok_stride != s.c_tok_stride || u.c_tok_stride != u.R * u.C) return false;
    return strides(s.crow, 1) && strides(s.ccol, s.R) && strides(u.crow, u.C) && strides(u.ccol, 1);
}

// The form that holds a pair with the least work; of two alike, on the way out the one that stores whole rows where there is much to store. us of a
// layer of one such pair at 8192 tokens, so / by the least LDS, which all forms of 160 x 160 share: out-factors 80 x 80 from ranks of 32 49 / 94,
// 96 x 96 from ranks of 48 68 / 108, 64 x 64 from ranks of 16 28 / 34.
int factor_pair_config(const tn::Step& s, const tn::Step& u) {
    if (!is_factor_pair(s, u)) return -1;
    const bool out = s.R * s.K < s.C * u.C;
    int best = -1;
    for (int i = 0; i < kFactorPairConfigs; ++i) {
        const FactorPairConfig& c = factor_pair_configs()[i];
        if (!(c.in ? s.R <= c.A && s.K <= c.B && u.C <= c.P && s.C <= c.Q : s.C <= c.A && u.C <= c.B && s.K <= c.P && s.R <= c.Q)) continue;
        const FactorPairConfig* b = best < 0 ? nullptr : &factor_pair_configs()[best];
        if (!b || c.work() < b->work() || (c.work() == b->work() && b->in && !c.in && out && 2 * s.C * u.C > int64_t(c.A) * c.B)) best = i;
    }
    return best;
}

// Where step_chain2_kernel holds a pair too, with a wave to a token and no padding of small extents, it is the faster one for many tokens where the
// ranks are no more than 32 on the way in (K up to 96), or a mode is on the way out: from more than a round of two workgroups on a
// compute unit, and for ever unless the modes fill half of the form. us of a layer of one such pair there / here at 512, 1000, 2000 and 8192
// tokens: in-factors 64 x 80 to ranks of 32 10.0 / 10.2, 10.7 / 11.4, 14.9 / 14.9, 31 / 29; 80 x 80 to 16 8.2 / 8.5, 8.5 / 10.7, 15.3 / 16.9, 38 / 43;
// 48 x 48 to 32 10.0 / 10.2, 10.6 / 11.3, 14.1 / 14.8, 25.7 / 26.5; out-factors 32 x 32 from 16 7.1 / 7.2, 7.6 / 8.2, 11.3 / 11.6, 20.5 / 23.5. Not so: in-factors
// 64 x 80 to ranks of 48 14.2 / 13.9, 18.2 / 16.9, 22.9 / 20.2, 45 / 38, and a K of 97 to 128 or larger out-modes whatever the ranks. Out-factors of
// one small mode or from one small rank that are three quarters padding on a form of 160 x 160 stay there (128 x 64 from 96 and 32 at 128 and
// 8192 tokens 8.8 / 9.8, 85 / 108; 160 x 32 from 48 and 16 at 16 and 200 28.9 / 30.0, 29.2 / 30.1 in a layer of in-factors 32 x 160). Over 98 pairs
// of modes 32 to 160 and ranks 16 to 96.
void share_factor_pair(DevStep* a, const tn::Step& u) {
    const tn::Step& s = a->plan;
    const FactorPairConfig& c = factor_pair_configs()[a->pair_cfg];
    const bool in = s.R * s.K >= s.C * u.C, small = in ? a->chain_cfg != 1 && std::max(s.C, u.C) <= 32 : a->chain_cfg == 2 && std::min(s.C, u.C) <= 32;
    const bool padding = 4 * (s.R * s.K * s.C + s.R * s.C * u.C) < c.work() * c.per_cu;
    if (!in && padding && (a->chain_cfg == 1 || (small && c.A > 64))) a->pair_cfg = -1;
    else if (small) {
        a->pair_gap[0] = 512;
        a->pair_gap[1] = 2 * (in ? s.R * s.K : s.C * u.C) > int64_t(c.A) * c.B ? 2048 : std::numeric_limits<int64_t>::max();
    }
}

// Calls of more (token, 32 columns) items than step_chain2_fine_kernel takes, which spreads a token over several compute units: below,
// that is what counts. us of a layer of one pair there / here: out-factors 160 x 160 from ranks of 96 at 8 tokens (40 items) 8.6 / 10.0, at 16
// 11.2 / 10.2; 128 x 128 from 96 at 16 (64 items) 8.9 / 10.1, at 32 12.1 / 11.1; in-factors 96 x 96 to 64 at 32 (64 items) 12.4 / 13.3, at 64 16.0 / 15.7.
constexpr int64_t kChain2FineMaxItems = 64;      // (token, c1 tile) items up to which every c2 tile gets a wave of its own

bool factor_pair_applies(const DevStep& s1, int64_t tokens) {
    if (s1.pair_cfg < 0 || s1.chain_cfg == 3) return s1.pair_cfg >= 0;
    return tokens * ((s1.plan.C + 31) / 32) > kChain2FineMaxItems && (tokens <= s1.pair_gap[0] || tokens >= s1.pair_gap[1]);
}

FactorPairArgs factor_pair_args(const DevStep& s1, const DevStep& s2, const void* in, void* out, int64_t tokens) {
    FactorPairArgs a;
    a.in = static_cast<const bf16_t*>(in);
    a.out = static_cast<bf16_t*>(out);
    a.first = static_cast<const bf16_t*>(s1.packed);
    a.second = static_cast<const bf16_t*>(s2.packed);
    a.nks_first = s1.Kp >> 4;
    a.nks_second = s2.Kp >> 4;
    a.size_first = s1.Cp * s1.Kp * 2;
    a.size_second = s2.Cp * s2.Kp * 2;
    const bool i = factor_pair_configs()[s1.pair_cfg].in;
    const int32_t R = int32_t(s1.plan.R), K = int32_t(s1.plan.K), C1 = int32_t(s1.plan.C), C2 = int32_t(s2.plan.C);
    a.A = i ? R : C1;
    a.B = i ? K : C2;
    a.P = i ? C2 : K;
    a.Q = i ? C1 : R;
    a.tokens = int32_t(tokens);
    return a;
}

// One launch for a pair of one layer (p1 == nullptr) or of two layers with the same instantiation.
int launch_factor_pair(const tn_linear_s* h, int cfg, const FactorPairArgs& p0, const FactorPairArgs* p1, hipStream_t st) {
    const FactorPairConfig& c = factor_pair_configs()[cfg];
    const int64_t wgs = std::min<int64_t>(p0.tokens, int64_t(h->num_cus) * c.per_cu / (p1 ? 2 : 1));
    hipLaunchKernelGGL(c.kern, dim3(uint32_t(wgs), p1 ? 2 : 1), dim3(256), c.smem, st, p0, p1 ? *p1 : p0);
    return hipGetLastError() == hipSuccess ? TN_OK : TN_ERR_HIP;
}

// Pairs of steps the transposing chain kernel can run (see step_chain2_kernel): both plain, the
// first step's output stored transposed ([c1][r], which is what the second step reads as rows c1
// with K = r), the output in aligned runs of 8 along c1 or along c2, and sizes within one of the
// two instantiations.
int plan_chain2(tn_linear_s* h, hipStream_t st) {
    if (h->plan.dtype != TN_DTYPE_BF16 || (h->flags & (TN_FLAG_SCALAR_KERNELS | TN_FLAG_NO_CHAIN2)) ||
        h->pair || h->kron)
        return TN_OK;
    const std::vector<int> pairs = tn::chain2_pairs(h->plan);
    for (size_t i = 0; i + 1 < h->steps.size(); ++i) {
        DevStep& a = h->steps[i];
        DevStep& b = h->steps[i + 1];
        if (!pairs[i] || a.variant == VAR_SCALAR || b.variant == VAR_SCALAR) continue;
        int cfg = 0, run_c1 = 0;
        if (!tn::chain2_shape(h->plan, a.plan, b.plan, &cfg, &run_c1)) continue;
        const int C2T = cfg == 0 ? 5 : 2, KS = cfg == 0 ? 6 : 4;
        size_t elems = size_t(C2T) * KS * 512;
        if (hipMalloc(&a.chain_bbf, elems * sizeof(bf16_t)) != hipSuccess) return TN_ERR_ALLOC;
        h->packed_bytes += int64_t(elems * sizeof(bf16_t));
        hipLaunchKernelGGL(chain2_repack_kernel, dim3(uint32_t((elems + 255) / 256)), dim3(256), 0, st,
                           static_cast<const bf16_t*>(b.packed), static_cast<bf16_t*>(a.chain_bbf), C2T, KS, b.Kp >> 4,
                           b.Cp, b.Kp);
        if (hipGetLastError() != hipSuccess) return TN_ERR_HIP;
        a.fuse_next = true;
        if (cfg == 1 && a.plan.K <= 80) cfg = 2;         // <2,5,2>: the same layouts with 5 k-steps instead of 8
        a.chain_cfg = cfg;
        a.chain_run_c1 = run_c1;
    }
    // pairs for the kernels with a workgroup to a token: those above, and what has more rows or a longer K than they take
    if (((h->flags >> TN_FLAG_VARIANT_SHIFT) & 0xff) != 0) return TN_OK;
    for (size_t i = 0; i + 1 < h->steps.size(); ++i) {
        DevStep& a = h->steps[i];
        const DevStep& b = h->steps[i + 1];
        if (a.variant == VAR_SCALAR || b.variant == VAR_SCALAR || (!a.fuse_next && (b.fuse_next || (i > 0 && h->steps[i - 1].fuse_next)))) continue;
        a.pair_cfg = factor_pair_config(a.plan, b.plan);
        if (a.pair_cfg < 0) continue;
        if (a.fuse_next) {
            share_factor_pair(&a, b.plan);
            continue;
        }
        a.fuse_next = true;
        a.chain_cfg = 3;
    }
    return TN_OK;
}

Chain2Args chain2_args(const DevStep& s1, const DevStep& s2, const void* A, void* Out, int64_t tokens) {
    Chain2Args p;
    p.In = A;
    p.Out = Out;
    p.Ba = s1.packed;
    p.Bbf = s1.chain_bbf;
    p.off1 = s2.crow;
    p.off2 = s2.ccol;
    p.in_tok_stride = s1.plan.a_tok_stride;
    p.out_tok_stride = s2.plan.c_tok_stride;
    p.tokens = int32_t(tokens);
    p.R1 = int32_t(s1.plan.R);
    p.K1 = int32_t(s1.plan.K);
    p.C1 = int32_t(s1.plan.C);
    p.C2 = int32_t(s2.plan.C);
    p.nks_a = s1.Kp >> 4;
    p.c1_tiles = (p.C1 + 31) / 32;
    p.tiles_per_item = 1;
    return p;
}

// Few tokens: every (token, c1 tile) item of a chained pair gets a wave of its own, operands requested up front.
bool chain2_small_applies(const tn_linear_s* h, const DevStep& s1, int64_t tokens) {
    return tokens * ((s1.plan.C + 31) / 32) <= int64_t(h->num_cus) * 4 && !(h->flags & TN_FLAG_NO_DECODE_FUSION) &&
           !factor_pair_applies(s1, tokens);
}

// One launch for the pair of one layer (p1 == nullptr) or of two layers with the same instantiation.
int launch_chain2_small(const DevStep& s1, const Chain2Args& p0, const Chain2Args* p1, hipStream_t st) {
    using k_t = void (*)(Chain2Args, Chain2Args);
    static const k_t small[6] = {step_chain2_small_kernel<3, 6, 5, 0>, step_chain2_small_kernel<3, 6, 5, 1>,
                                 step_chain2_small_kernel<2, 8, 2, 0>, step_chain2_small_kernel<2, 8, 2, 1>,
                                 step_chain2_small_kernel<2, 5, 2, 0>, step_chain2_small_kernel<2, 5, 2, 1>};
    int64_t items = int64_t(p0.tokens) * p0.c1_tiles;
    if (p1) items = std::max(items, int64_t(p1->tokens) * p1->c1_tiles);
    if (items <= kChain2FineMaxItems) {
        // few items: one wave per (token, c1 tile, c2 tile)
        static const k_t fine[6] = {step_chain2_fine_kernel<3, 6, 0>, step_chain2_fine_kernel<3, 6, 1>,
                                    step_chain2_fine_kernel<2, 8, 0>, step_chain2_fine_kernel<2, 8, 1>,
                                    step_chain2_fine_kernel<2, 5, 0>, step_chain2_fine_kernel<2, 5, 1>};
        int64_t fine_items = int64_t(p0.tokens) * p0.c1_tiles * ((p0.C2 + 31) / 32);
        if (p1) fine_items = std::max(fine_items, int64_t(p1->tokens) * p1->c1_tiles * ((p1->C2 + 31) / 32));
        hipLaunchKernelGGL(fine[s1.chain_cfg * 2 + s1.chain_run_c1], dim3(uint32_t(fine_items), p1 ? 2 : 1), dim3(64), 0, st, p0,
                           p1 ? *p1 : p0);
        return hipGetLastError() == hipSuccess ? TN_OK : TN_ERR_HIP;
    }
    hipLaunchKernelGGL(small[s1.chain_cfg * 2 + s1.chain_run_c1], dim3(uint32_t((items + 3) / 4), p1 ? 2 : 1), dim3(256), 0, st,
                       p0, p1 ? *p1 : p0);
    return hipGetLastError() == hipSuccess ? TN_OK : TN_ERR_HIP;
}

int launch_chain2(const tn_linear_s* h, const DevStep& s1, const DevStep& s2, const void* A, void* Out, int64_t tokens,
                  hipStream_t st) {
    using k_t = void (*)(Chain2Args);
    static const k_t kerns[6] = {step_chain2_kernel<3, 6, 5, 0>, step_chain2_kernel<3, 6, 5, 1>,
                                 step_chain2_kernel<2, 8, 2, 0>, step_chain2_kernel<2, 8, 2, 1>,
                                 step_chain2_kernel<2, 5, 2, 0>, step_chain2_kernel<2, 5, 2, 1>};
    static const size_t smem[3] = {chain2_smem_bytes<3, 6, 5>(), chain2_smem_bytes<2, 8, 2>(), chain2_smem_bytes<2, 5, 2>()};
    if (!s1.packed) {                      // configuration call (create time)
        for (int i = 0; i < 6; ++i)
            if (hipFuncSetAttribute(reinterpret_cast<const void*>(kerns[i]), hipFuncAttributeMaxDynamicSharedMemorySize,
                                    int(smem[i / 2])) != hipSuccess)
                return TN_ERR_HIP;
        return TN_OK;
    }
    if (factor_pair_applies(s1, tokens)) return launch_factor_pair(h, s1.pair_cfg, factor_pair_args(s1, s2, A, Out, tokens), nullptr, st);
    Chain2Args p = chain2_args(s1, s2, A, Out, tokens);
    if (chain2_small_applies(h, s1, tokens)) return launch_chain2_small(s1, p, nullptr, st);
    // a wave per token when there are tokens enough to fill the chip, else a wave per (token, c1 tile)
    const int64_t waves = int64_t(h->num_cus) * 4;
    p.tiles_per_item = tokens >= waves ? p.c1_tiles : 1;
    const int64_t n_groups = (p.c1_tiles + p.tiles_per_item - 1) / p.tiles_per_item;
    const int64_t items = tokens * n_groups;
    // the narrow instantiation leaves room for two workgroups per CU
    const int64_t wgs = int64_t(h->num_cus) * (s1.chain_cfg == 2 ? 2 : 1);
    dim3 grid(uint32_t(std::min<int64_t>((items + 3) / 4, wgs)));
    hipLaunchKernelGGL(kerns[s1.chain_cfg * 2 + s1.chain_run_c1], grid, dim3(256), smem[s1.chain_cfg], st, p);
    return hipGetLastError() == hipSuccess ? TN_OK : TN_ERR_HIP;
}

// A chained factor pair and the wide step after it as one launch (step_chain2_split_kernel), for calls of a few
// tokens: applicable when the pair runs on one of the two small instantiations, the wide step would run on the
// split-K kernel with one split and 8 waves, its rows are the tokens themselves (R = 1), its K fits the kernel's
// register budget and every (token, column tile) item of the pair gets a wave of its own.
constexpr int64_t kFusedDecodeMaxZBytes = 32 * 1024;
constexpr size_t kFusedDecodeRedBytes = 8 * 1024 * sizeof(float);
constexpr int kFusedDecodeKPW = 5;           // pieces of 64 k of the wide step per wave: K <= 8 * 5 * 64 = 2560

bool chain2_split_applies(const tn_linear_s* h, const DevStep& s1, const DevStep& s3, int64_t tokens) {
    if (!s1.fuse_next || s1.chain_cfg == 0 || s1.chain_cfg == 3 || (h->flags & (TN_FLAG_NO_SPLIT_K | TN_FLAG_NO_DECODE_FUSION))) return false;
    if (s3.fuse_next || s3.variant == VAR_SCALAR || s3.amode != 0 || s3.plan.R != 1) return false;
    if (tokens * ((s1.plan.C + 31) / 32) > 8 || s3.Kp > 8 * kFusedDecodeKPW * 64) return false;
    if (tokens * s3.plan.a_tok_stride * 2 > kFusedDecodeMaxZBytes) return false;
    const SplitCfg sc = split_config(s3, tokens);
    // (however many splits the wide step would take on its own: here a workgroup always walks the whole K, which for a
    // core this small is a few hundred KB per workgroup at most)
    return sc.use && sc.tm == 1 && sc.nw == 8 && sc.row_tiles == 1;
}

struct Chain2SplitArgs {
    Chain2Args c;
    StepArgs a;
    int z_bytes = 0;
    int kern = 0;
    uint32_t col_blocks = 0;
};

Chain2SplitArgs chain2_split_args(const DevStep& s1, const DevStep& s2, const DevStep& s3, const void* A, void* Out,
                                  int64_t tokens) {
    Chain2SplitArgs r;
    r.c = chain2_args(s1, s2, A, nullptr, tokens);      // the pair's result stays in LDS
    StepArgs& a = r.a;
    a.A = nullptr;                                       // likewise
    a.B = s3.q4_codes ? s3.q4_codes : s3.packed;
    a.Bs = s3.q4_scales;
    a.Out = Out;
    a.arow = nullptr;
    a.acol = nullptr;
    a.crow = s3.crow;
    a.ccol = s3.ccol;
    a.a_tok_stride = s3.plan.a_tok_stride;
    a.c_tok_stride = s3.plan.c_tok_stride;
    a.total_rows = uint32_t(tokens);
    a.R = 1;
    a.K = int32_t(s3.plan.K);
    a.Kp = s3.Kp;
    a.C = int32_t(s3.plan.C);
    a.Cp = s3.Cp;
    r.z_bytes = int((tokens * s3.plan.a_tok_stride * 2 + 255) & ~int64_t(255));
    r.kern = (s1.chain_cfg - 1) * 2 + s1.chain_run_c1 + (s3.q4_codes ? 4 : 0);
    r.col_blocks = uint32_t((s3.plan.C + 31) / 32);
    return r;
}

// One launch for one layer (p1 == nullptr) or for two layers on the same instantiation (grid.y = 2).
int launch_chain2_split(const tn_linear_s* h, const Chain2SplitArgs* p0, const Chain2SplitArgs* p1, hipStream_t st) {
    using k_t = void (*)(Chain2Args, StepArgs, int, Chain2Args, StepArgs, int);
    static const k_t kerns[16] = {                                  // a block to a workgroup, several
        step_chain2_split_kernel<8, 0, kFusedDecodeKPW, 0, 0>, step_chain2_split_kernel<8, 0, kFusedDecodeKPW, 0, 1>,
        step_chain2_split_kernel<8, 1, kFusedDecodeKPW, 0, 0>, step_chain2_split_kernel<8, 1, kFusedDecodeKPW, 0, 1>,
        step_chain2_split_kernel<5, 0, kFusedDecodeKPW, 0, 0>, step_chain2_split_kernel<5, 0, kFusedDecodeKPW, 0, 1>,
        step_chain2_split_kernel<5, 1, kFusedDecodeKPW, 0, 0>, step_chain2_split_kernel<5, 1, kFusedDecodeKPW, 0, 1>,
        step_chain2_split_kernel<8, 0, kFusedDecodeKPW, 1, 0>, step_chain2_split_kernel<8, 0, kFusedDecodeKPW, 1, 1>,
        step_chain2_split_kernel<8, 1, kFusedDecodeKPW, 1, 0>, step_chain2_split_kernel<8, 1, kFusedDecodeKPW, 1, 1>,
        step_chain2_split_kernel<5, 0, kFusedDecodeKPW, 1, 0>, step_chain2_split_kernel<5, 0, kFusedDecodeKPW, 1, 1>,
        step_chain2_split_kernel<5, 1, kFusedDecodeKPW, 1, 0>, step_chain2_split_kernel<5, 1, kFusedDecodeKPW, 1, 1>};
    if (!p0) {                             // configuration call (create time)
        for (int i = 0; i < 16; ++i)
            if (hipFuncSetAttribute(reinterpret_cast<const void*>(kerns[i]), hipFuncAttributeMaxDynamicSharedMemorySize,
                                    int(kFusedDecodeRedBytes + size_t(kFusedDecodeMaxZBytes))) != hipSuccess)
                return TN_ERR_HIP;
        return TN_OK;
    }
    const Chain2SplitArgs& q = p1 ? *p1 : *p0;
    // one workgroup to a compute unit (registers), each with the same number of blocks where the layers are alike
    const uint32_t most = std::max(p0->col_blocks, q.col_blocks), all = p0->col_blocks + (p1 ? p1->col_blocks : 0);
    const uint32_t cus = uint32_t(h->num_cus), per = (all + cus - 1) / cus, blocks = (most + per - 1) / per;
    const size_t smem = kFusedDecodeRedBytes + size_t(std::max(p0->z_bytes, q.z_bytes));
    hipLaunchKernelGGL(kerns[2 * p0->kern + (per > 1 ? 1 : 0)], dim3(blocks, p1 ? 2 : 1), dim3(512), smem, st, p0->c, p0->a, p0->z_bytes, q.c, q.a,
                       q.z_bytes);
    return hipGetLastError() == hipSuccess ? TN_OK : TN_ERR_HIP;
}

// 4-bit streams for the decode-size launches of a quantised layer: a step qualifies when its tensor is one of the
// caller's (not merged, no traced index pair), its k walks that tensor in memory order (K consecutive elements per
// column, K a multiple of 32) and every column starts on a block boundary. Such a step's split-K launches then read
// 0.53 bytes per parameter instead of 2. The bf16 packed tensor stays: larger calls run on it.
bool q4_streamable(const tn_linear_s* h, const tn::Step& p) {
    if (p.slot < 0 || p.slot >= h->plan.n_caller_tensors || p.trace_extent != 1 || p.K % 32 || p.kdims.empty()) return false;
    int64_t run = 1;
    for (size_t j = p.kdims.size(); j-- > 0;) {
        if (p.kdims[j].stride != run) return false;
        run *= p.kdims[j].extent;
    }
    for (const tn::GatherDim& d : p.cdims)
        if (d.stride % 32) return false;
    return true;
}

int prepare_q4_stream(tn_linear_s* h, hipStream_t st) {
    if (!(h->flags & TN_FLAG_QUANT_MXFP4) || (h->flags & (TN_FLAG_NO_Q4_STREAM | TN_FLAG_SCALAR_KERNELS | TN_FLAG_NO_SPLIT_K)) ||
        h->plan.dtype != TN_DTYPE_BF16)
        return TN_OK;
    for (DevStep& s : h->steps) {
        const tn::Step& p = s.plan;
        if (s.variant == VAR_SCALAR || !q4_streamable(h, p)) continue;
        // worth it only where a decode-size launch is a stream of this tensor: the split-K kernel must take one-row calls
        if (!split_config(s, p.R).use) continue;
        const int n_chunks = s.Kp / 64, col_blocks = int((p.C + 31) / 32);
        const int64_t pieces = int64_t(col_blocks) * n_chunks * 64;
        const int64_t code_bytes = pieces * 16, scale_bytes = (pieces + 255) & ~int64_t(255);
        if (hipMalloc(&s.q4_codes, size_t(code_bytes + scale_bytes)) != hipSuccess) return TN_ERR_ALLOC;
        s.q4_scales = static_cast<char*>(s.q4_codes) + code_bytes;
        h->packed_bytes += code_bytes + scale_bytes;
        h->q4_stream_bytes += code_bytes + scale_bytes;
        Q4PackArgs a;
        memset(&a, 0, sizeof(a));
        a.codes = static_cast<const unsigned char*>(h->quant_codes[size_t(p.slot)]);
        a.exps = static_cast<const signed char*>(h->quant_exps[size_t(p.slot)]);
        a.out_codes = static_cast<uint4*>(s.q4_codes);
        a.out_scales = static_cast<unsigned char*>(s.q4_scales);
        a.C = int32_t(p.C);
        a.K = int32_t(p.K);
        a.n_chunks = n_chunks;
        a.col_blocks = col_blocks;
        a.nc = int32_t(p.cdims.size());
        for (size_t j = 0; j < p.cdims.size(); ++j) {
            a.cext[j] = p.cdims[j].extent;
            a.cstr[j] = p.cdims[j].stride;
        }
        hipLaunchKernelGGL(q4_stream_pack_kernel, dim3(uint32_t(std::min<int64_t>((pieces + 255) / 256, 16384))), dim3(256), 0, st, a);
        if (hipGetLastError() != hipSuccess) return TN_ERR_HIP;
    }
    return TN_OK;
}

// Kernels that use more than 64 KB of LDS need their limit raised once per device. Done at create
// time (never inside tn_linear_forward, which must stay legal under stream capture from its first
// call). The launchers double as configurators: called with an empty step they set the attribute of
// every kernel they can launch and return.
// Device address of the static scratch array on each GPU, looked up once per device at create time with that
// device current (every GPU holds its own copy of the array at its own address).
void* g_scratch_ptr[64] = {};

int configure_kernels(int device) {
    static bool done[64] = {};
    static std::mutex lock;                // handles may be created from several host threads
    std::lock_guard<std::mutex> guard(lock);
    if (device >= 0 && device < 64 && done[device]) return TN_OK;
    const DevStep none;                    // packed == nullptr: configuration call
    const StepArgs a{};
    const tn_linear_s* no_handle = nullptr;
    int rc = launch_pipe<2, 2, 2, 4, 1, 2>(none, a, 0, nullptr);
    if (rc == TN_OK) rc = launch_pipe<4, 1, 2, 4, 1, 2>(none, a, 0, nullptr);
    if (rc == TN_OK) rc = configure_gemm();
    if (rc == TN_OK) rc = launch_chain2(no_handle, none, none, nullptr, nullptr, 0, nullptr);
    if (rc == TN_OK) rc = launch_chain2_split(nullptr, nullptr, nullptr, nullptr);
    for (int i = 0; i < kSkinnyKernels && rc == TN_OK; ++i)
        if (hipFuncSetAttribute(reinterpret_cast<const void*>(skinny_kernels()[i]), hipFuncAttributeMaxDynamicSharedMemorySize,
                                int(kSplitLdsRowBytes)) != hipSuccess)
            rc = TN_ERR_HIP;
    for (int i = 0; i < kSplitLdsKernels && rc == TN_OK; ++i)
        if (hipFuncSetAttribute(reinterpret_cast<const void*>(split_lds_kernels()[i]), hipFuncAttributeMaxDynamicSharedMemorySize,
                                int(kSplitLdsRowBytes)) != hipSuccess)
            rc = TN_ERR_HIP;
    if (rc == TN_OK &&
        (hipFuncSetAttribute(reinterpret_cast<const void*>(&step_pair_kernel<kPairStages, kPairBar>),
                             hipFuncAttributeMaxDynamicSharedMemorySize, int(kPairSmemBytes)) != hipSuccess ||
         hipFuncSetAttribute(reinterpret_cast<const void*>(bond_grad_kernel<1>),
                             hipFuncAttributeMaxDynamicSharedMemorySize, int(BondGradShape<1>::SMEM)) != hipSuccess ||
         hipFuncSetAttribute(reinterpret_cast<const void*>(bond_grad_kernel<2>),
                             hipFuncAttributeMaxDynamicSharedMemorySize, int(BondGradShape<2>::SMEM)) != hipSuccess ||
         hipFuncSetAttribute(reinterpret_cast<const void*>(bond_grad_kernel<3>),
                             hipFuncAttributeMaxDynamicSharedMemorySize, int(BondGradShape<3>::SMEM)) != hipSuccess))
        rc = TN_ERR_HIP;
    for (int i = 0; i < kFactorPairConfigs && rc == TN_OK; ++i)
        if (hipFuncSetAttribute(reinterpret_cast<const void*>(factor_pair_configs()[i].kern), hipFuncAttributeMaxDynamicSharedMemorySize,
                                int(factor_pair_configs()[i].smem)) != hipSuccess)
            rc = TN_ERR_HIP;
    for (int i = 0; i < 4 && rc == TN_OK; ++i)
        if (hipFuncSetAttribute(reinterpret_cast<const void*>(small_chain_kernel_of((i & 1) != 0, (i & 2) != 0)),
                                hipFuncAttributeMaxDynamicSharedMemorySize, int(kSmallChainMaxLds)) != hipSuccess)
            rc = TN_ERR_HIP;
    for (int cfg = 0; cfg < tn::kKronConfigs && rc == TN_OK; ++cfg) rc = kron_dispatch(cfg, nullptr, 0, nullptr);
    for (int cfg = 0; cfg < tn::kDirectConfigs; ++cfg)
        for (int steps = 1; steps <= tn::kDirectMaxSteps && rc == TN_OK; ++steps) rc = direct_dispatch(cfg, steps, nullptr, 0, nullptr);
    if (rc == TN_OK) rc = gen_mfma_dispatch(nullptr, 0, nullptr);
    if (rc == TN_OK) rc = gen_mfma_both_dispatch(nullptr, nullptr, 0, nullptr);
    if (rc == TN_OK && device >= 0 && device < 64) {
        void* ptr = nullptr;
        if (hipGetSymbolAddress(&ptr, HIP_SYMBOL(scratch)) != hipSuccess || !ptr) rc = TN_ERR_HIP;
        else g_scratch_ptr[device] = ptr;
    }
    if (rc == TN_OK && device >= 0 && device < 64) done[device] = true;
    return rc;
}

int plan_value(const tn::Plan& p, int32_t what, int64_t* value) {
    switch (what) {
        case TN_QUERY_PARAM_COUNT: *value = p.params; return TN_OK;
        case TN_QUERY_FLOPS_PER_TOKEN: *value = p.flops; return TN_OK;
        case TN_QUERY_NUM_STEPS: *value = int64_t(p.steps.size()); return TN_OK;
        case TN_QUERY_MAX_INTERMEDIATE: *value = p.max_intermediate; return TN_OK;
        case TN_QUERY_OUT_FEATURES: *value = p.M; return TN_OK;
        case TN_QUERY_IN_FEATURES: *value = p.N; return TN_OK;
        case TN_QUERY_NUM_MERGES: *value = int64_t(p.merges.size()); return TN_OK;
        case TN_QUERY_PAIR_CHAINABLE: *value = tn::pair_chainable(p) ? 1 : 0; return TN_OK;
        case TN_QUERY_KRON_CHAINABLE: {
            tn::KronDims d;
            *value = (!tn::pair_chainable(p) && tn::kron_shape(p, &d)) ? 1 + d.cfg : 0;
            return TN_OK;
        }
        default: break;
    }
    if (what >= TN_QUERY_STEP_BASE) {
        int s = (what - TN_QUERY_STEP_BASE) / 10, f = (what - TN_QUERY_STEP_BASE) % 10;
        if (s >= int(p.steps.size())) return TN_ERR_INVALID_ARG;
        const tn::Step& st = p.steps[size_t(s)];
        switch (f) {
            case 0: *value = st.R; return TN_OK;
            case 1: *value = st.K; return TN_OK;
            case 2: *value = st.C; return TN_OK;
            case 3: *value = st.flops; return TN_OK;
            case 4: *value = st.slot; return TN_OK;
            case 7: {
                int cfg = 0, run_c1 = 0;
                *value = (size_t(s) + 1 < p.steps.size() && !tn::pair_chainable(p) &&
                          tn::chain2_shape(p, st, p.steps[size_t(s) + 1], &cfg, &run_c1)) ? 1 + cfg : 0;
                return TN_OK;
            }
            default: return TN_ERR_INVALID_ARG;
        }
    }
    return TN_ERR_INVALID_ARG;
}

// Offsets of every flat index over `dims` (outer -> inner) as an int32 table.
std::vector<int32_t> gather_table(const std::vector<tn::GatherDim>& dims, int64_t total) {
    std::vector<int32_t> tab(static_cast<size_t>(total));
    for (int64_t f = 0; f < total; ++f) {
        int64_t off = 0, rem = f;
        for (int j = int(dims.size()) - 1; j >= 0; --j) {
            off += (rem % dims[size_t(j)].extent) * dims[size_t(j)].stride;
            rem /= dims[size_t(j)].extent;
        }
        tab[size_t(f)] = int32_t(off);
    }
    return tab;
}

void fill_pack_dims(PackArgs* pa, const std::vector<tn::GatherDim>& kd, const std::vector<tn::GatherDim>& cd) {
    pa->nk = int32_t(kd.size());
    pa->nc = int32_t(cd.size());
    for (int j = 0; j < pa->nk; ++j) {
        pa->kext[j] = kd[size_t(j)].extent;
        pa->kstr[j] = kd[size_t(j)].stride;
    }
    for (int j = 0; j < pa->nc; ++j) {
        pa->cext[j] = cd[size_t(j)].extent;
        pa->cstr[j] = cd[size_t(j)].stride;
    }
}

void launch_pack(const PackArgs& pa, int elt, hipStream_t st) {
    int64_t total = int64_t(pa.Cp) * pa.Kp;
    uint32_t blocks = uint32_t(std::min<int64_t>((total + 255) / 256, 65535));
    if (elt == 2)
        hipLaunchKernelGGL(pack_kernel<bf16_t>, dim3(blocks), dim3(256), 0, st, pa);
    else
        hipLaunchKernelGGL(pack_kernel<float>, dim3(blocks), dim3(256), 0, st, pa);
}

// ---- gradients with respect to the parameter tensors (TN_FLAG_TRAINABLE) ----
constexpr int64_t kMaxGradPartialBytes = int64_t(256) << 20;
constexpr int64_t kGradMfmaMinExtent = 32;

// Row ranges a gradient launch is split into: enough workgroups to fill the chip, at least 64 rows each, partial
// tiles within `cap` bytes.
// How grad_param_mfma_kernel loads dOut (d) and In (i) of a step: 1 = 16-byte pieces along the columns, 2 = 16-byte
// pieces along the rows (dOut only), 0 = element by element.
struct GradModes {
    int d = 0, i = 0;
};

GradModes grad_modes(const tn::Step& p) {
    GradModes m;
    if (p.c_vec == 8 && p.C % 8 == 0) m.d = 1;
    else if (p.r_vec == 8 && p.R % 8 == 0) m.d = 2;
    if (p.K % 8 == 0 && p.a_tok_stride % 8 == 0 && (p.a_plain || p.a_vec == 8)) m.i = 1;
    return m;
}

// bf16 steps whose tensor is at least a quarter of a 128 x 128 tile in both directions run on the matrix cores, and so
// do skinny ones (8 to 31 one way, 32 or more the other: the boundary cores of a train) when both operands come in
// 16-byte pieces: those are bound by reading the long operand once, which the tile kernel does in full lines
bool grad_on_mfma(const tn_linear_s* h, const tn::Step& p) {
    if (h->elt != 2) return false;
    if (p.C >= kGradMfmaMinExtent && p.K >= kGradMfmaMinExtent) return true;
    const GradModes m = grad_modes(p);
    return m.d != 0 && m.i != 0 && std::min(p.C, p.K) >= 8 && std::max(p.C, p.K) >= kGradMfmaMinExtent;
}

int grad_splits(const tn_linear_s* h, const tn::Step& p, int64_t rows, int64_t cap) {
    const int64_t edge = grad_on_mfma(h, p) ? 128 : 64;
    const int64_t tiles = ((p.C + edge - 1) / edge) * ((p.K + edge - 1) / edge);
    int64_t n = std::max<int64_t>(1, ((edge == 128 ? 2 : 4) * int64_t(h->num_cus) + tiles - 1) / tiles);
    n = std::min<int64_t>(n, std::max<int64_t>(1, rows / 64));
    n = std::min<int64_t>(n, std::max<int64_t>(1, cap / (p.C * p.K * 4)));
    n = std::min<int64_t>(n, 65535);
    // the matrix-core kernel keeps the tiles of a split on one XCD when the splits come in eights
    if (edge == 128 && n > 8 && (n + 7) / 8 * 8 * p.C * p.K * 4 <= cap && (n + 7) / 8 * 8 <= std::max<int64_t>(1, rows / 64)) n = (n + 7) / 8 * 8;
    return int(n);
}

int64_t grad_tokens_pad(int64_t tokens) { return (tokens + 63) / 64 * 64; }

TransposeArgs transpose_args(const void* src, void* dst, int64_t T, int64_t D, int64_t Tp, bool packed, const int32_t* to = nullptr) {
    return TransposeArgs{static_cast<const bf16_t*>(src), static_cast<bf16_t*>(dst), T, D, Tp, packed ? 1 : 0, to};
}

// Up to kTransposeMany matrices at a time.
void launch_transposes(const TransposeArgs* m, int n, hipStream_t st) {
    TransposeMany many;
    memset(&many, 0, sizeof(many));
    int64_t most = 0;
    for (int i = 0; i < n; ++i) {
        many.m[i] = m[i];
        most = std::max(most, (m[i].D + 63) / 64 * (m[i].Tp / 64));
    }
    hipLaunchKernelGGL(transpose_kernel, dim3(uint32_t(most), uint32_t(n)), dim3(256), 0, st, many);
}

// A step's gradient as one product over the tokens, straight into the caller's tensor: one row per token, both operands plain
// matrices, k and c the tensor's inner and outer axes in any order. From kGradProductElems elements on, where a pass of fp32
// sums through memory is what the tile kernel takes its time for (core of 9216 x 2304 at 500 tokens: 71 us and 109 to put the
// sums in place; 34 us here and 10 for the transposed copies).
constexpr int64_t kGradProductElems = int64_t(1) << 20;

bool grad_product_perms(const tn_linear_s* h, const tn::Step& p, std::vector<int32_t>* rows, std::vector<int32_t>* cols) {
    if (h->elt != 2 || (h->flags & TN_FLAG_SCALAR_KERNELS) || ((h->flags >> TN_FLAG_VARIANT_SHIFT) & 0xff) != 0) return false;
    if (p.R != 1 || !p.a_plain || p.trace_extent != 1 || p.K % 8 || p.C % 8 || p.K * p.C < kGradProductElems ||
        p.K * p.C >= (int64_t(1) << 31) || p.c_tok_stride != p.C || p.a_tok_stride != p.K || p.crow[0] != 0)
        return false;
    for (int64_t c = 0; c < p.C; ++c)
        if (p.ccol[size_t(c)] != c) return false;
    *rows = gather_table(p.cdims, p.C);
    *cols = gather_table(p.kdims, p.K);
    std::vector<char> row_hit(size_t(p.C), 0), col_hit(size_t(p.K), 0);
    for (int32_t& r : *rows) {
        if (r % p.K || r / p.K >= p.C || row_hit[size_t(r / p.K)]) return false;
        r = int32_t(r / p.K);
        row_hit[size_t(r)] = 1;
    }
    for (int32_t c : *cols) {
        if (c >= p.K || col_hit[size_t(c)]) return false;
        col_hit[size_t(c)] = 1;
    }
    return true;
}

// Bytes of the two transposed operands.
int64_t grad_product_bytes(const tn::Step& p, int64_t tokens) {
    return (p.C + (p.K + tn::kMatrixColPad - 1) / tn::kMatrixColPad * tn::kMatrixColPad) * grad_tokens_pad(tokens) * 2;
}

int launch_grad_product(const tn_linear_s* h, const DevStep& s, const void* dOut, const void* In, float* grad, int64_t tokens, hipStream_t st) {
    const tn::Step& p = s.plan;
    const int64_t tp = grad_tokens_pad(tokens);
    char* a = static_cast<char*>(h->grad_product_mem);
    char* b = a + p.C * tp * 2;
    const TransposeArgs both[2] = {transpose_args(dOut, a, tokens, p.C, tp, false, s.grad_row), transpose_args(In, b, tokens, p.K, tp, true, s.grad_col)};
    launch_transposes(both, 2, st);
    DevStep g;
    g.plan.R = p.C;
    g.plan.K = tp;
    g.plan.C = p.K;
    g.Kp = int(tp);
    g.Cp = round_up(int(p.K), tn::kMatrixColPad);
    g.cmode = 1;
    g.variant = VAR_GEMM;
    GemmSums f{grad, p.K, 1};
    return launch_product_of(h, g, a, b, nullptr, nullptr, 0, st, &f);
}

int prepare_backward(tn_linear_s* h, const tn_linear_desc* desc, hipStream_t st) {
    const size_t n = h->steps.size();
    if (!h->plan.merges.empty()) return TN_ERR_UNSUPPORTED;
    h->bwd.resize(n);
    std::vector<int32_t> tab;
    std::vector<size_t> off(n, 0);
    for (size_t s = 1; s < n; ++s) {
        const tn::Step& f = h->steps[s].plan;
        if (!f.a_plain) return TN_ERR_UNSUPPORTED;      // only a first step gathers
        off[s] = tab.size();
        for (int64_t r = 0; r < f.R; ++r) tab.push_back(int32_t(r * f.K));
        for (int64_t k = 0; k < f.K; ++k) tab.push_back(int32_t(k));
    }
    std::vector<size_t> grad_at(n, 0);
    std::vector<char> as_product(n, 0);
    for (size_t s = 0; s < n; ++s) {
        std::vector<int32_t> rows, cols;
        if (!grad_product_perms(h, h->steps[s].plan, &rows, &cols)) continue;
        as_product[s] = 1;
        grad_at[s] = tab.size();
        tab.insert(tab.end(), rows.begin(), rows.end());
        tab.insert(tab.end(), cols.begin(), cols.end());
    }
    if (hipMalloc(reinterpret_cast<void**>(&h->bwd_tables), std::max<size_t>(1, tab.size()) * sizeof(int32_t)) != hipSuccess)
        return TN_ERR_ALLOC;
    if (hipMemcpyAsync(h->bwd_tables, tab.data(), tab.size() * sizeof(int32_t), hipMemcpyHostToDevice, st) != hipSuccess ||
        hipStreamSynchronize(st) != hipSuccess)
        return TN_ERR_HIP;
    for (size_t s = 1; s < n; ++s) {
        const DevStep& fs = h->steps[s];
        const tn::Step& f = fs.plan;
        DevStep& b = h->bwd[s];
        b.plan.tensor = f.tensor;
        b.plan.slot = f.slot;
        b.plan.R = f.R;
        b.plan.K = f.C;
        b.plan.C = f.K;
        // dOut is read through the forward step's scatter tables, or as it stands where those leave a plain matrix (the core
        // of a Tucker layer, one row per token: 500 tokens x 9216 x 2304 in 48 us on the matrix-product kernel, 1116 us
        // gathered on the split-K kernel)
        b.plan.a_plain = f.c_tok_stride == f.R * f.C;
        for (int64_t r = 0; r < f.R && b.plan.a_plain; ++r) b.plan.a_plain = f.crow[size_t(r)] == r * f.C;
        for (int64_t c = 0; c < f.C && b.plan.a_plain; ++c) b.plan.a_plain = f.ccol[size_t(c)] == c;
        b.plan.a_tok_stride = f.c_tok_stride;
        b.plan.c_tok_stride = f.a_tok_stride;
        b.plan.c_vec = (f.K % 8 == 0) ? 8 : 1;
        b.plan.r_vec = 1;
        b.plan.a_vec = (f.c_vec == 8 && f.C % 8 == 0) ? 8 : 1;       // dOut's columns in 16-byte runs: gathered as such
        b.plan.kdims = f.cdims;
        b.plan.cdims = f.kdims;
        b.plan.trace_extent = f.trace_extent;
        b.plan.trace_stride = f.trace_stride;
        b.plan.flops = f.flops;
        b.arow = fs.crow;
        b.acol = fs.ccol;
        b.crow = h->bwd_tables + off[s];
        b.ccol = b.crow + f.R;
        choose_variant(h, &b, desc->flags);
        // dOut's rows in 16-byte runs (the forward step's output runs along them): the tile of 256 rows turns them round as it loads
        // them, and no other kernel can; 128 columns at a time cost a second read of dOut, from L2, where there are more
        if (b.amode == 1 && f.r_vec == 8 && f.R % 8 == 0 && f.c_tok_stride % 8 == 0 &&
            (b.variant == VAR_PIPE_128x256 || b.variant == VAR_PIPE_256x128) && ((desc->flags >> TN_FLAG_VARIANT_SHIFT) & 0xff) == 0) {
            b.variant = VAR_PIPE_256x128;
            b.amode = 3;
            b.bm = 256;
            b.bn = 128;
            b.Cp = round_up(int(b.plan.C), 128);
        }
        const int64_t bytes = int64_t(b.Cp) * b.Kp * h->elt;
        if (hipMalloc(&b.packed, size_t(bytes)) != hipSuccess) return TN_ERR_ALLOC;
        h->packed_bytes += bytes;
        PackArgs pa;
        memset(&pa, 0, sizeof(pa));
        pa.src = desc->tensors[f.slot];
        pa.dst = b.packed;
        pa.K = int32_t(b.plan.K);
        pa.Kp = b.Kp;
        pa.C = int32_t(b.plan.C);
        pa.Cp = b.Cp;
        fill_pack_dims(&pa, b.plan.kdims, b.plan.cdims);
        pa.trace_extent = f.trace_extent;
        pa.trace_stride = f.trace_stride;
        launch_pack(pa, h->elt, st);
        if (hipGetLastError() != hipSuccess) return TN_ERR_HIP;
    }
    // workspace of a backward pass: the saved inputs of steps 1 .. n-1 and two gradient buffers
    h->bwd_saved_off.assign(n, 0);
    int64_t saved = 0;
    for (size_t s = 1; s < n; ++s) {
        h->bwd_saved_off[s] = saved;
        saved += (h->steps[s].plan.a_tok_stride + 127) & ~int64_t(127);
    }
    h->bwd_saved_elems = saved;
    const int64_t dbuf = (h->plan.max_intermediate + 127) & ~int64_t(127);
    const int64_t per_token = (saved + 2 * dbuf) * h->elt;
    int64_t max_r = 1;
    for (const auto& s : h->steps) max_r = std::max(max_r, s.plan.R);
    const int64_t limit = desc->workspace_limit_bytes > 0 ? desc->workspace_limit_bytes : kDefaultWorkspaceBytes;
    int64_t chunk = h->max_tokens;
    if (h->mgrad) chunk = std::min<int64_t>(chunk, std::max<int64_t>(1, h->mgrad_min_tokens - 1));      // larger calls go through dW
    if (per_token > 0) chunk = std::min<int64_t>(chunk, std::max<int64_t>(1, limit / per_token));
    chunk = std::max<int64_t>(1, std::min<int64_t>(chunk, ((int64_t(1) << 31) - 1024) / max_r));
    h->bwd_chunk = chunk;
    const int64_t chain_bytes = (chunk * per_token + 255) & ~int64_t(255);
    int64_t product_bytes = 0;
    for (size_t s = 0; s < n; ++s)
        if (as_product[s] && chain_bytes + grad_product_bytes(h->steps[s].plan, chunk) <= limit) {
            product_bytes = std::max(product_bytes, grad_product_bytes(h->steps[s].plan, chunk));
            h->steps[s].grad_row = h->bwd_tables + grad_at[s];
            h->steps[s].grad_col = h->steps[s].grad_row + h->steps[s].plan.C;
        }
    h->bwd_ws_bytes = std::max<int64_t>(std::max<int64_t>(256, h->bwd_ws_bytes), chain_bytes + product_bytes);
    if (hipMalloc(&h->bwd_ws, size_t(h->bwd_ws_bytes)) != hipSuccess) return TN_ERR_ALLOC;
    h->grad_product_mem = static_cast<char*>(h->bwd_ws) + chain_bytes;
    int64_t need = h->bwd_partial_bytes;
    for (const auto& s : h->steps)
        need = std::max(need, int64_t(grad_splits(h, s.plan, chunk * s.plan.R, kMaxGradPartialBytes)) * s.plan.C * s.plan.K * 4);
    h->bwd_partial_bytes = need;
    if (hipMalloc(reinterpret_cast<void**>(&h->bwd_partial), size_t(need)) != hipSuccess) return TN_ERR_ALLOC;
    h->trainable = true;
    return TN_OK;
}

void fill_grad_dims(GradOutArgs* o, const std::vector<tn::GatherDim>& rows, const std::vector<tn::GatherDim>& cols) {
    o->nc = int32_t(rows.size());
    o->nk = int32_t(cols.size());
    for (size_t j = 0; j < rows.size(); ++j) {
        o->cext[j] = uint32_t(rows[j].extent);
        o->cstr[j] = rows[j].stride;
    }
    for (size_t j = 0; j < cols.size(); ++j) {
        o->kext[j] = uint32_t(cols[j].extent);
        o->kstr[j] = cols[j].stride;
    }
}

// Waves that share an element's splits: measured on 512 splits of 96 x 160 (and on 8 of 9216 x 2304, where one is best).
int launch_grad_reduce(GradOutArgs o, hipStream_t st) {
    const uint32_t rows = uint32_t((int64_t(1) << 31) / o.K - 1);      // a launch counts its elements in 31 bits
    for (const uint32_t C = o.C; o.c0 < C; o.c0 += rows) {
        o.C = std::min(rows, C - o.c0);
        const int64_t total = int64_t(o.C) * o.K;
        auto blocks = [&](int64_t per) { return dim3(uint32_t(std::min<int64_t>((total + per - 1) / per, 16384))); };
        if (o.n_split >= 64) hipLaunchKernelGGL(grad_reduce_kernel<16>, blocks(64), dim3(1024), 0, st, o);
        else if (o.n_split >= 16) hipLaunchKernelGGL(grad_reduce_kernel<4>, blocks(64), dim3(256), 0, st, o);
        else hipLaunchKernelGGL(grad_reduce_kernel<1>, blocks(256), dim3(256), 0, st, o);
    }
    return hipGetLastError() == hipSuccess ? TN_OK : TN_ERR_HIP;
}

// Tensors of under 2^31 elements, up to kGradOutMany of them in one launch.
void launch_grad_reduce_many(const GradOutMany& m, int count, hipStream_t st) {
    int64_t most = 0;
    int n_split = 0;
    bool pairs = true;
    for (int i = 0; i < count; ++i) {
        const GradOutArgs& o = m.o[i];
        most = std::max(most, int64_t(o.C) * o.K);
        n_split = std::max(n_split, o.n_split);
        pairs = pairs && o.K % 2 == 0 && o.ld % 2 == 0 && o.split_stride % 2 == 0;
    }
    using reduce_t = void (*)(GradOutMany);
    static const reduce_t kerns[4] = {grad_reduce_many_kernel<1, 1>, grad_reduce_many_kernel<1, 2>, grad_reduce_many_kernel<4, 1>,
                                      grad_reduce_many_kernel<4, 2>};
    const int y = n_split >= 16 ? 1 : 0;                     // (up to 32: the matrix-product kernel's ranges of K)
    const int64_t per = (y ? 64 : 256) * (pairs ? 2 : 1);
    hipLaunchKernelGGL(kerns[2 * y + (pairs ? 1 : 0)], dim3(uint32_t(std::min<int64_t>((most + per - 1) / per, 4096)), uint32_t(count)), dim3(256), 0, st, m);
}

// dP of one step from dOut and the step's saved input, into the caller's tensor.
int launch_param_gradient(const tn_linear_s* h, const DevStep& s, const void* dOut, const void* In, float* grad,
                          int64_t grad_elems, int64_t tokens, bool accumulate, hipStream_t st) {
    const tn::Step& p = s.plan;
    if (s.grad_row && !accumulate && (reinterpret_cast<uintptr_t>(grad) & 15) == 0)
        return launch_grad_product(h, s, dOut, In, grad, tokens, st);
    const int64_t rows = tokens * p.R;
    const int n_split = grad_splits(h, p, rows, h->bwd_partial_bytes);
    if (int64_t(n_split) * p.C * p.K * 4 > h->bwd_partial_bytes) return TN_ERR_UNSUPPORTED;
    GradArgs a;
    a.dOut = dOut;
    a.In = In;
    a.partial = h->bwd_partial;
    a.crow = s.crow;
    a.ccol = s.ccol;
    a.arow = s.arow;
    a.acol = s.acol;
    a.c_tok_stride = p.c_tok_stride;
    a.a_tok_stride = p.a_tok_stride;
    a.total_rows = uint32_t(rows);
    a.R = uint32_t(p.R);
    a.K = int32_t(p.K);
    a.C = int32_t(p.C);
    a.rows_per_split = uint32_t((rows + n_split - 1) / n_split);
    const bool mfma = grad_on_mfma(h, p);
    if (mfma) a.rows_per_split = (a.rows_per_split + 31u) & ~31u;        // the tile kernel's row ranges start at multiples of 32
    const GradModes gm = grad_modes(p);
    a.d_mode = gm.d;
    a.i_mode = gm.i;
    const int64_t edge = mfma ? 128 : 64;
    dim3 grid(uint32_t((p.C + edge - 1) / edge), uint32_t((p.K + edge - 1) / edge), uint32_t(n_split));
    if (grid.y > 65535) return TN_ERR_UNSUPPORTED;
    a.c_tiles = int32_t(grid.x);
    a.k_tiles = int32_t(grid.y);
    a.n_split = n_split;
    if (mfma) {
        const int64_t wgs = int64_t(grid.x) * grid.y * n_split;
        if (wgs > (int64_t(1) << 30)) return TN_ERR_UNSUPPORTED;
        hipLaunchKernelGGL(grad_param_mfma_kernel, dim3(uint32_t(wgs)), dim3(256), 0, st, a);
    }
    else if (h->elt == 2)
        hipLaunchKernelGGL(grad_param_kernel<bf16_t>, grid, dim3(256), 0, st, a);
    else
        hipLaunchKernelGGL(grad_param_kernel<float>, grid, dim3(256), 0, st, a);
    if (p.trace_extent > 1 && !accumulate)
        hipLaunchKernelGGL(grad_fill_kernel, dim3(uint32_t(std::min<int64_t>((grad_elems + 255) / 256, 4096))), dim3(256), 0, st,
                           grad, grad_elems);
    GradOutArgs o;
    memset(&o, 0, sizeof(o));
    o.partial = h->bwd_partial;
    o.grad = grad;
    o.C = uint32_t(p.C);
    o.K = uint32_t(p.K);
    o.ld = p.K;
    o.split_stride = p.C * p.K;
    o.n_split = n_split;
    o.accumulate = accumulate ? 1 : 0;
    fill_grad_dims(&o, p.cdims, p.kdims);
    o.trace_extent = p.trace_extent;
    o.trace_stride = p.trace_stride;
    return launch_grad_reduce(o, st);
}

// ---- the same gradients through dW ----
constexpr int64_t kGradMinTokens = 16;        // one token range is padded to 64
constexpr int64_t kMatrixTogetherBytes = int64_t(32) << 20;      // of a half's dH, twice, in two parts
constexpr int kGradSumsPad = 128;             // columns of the core gradients (a bond): padded to the narrow tiles

// bond_grad_kernel takes halves of two cores each (a half of one core has no low part, and the kernel reads both parts of both) over
// a bond of 32, 64 or 96 (its sums and its operand stay in registers); the columns are cut into as many ranges as leave the least to the
// busiest compute unit, at least 4 tiles each, the sums within kMaxGradPartialBytes.
bool plan_bond_grad(tn_linear_s* h, const tn::MatrixPlan& m, const tn::MatrixGrad& g) {
    const int64_t F0 = m.half[0].F, F1 = m.half[1].F, S = m.Kr;
    if (!g.half[0].pair || !g.half[1].pair || S % 32 || S > 96 || F0 % 64 || F1 % 64 || F1 > (int64_t(1) << 21) || F0 > (int64_t(1) << 24) ||
        F0 * F1 > (int64_t(1) << 29))      // 31-bit offsets in bytes
        return false;
    const int64_t panels = (F0 + kBondRows - 1) / kBondRows, tiles = F1 / kBondCols;
    int64_t best = 0;
    for (int64_t n = 1; n <= 64 && (n == 1 || 4 * n <= tiles); ++n) {
        const int64_t per = (tiles + n - 1) / n;
        if ((tiles + per - 1) / per != n) continue;                               // an empty range
        const int64_t bytes0 = (n * F0 * S * 4 + 255) & ~int64_t(255), bytes1 = (panels * F1 * S * 4 + 255) & ~int64_t(255);
        if (panels * n >= (int64_t(1) << 31) || bytes0 + bytes1 > kMaxGradPartialBytes) break;
        // a workgroup's start and end take about 8 tiles' time (4096 columns of 40 panels: 6 ranges 69 us, 32 ranges 95, before dW came in tiles)
        const int64_t cost = (panels * n + h->num_cus - 1) / h->num_cus * (per + 8);
        if (best && cost >= best) continue;
        best = cost;
        h->bond_ranges = int32_t(n);
        h->bond_tiles_per_range = int32_t(per);
        h->bond_sums_bytes[0] = bytes0;
        h->bond_sums_bytes[1] = bytes1;
    }
    return best > 0;
}

int launch_bond_grad(const tn_linear_s* h, const void* D, const void* P0, const void* P1, int64_t p0_lo, int64_t p1_lo, hipStream_t st) {
    BondGradArgs a;
    a.D = D;
    a.P0 = P0;
    a.P1 = P1;
    a.d_lo = h->plan.M * h->plan.N;
    a.p0_lo = p0_lo;
    a.p1_lo = p1_lo;
    a.sums0 = h->bwd_partial;
    a.sums1 = reinterpret_cast<float*>(reinterpret_cast<char*>(h->bwd_partial) + h->bond_sums_bytes[0]);
    a.F0 = h->mgrad_f[0];
    a.F1 = h->mgrad_f[1];
    a.S = int32_t(h->mgrad_half[0].dh.plan.C);
    a.tiles = int32_t(a.F1 / kBondCols);
    a.tiles_per_range = h->bond_tiles_per_range;
    a.ranges = h->bond_ranges;
    const dim3 grid(uint32_t((a.F0 + kBondRows - 1) / kBondRows * a.ranges));
    switch (a.S) {
        case 32: hipLaunchKernelGGL(bond_grad_kernel<1>, grid, dim3(256), BondGradShape<1>::SMEM, st, a); break;
        case 64: hipLaunchKernelGGL(bond_grad_kernel<2>, grid, dim3(256), BondGradShape<2>::SMEM, st, a); break;
        default: hipLaunchKernelGGL(bond_grad_kernel<3>, grid, dim3(256), BondGradShape<3>::SMEM, st, a); break;
    }
    return hipGetLastError() == hipSuccess ? TN_OK : TN_ERR_HIP;
}

// Decide whether gradients of many tokens go through dW, and prepare it. dW and dH are sums over the tokens and the products of
// two cores meet such a sum: they are kept in two parts each, as the caller gets fp32 (in one
// part, core gradients of the rank-64 train 5120 -> 8192 at 1024 tokens with a common component are 2.9e-3 off in the 2-norm, in
// two 5e-6; the steps, whose roundings average out over the tokens, leave 0.9 to 1.8e-4). The steps are priced at 0.35e9 FLOP per us and 40 us
// a step (train 5120 -> 8192 of rank 64: 9.7 ms at 1024 tokens; ring 25600 -> 5120 of rank 32: 12.5 ms at 64). Through dW / step by
// step in us at the first count that takes dW, and at 204 tokens, trains of rank 32, 64 and 96: 5120 -> 8192 129 / 206 at 40 tokens, 153 / 247 at
// 16, 191 / 362 at 16 (204: 140 / 668, 168 / 1893, 205 / 3725); 5120 -> 25600 344 / 639 at 102 (the first is 81), 367 / 429 at 24, 414 / 533 at 16;
// 25600 -> 5120 of rank 64 386 / 388 at 24; 5120 -> 1024 at 16: 84 / 150, 89 / 275, 99 / 261; rings at 16, by 1.6 times and more. At no count of 270 this order is the slower one where it is taken.
int prepare_matrix_grad(tn_linear_s* h, const tn_linear_desc* desc, hipStream_t st) {
    const int64_t M = h->plan.M, N = h->plan.N;
    if (h->plan.dtype != TN_DTYPE_BF16 || N % 64 || M % 8 || desc->max_tokens < kGradMinTokens ||
        (desc->flags & (TN_FLAG_SCALAR_KERNELS | TN_FLAG_NO_MERGE | TN_FLAG_NO_LAZY_MERGE)) ||
        ((desc->flags >> TN_FLAG_VARIANT_SHIFT) & 0xff) != 0)
        return TN_OK;
    const bool dense = h->plan.format == TN_FORMAT_DENSE;
    if (dense && (desc->flags & TN_FLAG_TRANSPOSE)) return TN_OK;
    const tn::MatrixPlan& m = h->matrix_plans.m;
    tn::MatrixGrad g;
    if (!dense) {
        if (!matrix_plan_of(h, desc)) return TN_OK;
        // dW in tiles where one pass over it gives both halves' gradients, as a matrix for the products
        h->mgrad_bond = tn::make_matrix_grad(h->matrix_plans.net, m, &g, true) && g.tiled && plan_bond_grad(h, m, g);
        if (!h->mgrad_bond) {
            g = tn::MatrixGrad();
            if (!tn::make_matrix_grad(h->matrix_plans.net, m, &g)) return TN_OK;
        }
    }
    auto step = [&](DevStep* s, int64_t R, int64_t K, int64_t C, int64_t out_elems, int pad) {
        s->plan.R = R;
        s->plan.K = K;
        s->plan.C = C;
        s->plan.c_tok_stride = out_elems;
        s->variant = VAR_GEMM;
        s->cmode = 1;
        s->Kp = int(K);
        s->Cp = round_up(int(C), pad);
    };
    if (M > (int64_t(1) << 24) || M * N > tn::kMatrixMaxElems) return TN_OK;
    step(&h->mgrad_dw, M, 64, N, M * N, tn::kMatrixColPad);
    // what a call moves beside its products, their times, and the memory it works in
    int64_t fixed = 0;
    auto room = [&](int i, int64_t elems) {
        h->mgrad_off[i] = fixed;
        fixed += (elems * 4 + 255) & ~int64_t(255);      // two parts
    };
    float us = 20.f;
    int64_t sums = 0;
    std::vector<int64_t> second;              // of the second half's dH and its transpose, where they may have room of their own
    if (!dense) {
        room(2, M * N);
        if (!h->mgrad_bond) room(3, M * N);
        h->mgrad_dw.out_lo = M * N;
        if (h->mgrad_bond)      // 51 us and 17 for the two launches that add the sums, of 168 MB in two parts and 59 MB of sums
            us += 12.f + float(M * N) * 4.f / 3.6e6f + float(h->bond_sums_bytes[0] + h->bond_sums_bytes[1]) / 5e6f;
        else us += 6.f + float(M * N) * 8.f / 3.5e6f;
        int64_t dh = 0, dht = 0;
        for (int i = 0; i < 2; ++i) {
            const tn::MatrixGradHalf& G = g.half[i];
            auto& H = h->mgrad_half[i];
            const int64_t F = m.half[i].F, Fo = m.half[1 - i].F;
            h->mgrad_f[i] = F;
            H.pair = G.pair;
            H.F1 = G.F1;
            H.F2 = G.F2;
            H.S = G.pair ? G.a.R : 0;
            H.out_a = G.out_a;
            H.out_b = G.out_b;
            step(&H.dh, F, Fo, m.Kr, F * m.Kr, G.pair ? tn::kMatrixColPad : kGradSumsPad);
            H.dh.a_lo = M * N;
            H.dh.b_lo = g.half[1 - i].pair ? g.half[1 - i].op.out_elems : 0;
            H.dh.out_lo = G.pair ? F * m.Kr : 0;
            if (!h->mgrad_bond) us += 3.f + std::max(gemm_choice(h, H.dh, F, kMaxGradPartialBytes).us, float(F * (Fo + m.Kr)) * 4.f / 3.5e6f);
            h->mgrad_flops += 2 * F * Fo * m.Kr * H.dh.segments();
            if (!G.pair) {
                sums = std::max(sums, F * H.dh.Cp * 4);
                continue;
            }
            if (F * m.Kr > tn::kMatrixMaxElems) return TN_OK;
            fill_product_step(&H.op.s, G.op);
            H.op.s.out_lo = G.op.out_elems;
            h->mgrad_flops += 2 * G.op.R * G.op.C * G.op.K + 2 * 2 * 2 * G.F1 * G.F2 * H.S;      // dA and dB, two parts of dH each
            us += product_us(h, H.op.s);
            room(4 + i, G.op.out_elems);
            dh = std::max(dh, G.F1 * G.F2);
            dht = std::max(dht, tn::detail::round64(G.F1) * G.F2);
            sums = std::max(sums, std::max(G.F1, G.F2) * round_up(int(H.S), kGradSumsPad) * 4);
            us += 46.f + float(G.F1 * G.F2) * 12.f / 3.5e6f;
        }
        room(6, dh);
        room(7, dht);
        // (a ring's dH may be as large as dW: one after the other then)
        if (h->mgrad_half[0].pair && h->mgrad_half[1].pair && (h->mgrad_bond || (dh + dht) * 4 <= kMatrixTogetherBytes)) second = {dh, dht};
    }
    // tokens per pass: X and dY transposed, tokens padded to 64
    const int64_t limit = desc->workspace_limit_bytes > 0 ? desc->workspace_limit_bytes : kDefaultWorkspaceBytes;
    const int64_t x_row = (N + tn::kMatrixColPad - 1) / tn::kMatrixColPad * tn::kMatrixColPad * 2, y_row = M * 2;
    auto tokens_in = [&](int64_t taken) {
        return std::min<int64_t>(grad_tokens_pad(desc->max_tokens), (limit - taken - 512) / (x_row + y_row) / 64 * 64);
    };
    const int64_t chunk = tokens_in(fixed);
    if (limit < fixed || chunk < 64) return TN_OK;
    // both halves' cores in shared launches (44 us of launches less) where the second half's room takes no tokens from a pass, each of
    // which moves dW again (rank-64 train 5120 -> 8192: 168 MB)
    const int64_t without = fixed;
    for (size_t i = 0; i < second.size(); ++i) room(8 + int(i), second[i]);
    h->mgrad_together = !second.empty() && tokens_in(fixed) == chunk;
    if (!h->mgrad_together) {
        fixed = without;
        h->mgrad_off[8] = h->mgrad_off[6];
        h->mgrad_off[9] = h->mgrad_off[7];
    }
    int64_t from = 0;
    const float flops = 3.f * float(h->plan.flops);
    for (int64_t t = kGradMinTokens; t <= desc->max_tokens && !from; t += t < 64 ? 8 : t / 8) {
        DevStep dw = h->mgrad_dw;
        dw.Kp = int(grad_tokens_pad(std::min(t, chunk)));
        const float product = std::max(gemm_choice(h, dw, M, 0).us, float(M * N) * 4.f / 3.5e6f);
        if (us + product + float(t) * float(M + N) * 4.f / 3.5e6f < float(t) * flops / 0.35e9f + 40.f * float(h->steps.size())) from = t;
    }
    if (!from) return TN_OK;
    h->mgrad_off[0] = fixed;
    h->mgrad_off[1] = fixed + ((chunk * x_row + 255) & ~int64_t(255));
    // tables, and the operands kept
    std::vector<int32_t> tab;
    auto put = [&](const std::vector<int32_t>& v) {
        const size_t at = tab.size();
        tab.insert(tab.end(), v.begin(), v.end());
        return at;
    };
    std::vector<std::pair<DevStep*, std::pair<size_t, size_t>>> where;
    auto tables_of = [&](DevStep* s, const std::vector<int32_t>& r, const std::vector<int32_t>& c) {
        const size_t ra = put(r);
        where.push_back({s, {ra, put(c)}});
    };
    if (!dense) {
        tables_of(&h->mgrad_dw, g.dw_row, g.dw_col);
        for (int i = 0; i < 2; ++i) {
            auto& H = h->mgrad_half[i];
            if (!H.pair) continue;          // its gradient is left as sums, which use no tables
            tables_of(&H.dh, g.half[i].row_off, g.half[i].col_off);
            tables_of(&H.op.s, g.half[i].op.row_off, g.half[i].op.col_off);
        }
    }
    void* tables = nullptr;
    if (hipMalloc(&tables, std::max<size_t>(1, tab.size()) * sizeof(int32_t)) != hipSuccess) return TN_ERR_ALLOC;
    h->mat_kept.push_back(tables);
    if (!tab.empty() && upload_tables(h, std::move(tab), tables, st) != TN_OK) return TN_ERR_HIP;
    for (auto& w : where) {
        w.first->crow = static_cast<const int32_t*>(tables) + w.second.first;
        w.first->ccol = static_cast<const int32_t*>(tables) + w.second.second;
    }
    for (int i = 0; i < 2 && !dense; ++i) {
        auto& H = h->mgrad_half[i];
        const tn::MatrixGradHalf& G = g.half[i];
        int rc;
        if (!H.pair) {
            rc = keep_operand(h, desc, G.op_keep, G.op_keep.K, true, &H.op.s.packed);
        } else {
            void* a = nullptr;
            rc = keep_operand(h, desc, G.op.a, G.op.Kp, false, &a);
            H.op.a = a;
            if (rc == TN_OK) rc = keep_operand(h, desc, G.op.b, G.op.Kp, true, &H.op.s.packed);
            if (rc == TN_OK) rc = keep_operand(h, desc, G.a, tn::detail::round64(G.F1), true, &H.a);
            if (rc == TN_OK) rc = keep_operand(h, desc, G.b, G.F2, true, &H.b);
        }
        if (rc != TN_OK) return rc;
    }
    h->mgrad = true;
    h->mgrad_min_tokens = from;
    h->mgrad_chunk = chunk;
    h->bwd_ws_bytes = h->mgrad_off[1] + chunk * y_row;
    if (dense) sums = M * h->mgrad_dw.Cp * 4;
    // (the large products' sums of K ranges, where there are such products)
    else sums = std::max(sums, std::min(kMaxGradPartialBytes, std::max(4 * sums, h->mgrad_bond ? kMaxPartialBytes / 4 : kMaxPartialBytes)));
    h->bwd_partial_bytes = sums + (h->mgrad_bond ? h->bond_sums_bytes[0] + h->bond_sums_bytes[1] : 0);
    return TN_OK;
}

GradOutArgs sums_out(const GemmSums& f, const tn::GradOut& out, int64_t rows, int64_t cols, float* grad, bool accumulate) {
    GradOutArgs o;
    memset(&o, 0, sizeof(o));
    o.partial = f.sums;
    o.grad = grad;
    o.C = uint32_t(rows);
    o.K = uint32_t(cols);
    o.ld = f.ld;
    o.split_stride = rows * f.ld;
    o.n_split = f.n_split;
    o.accumulate = accumulate ? 1 : 0;
    fill_grad_dims(&o, out.rows, out.cols);
    o.trace_extent = 1;
    return o;
}

// The gradients of the cores of halves `first` to `last`, from the halves' own in two parts: transposed copies for the second core of a
// pair, the products, and their sums put in place, a launch each (one after the other they were 12 launches of 4.6 us and up, on an
// idle chip: 66 us of a rank-64 train's 244, 22 so).
int core_gradients(const tn_linear_s* h, int first, int last, void* const* grads, void* part, int64_t part_bytes, bool add, hipStream_t st) {
    char* base = static_cast<char*>(h->bwd_ws);
    TransposeArgs turn[kTransposeMany];
    DevStep steps[kGemmMany];
    ProductJob jobs[kGemmMany];
    const tn::GradOut* outs[kGemmMany];
    float* to[kGemmMany];
    int turns = 0, n = 0;
    for (int i = first; i <= last; ++i) {
        const auto& H = h->mgrad_half[i];
        char *dh = base + h->mgrad_off[6 + 2 * i], *dht = base + h->mgrad_off[7 + 2 * i];
        const int64_t f1p = tn::detail::round64(H.F1);
        for (int side = 0; side < 2; ++side) {
            outs[n] = side == 0 ? &H.out_a : &H.out_b;
            to[n] = static_cast<float*>(grads[outs[n]->slot]);
            if (!to[n]) continue;
            if (side == 1)
                for (int p = 0; p < 2; ++p)      // the low part right after the high one
                    turn[turns++] = transpose_args(dh + p * H.F1 * H.F2 * 2, dht + p * H.F2 * f1p * 2, H.F1, H.F2, f1p, false);
            DevStep& s = steps[n];
            s.plan.R = side == 0 ? H.F1 : H.F2;
            s.plan.C = H.S;
            s.plan.K = side == 0 ? H.F2 : f1p;
            s.a_lo = side == 0 ? H.F1 * H.F2 : H.F2 * f1p;
            s.Kp = int(s.plan.K);
            s.Cp = round_up(int(H.S), kGradSumsPad);
            s.cmode = 1;
            s.variant = VAR_GEMM;
            jobs[n] = ProductJob{&s, side == 0 ? dh : dht, side == 0 ? H.b : H.a, nullptr, {}};
            ++n;
        }
    }
    if (turns) launch_transposes(turn, turns, st);
    // all at once where their sums have room beside each other and a launch can count their elements
    int64_t need = 0;
    bool together = true;
    for (int j = 0; j < n; ++j) {
        need += one_range_bytes(steps[j]);
        together = together && steps[j].plan.R * steps[j].plan.C < (int64_t(1) << 31);
    }
    together = together && need <= part_bytes;
    for (int j = 0; j < n; j += together ? n : 1) {
        const int rc = launch_products(h, jobs + j, together ? n : 1, true, part, part_bytes, st);
        if (rc != TN_OK) return rc;
        if (!together) {
            const int rr = launch_grad_reduce(sums_out(jobs[j].f32, *outs[j], steps[j].plan.R, steps[j].plan.C, to[j], add), st);
            if (rr != TN_OK) return rr;
        }
    }
    if (!together || n == 0) return TN_OK;
    GradOutMany m;
    memset(&m, 0, sizeof(m));
    for (int j = 0; j < n; ++j) m.o[j] = sums_out(jobs[j].f32, *outs[j], steps[j].plan.R, steps[j].plan.C, to[j], add);
    launch_grad_reduce_many(m, n, st);
    return hipGetLastError() == hipSuccess ? TN_OK : TN_ERR_HIP;
}

int matrix_gradients(tn_linear_s* h, const void* x, const void* dy, void* const* grads, int64_t tokens, hipStream_t st) {
    char* base = static_cast<char*>(h->bwd_ws);
    auto at = [&](int i) -> void* { return base + h->mgrad_off[i]; };
    const bool dense = h->plan.format == TN_FORMAT_DENSE;
    const int64_t M = h->plan.M, N = h->plan.N;
    // the sums of bond_grad_kernel come first, those of the products behind them
    const int64_t bond_bytes = h->mgrad_bond ? h->bond_sums_bytes[0] + h->bond_sums_bytes[1] : 0;
    void* part = reinterpret_cast<char*>(h->bwd_partial) + bond_bytes;
    const int64_t part_bytes = h->bwd_partial_bytes - bond_bytes;
    bool wanted[2] = {false, false};
    for (int i = 0; i < 2 && !dense; ++i) {
        const auto& H = h->mgrad_half[i];
        wanted[i] = grads[H.out_a.slot] || (H.pair && grads[H.out_b.slot]);
    }
    if (dense ? !grads[0] : !(wanted[0] || wanted[1])) return TN_OK;
    ProductJob ops[2];
    int n_ops = 0;
    for (int i = 0; i < 2 && !dense; ++i)
        if ((wanted[1 - i] || h->mgrad_bond) && h->mgrad_half[i].pair) {
            const DevProduct& op = h->mgrad_half[i].op;
            ops[n_ops++] = ProductJob{&op.s, op.a, op.s.packed, at(4 + i), {}};
        }
    {
        const int rc = launch_products(h, ops, n_ops, false, part, part_bytes, st);
        if (rc != TN_OK) return rc;
    }
    for (int64_t t0 = 0; t0 < tokens; t0 += h->mgrad_chunk) {
        const int64_t nt = std::min(h->mgrad_chunk, tokens - t0), tp = grad_tokens_pad(nt);
        const bool add = t0 > 0;
        const TransposeArgs acts[2] = {transpose_args(static_cast<const char*>(x) + t0 * N * h->elt, at(0), nt, N, tp, true),
                                       transpose_args(static_cast<const char*>(dy) + t0 * M * h->elt, at(1), nt, M, tp, false)};
        launch_transposes(acts, 2, st);
        DevStep dw = h->mgrad_dw;
        dw.plan.K = tp;
        dw.Kp = int(tp);
        int rc;
        if (dense) {
            // the gradient is dW: straight into the caller's tensor, or added to it from the sums of a later pass
            GemmSums f;
            const bool direct = !add && (reinterpret_cast<uintptr_t>(grads[0]) & 15) == 0;       // stored in pieces of 16 bytes
            if (direct) f = GemmSums{static_cast<float*>(grads[0]), N, 1};
            rc = launch_product_of(h, dw, at(1), at(0), nullptr, part, part_bytes, st, &f);
            if (rc == TN_OK && !direct) {
                tn::GradOut out;
                out.rows = {{M, N}};
                out.cols = {{N, 1}};
                rc = launch_grad_reduce(sums_out(f, out, M, N, static_cast<float*>(grads[0]), add), st);
            }
            if (rc != TN_OK) return rc;
            continue;
        }
        rc = launch_product_of(h, dw, at(1), at(0), at(2), part, part_bytes, st);
        if (rc != TN_OK) return rc;
        auto operand = [&](int i) -> const void* { return h->mgrad_half[i].pair ? at(4 + i) : h->mgrad_half[i].op.s.packed; };
        if (h->mgrad_bond) {
            // how far the low part of the operand made of a half is: known to the step that it is the column operand of
            rc = launch_bond_grad(h, at(2), at(4), at(5), h->mgrad_half[1].dh.b_lo, h->mgrad_half[0].dh.b_lo, st);
            if (rc != TN_OK) return rc;
        } else if (wanted[1]) {
            TransposeArgs parts[2];
            for (int p = 0; p < 2; ++p)
                parts[p] = transpose_args(static_cast<char*>(at(2)) + p * M * N * 2, static_cast<char*>(at(3)) + p * M * N * 2, h->mgrad_f[0],
                                          h->mgrad_f[1], h->mgrad_f[0], false);
            launch_transposes(parts, 2, st);
        }
        // one pass over dW: the sums of its ranges or row panels, in place and in two parts
        auto bond_sums = [&](int first, int last) {
            SplitReducePartsTwo two;
            memset(&two, 0, sizeof(two));
            int n = 0;
            int64_t most = 0;
            for (int i = first; i <= last; ++i) {
                if (!wanted[i]) continue;
                const auto& H = h->mgrad_half[i];
                SplitReduceParts& r = two.p[n++];
                r.a.Out = at(6 + 2 * i);
                r.a.crow = H.dh.crow;
                r.a.ccol = H.dh.ccol;
                r.a.total_rows = r.a.R = uint32_t(h->mgrad_f[i]);
                r.a.C = r.a.Cp = int32_t(H.dh.plan.C);
                r.partial = reinterpret_cast<const float*>(reinterpret_cast<const char*>(h->bwd_partial) + (i ? h->bond_sums_bytes[0] : 0));
                r.nsplit = i ? int((h->mgrad_f[0] + kBondRows - 1) / kBondRows) : h->bond_ranges;
                r.rows_pad = r.a.R;
                r.out_lo = H.dh.out_lo;
                most = std::max(most, h->mgrad_f[i] * H.dh.plan.C);
            }
            hipLaunchKernelGGL(step_split_reduce_parts_two_kernel, dim3(uint32_t(std::min<int64_t>((most + 255) / 256, 8192)), uint32_t(n)),
                               dim3(256), 0, st, two);
        };
        if (h->mgrad_bond && h->mgrad_together) bond_sums(0, 1);
        for (int i = 0; i < 2; ++i) {
            if (!wanted[i]) continue;
            const auto& H = h->mgrad_half[i];
            const void* op = operand(1 - i);
            if (!H.pair) {
                GemmSums f;
                rc = launch_product_of(h, H.dh, at(2 + i), op, nullptr, part, part_bytes, st, &f);
                if (rc == TN_OK)
                    rc = launch_grad_reduce(sums_out(f, H.out_a, h->mgrad_f[i], H.dh.plan.C, static_cast<float*>(grads[H.out_a.slot]), add), st);
                if (rc != TN_OK) return rc;
                continue;
            }
            if (!h->mgrad_bond) rc = launch_product_of(h, H.dh, at(2 + i), op, at(6 + 2 * i), part, part_bytes, st);
            else if (!h->mgrad_together) bond_sums(i, i);
            if (rc == TN_OK && !h->mgrad_together) rc = core_gradients(h, i, i, grads, part, part_bytes, add, st);
            if (rc != TN_OK) return rc;
        }
        if (h->mgrad_together) {
            rc = core_gradients(h, 0, 1, grads, part, part_bytes, add, st);
            if (rc != TN_OK) return rc;
        }
    }
    return hipGetLastError() == hipSuccess ? TN_OK : TN_ERR_HIP;
}

// Contract pairs of parameter tensors at create time (tn::MergeOp) with the plain FMA kernel
// (fp32 accumulate, one rounding to the storage type). `virt` receives one device buffer per merge;
// `temps` receives scratch buffers the caller frees once the stream has drained.
int materialise_merges(const tn::Plan& plan, const tn_linear_desc* desc, int elt, hipStream_t st,
                       std::vector<void*>* virt, std::vector<void*>* temps) {
    auto source = [&](int slot) -> const void* {
        return slot < plan.n_caller_tensors ? desc->tensors[slot] : (*virt)[size_t(slot - plan.n_caller_tensors)];
    };
    for (const tn::MergeOp& m : plan.merges) {
        void* out = nullptr;
        if (hipMalloc(&out, size_t(m.R * m.C) * elt) != hipSuccess) return TN_ERR_ALLOC;
        virt->push_back(out);
        int Kp = round_up(int(m.K), 64), Cp = round_up(int(m.C), 64);
        void* packed = nullptr;
        if (hipMalloc(&packed, size_t(Kp) * Cp * elt) != hipSuccess) return TN_ERR_ALLOC;
        temps->push_back(packed);
        PackArgs pa;
        memset(&pa, 0, sizeof(pa));
        pa.src = source(m.q_slot);
        pa.dst = packed;
        pa.K = int32_t(m.K);
        pa.Kp = Kp;
        pa.C = int32_t(m.C);
        pa.Cp = Cp;
        fill_pack_dims(&pa, m.kq, m.cdims);
        pa.trace_extent = 1;
        launch_pack(pa, elt, st);
        // tables: arow | acol | crow | ccol
        std::vector<int32_t> tab = gather_table(m.rdims, m.R);
        std::vector<int32_t> acol = gather_table(m.kp, m.K);
        tab.insert(tab.end(), acol.begin(), acol.end());
        for (int64_t r = 0; r < m.R; ++r) tab.push_back(int32_t(r * m.C));
        for (int64_t c = 0; c < m.C; ++c) tab.push_back(int32_t(c));
        int32_t* dtab = nullptr;
        if (hipMalloc(reinterpret_cast<void**>(&dtab), tab.size() * sizeof(int32_t)) != hipSuccess) return TN_ERR_ALLOC;
        temps->push_back(dtab);
        if (hipMemcpyAsync(dtab, tab.data(), tab.size() * sizeof(int32_t), hipMemcpyHostToDevice, st) != hipSuccess ||
            hipStreamSynchronize(st) != hipSuccess)
            return TN_ERR_HIP;
        StepArgs a;
        a.A = source(m.p_slot);
        a.B = packed;
        a.Out = out;
        a.arow = dtab;
        a.acol = dtab + m.R;
        a.crow = dtab + m.R + m.K;
        a.ccol = dtab + m.R + m.K + m.R;
        a.a_tok_stride = 0;
        a.c_tok_stride = 0;
        a.total_rows = uint32_t(m.R);
        a.R = uint32_t(m.R);
        a.K = int32_t(m.K);
        a.Kp = Kp;
        a.C = int32_t(m.C);
        a.Cp = Cp;
        dim3 grid(uint32_t((m.R + 63) / 64), uint32_t(Cp / 64));
        if (elt == 2)
            hipLaunchKernelGGL(step_scalar_kernel<bf16_t>, grid, dim3(256), 0, st, a);
        else
            hipLaunchKernelGGL(step_scalar_kernel<float>, grid, dim3(256), 0, st, a);
        if (hipGetLastError() != hipSuccess) return TN_ERR_HIP;
    }
    return TN_OK;
}

}  // namespace

extern "C" {

int tn_linear_version(void) { return 6; }

const char* tn_linear_strerror(int status) {
    switch (status) {
        case TN_OK: return "success";
        case TN_ERR_INVALID_ARG: return "invalid argument";
        case TN_ERR_UNSUPPORTED: return "unsupported configuration";
        case TN_ERR_ALLOC: return "allocation failed";
        case TN_ERR_HIP: return "HIP runtime error";
        case TN_ERR_SCRATCH: return "the call needs more scratch memory than the library's static buffer holds";
        default: return "unknown status";
    }
}

int tn_linear_plan_query(const tn_linear_desc* desc, int32_t what, int64_t* value) {
    if (!desc || !value) return TN_ERR_INVALID_ARG;
    tn::Plan p;
    int rc = tn::make_plan(desc, &p);
    if (rc != TN_OK) return rc;
    if (what == TN_QUERY_WORKSPACE_BYTES || what == TN_QUERY_CHUNK_TOKENS) {
        *value = 0;
        return TN_OK;
    }
    if (what == TN_QUERY_PACKED_BYTES) {
        int64_t elt = desc->dtype == TN_DTYPE_BF16 ? 2 : 4, total = 0;
        for (const auto& s : p.steps)
            total += int64_t(round_up(int(s.K), 64)) * round_up(int(s.C), 32) * elt;
        *value = total;   // lower bound: the tile width used for padding is chosen at create
        return TN_OK;
    }
    if (what >= TN_QUERY_STEP_BASE && (what - TN_QUERY_STEP_BASE) % 10 >= 5 &&
        (what - TN_QUERY_STEP_BASE) % 10 <= 6) {
        *value = 0;
        return TN_OK;
    }
    return plan_value(p, what, value);
}

int tn_linear_create(tn_linear_t* out, const tn_linear_desc* desc_in) {
    if (!out || !desc_in || !desc_in->tensors) return TN_ERR_INVALID_ARG;
    tn_linear_desc eff = *desc_in;             // the description create works with: tensors may be replaced below
    const tn_linear_desc* desc = &eff;
    std::vector<const void*> eff_tensors;
    if ((desc->flags & TN_FLAG_QUANT_MXFP4) && (desc->dtype != TN_DTYPE_BF16 || (desc->flags & TN_FLAG_TRAINABLE)))
        return TN_ERR_INVALID_ARG;
    tn_linear_s* h = new (std::nothrow) tn_linear_s;
    if (!h) return TN_ERR_ALLOC;
    int rc = tn::make_plan(desc, &h->plan);
    if (rc != TN_OK) {
        delete h;
        return rc;
    }
    for (int i = 0; i < desc->n_tensors; ++i)
        if (!desc->tensors[i]) {
            delete h;
            return TN_ERR_INVALID_ARG;
        }
    if (hipGetDevice(&h->device) != hipSuccess) {
        delete h;
        return TN_ERR_HIP;
    }
    {
        hipDeviceProp_t prop;
        if (hipGetDeviceProperties(&prop, h->device) != hipSuccess) {
            delete h;
            return TN_ERR_HIP;
        }
        if (strncmp(prop.gcnArchName, "gfx950", 6) != 0) {
            delete h;
            return TN_ERR_UNSUPPORTED;
        }
        h->num_cus = std::max(1, prop.multiProcessorCount);
        if (configure_kernels(h->device) != TN_OK) {
            delete h;
            return TN_ERR_HIP;
        }
    }
    hipStream_t st = static_cast<hipStream_t>(desc->stream);
    h->elt = desc->dtype == TN_DTYPE_BF16 ? 2 : 4;
    h->max_tokens = desc->max_tokens;
    h->flags = desc->flags;
    if (desc->flags & TN_FLAG_QUANT_MXFP4) {
        // quantise every tensor; everything below (merging, packing, lazily merged plans) sees the dequantised copies
        for (int i = 0; i < desc->n_tensors; ++i) {
            const int64_t n = tn::caller_tensor_elems(desc, i);
            void *codes = nullptr, *exps = nullptr, *deq = nullptr;
            if (n <= 0 || hipMalloc(&codes, size_t((n + 1) / 2)) != hipSuccess) {
                free_handle(h);
                return TN_ERR_ALLOC;
            }
            h->quant_codes.push_back(codes);
            if (hipMalloc(&exps, size_t((n + 31) / 32)) != hipSuccess) {
                free_handle(h);
                return TN_ERR_ALLOC;
            }
            h->quant_exps.push_back(exps);
            if (hipMalloc(&deq, size_t(n) * 2) != hipSuccess) {
                free_handle(h);
                return TN_ERR_ALLOC;
            }
            h->create_temps.push_back(deq);
            h->quant_elems.push_back(n);
            h->quant_bytes += (n + 1) / 2 + (n + 31) / 32;
            const int64_t blocks = (n + 31) / 32;
            hipLaunchKernelGGL(mxfp4_quantize_kernel, dim3(uint32_t(std::min<int64_t>((blocks + 255) / 256, 16384))), dim3(256), 0,
                               st, static_cast<const bf16_t*>(desc_in->tensors[i]), n, static_cast<unsigned char*>(codes),
                               static_cast<signed char*>(exps), static_cast<bf16_t*>(deq));
            eff_tensors.push_back(deq);
        }
        if (hipGetLastError() != hipSuccess) {
            (void)hipStreamSynchronize(st);
            free_handle(h);
            return TN_ERR_HIP;
        }
        eff.tensors = eff_tensors.data();
    }
    h->steps.resize(h->plan.steps.size());
    std::vector<void*> virt, temps;     // merged tensors and scratch: freed before create returns
    auto release_temps = [&]() {
        for (void* v : virt) (void)hipFree(v);
        for (void* v : temps) (void)hipFree(v);
    };
    rc = materialise_merges(h->plan, desc, h->elt, st, &virt, &temps);
    if (rc != TN_OK) {
        (void)hipStreamSynchronize(st);
        release_temps();
        free_handle(h);
        return rc;
    }
    // offset tables of every step (arow | acol | crow | ccol each): one allocation, one copy; the host copy
    // lives until create's final synchronisation
    std::vector<int32_t> host_tab;
    {
        std::vector<size_t> tab_off(h->steps.size());
        for (size_t i = 0; i < h->steps.size(); ++i) {
            DevStep& s = h->steps[i];
            s.plan = h->plan.steps[i];
            s.no_skinny = (desc->flags & TN_FLAG_NO_SKINNY) != 0;
            choose_variant(h, &s, desc->flags);
            const tn::Step& p = s.plan;
            tab_off[i] = host_tab.size();
            host_tab.insert(host_tab.end(), p.arow.begin(), p.arow.end());
            host_tab.insert(host_tab.end(), p.acol.begin(), p.acol.end());
            host_tab.insert(host_tab.end(), p.crow.begin(), p.crow.end());
            host_tab.insert(host_tab.end(), p.ccol.begin(), p.ccol.end());
        }
        if (hipMalloc(reinterpret_cast<void**>(&h->tables), std::max<size_t>(1, host_tab.size()) * sizeof(int32_t)) != hipSuccess ||
            hipMemcpyAsync(h->tables, host_tab.data(), host_tab.size() * sizeof(int32_t), hipMemcpyHostToDevice, st) != hipSuccess) {
            (void)hipStreamSynchronize(st);
            release_temps();
            free_handle(h);
            return TN_ERR_ALLOC;
        }
        for (size_t i = 0; i < h->steps.size(); ++i) {
            DevStep& s = h->steps[i];
            const tn::Step& p = s.plan;
            const int32_t* t = h->tables + tab_off[i];
            if (!p.a_plain) {
                s.arow = t;
                s.acol = t + p.arow.size();
            }
            s.crow = t + p.arow.size() + p.acol.size();
            s.ccol = s.crow + p.crow.size();
        }
    }
    for (size_t i = 0; i < h->steps.size(); ++i) {
        DevStep& s = h->steps[i];
        const tn::Step& p = s.plan;
        // packed parameter tensor
        int64_t bytes = int64_t(s.Cp) * s.Kp * h->elt;
        if (hipMalloc(&s.packed, size_t(bytes)) != hipSuccess) {
            (void)hipStreamSynchronize(st);
            release_temps();
            free_handle(h);
            return TN_ERR_ALLOC;
        }
        h->packed_bytes += bytes;
        PackArgs pa;
        memset(&pa, 0, sizeof(pa));
        pa.src = p.slot < h->plan.n_caller_tensors ? desc->tensors[p.slot]
                                                    : virt[size_t(p.slot - h->plan.n_caller_tensors)];
        pa.dst = s.packed;
        pa.K = int32_t(p.K);
        pa.Kp = s.Kp;
        pa.C = int32_t(p.C);
        pa.Cp = s.Cp;
        fill_pack_dims(&pa, p.kdims, p.cdims);
        pa.trace_extent = p.trace_extent;
        pa.trace_stride = p.trace_stride;
        launch_pack(pa, h->elt, st);
        if (hipGetLastError() != hipSuccess) {
            (void)hipStreamSynchronize(st);
            release_temps();
            free_handle(h);
            return TN_ERR_HIP;
        }
    }
    if (!virt.empty() || !temps.empty()) {
        // the pack kernels read the merged tensors: wait for them before the buffers go away
        if (hipStreamSynchronize(st) != hipSuccess) {
            release_temps();
            free_handle(h);
            return TN_ERR_HIP;
        }
        release_temps();
    }
    rc = plan_small_chain(h, st);
    if (rc == TN_OK) rc = prepare_pair(h, st);
    if (rc == TN_OK) rc = prepare_kron(h, st);
    if (rc == TN_OK) rc = plan_chain2(h, st);
    if (rc == TN_OK) rc = prepare_q4_stream(h, st);
    if (rc == TN_OK) {
        const int64_t before = h->packed_bytes;
        rc = prepare_lazy(h, desc, st);
        if (rc == TN_OK) rc = prepare_direct(h, desc, st);
        if (rc == TN_OK) rc = write_operands(h, st);
        h->lazy_kept_bytes = h->packed_bytes - before;
    }
    if (rc == TN_OK) {
        const int64_t before = h->packed_bytes;
        rc = prepare_matrix(h, desc, st);
        if (rc == TN_OK) rc = write_operands(h, st);
        h->create_sources.clear();
        h->mat_kept_count = h->mat_kept.size();
        h->mat_kept_bytes = h->packed_bytes - before;
        if (rc == TN_OK && h->matrix && !desc->workspace && hipMalloc(&h->mat_mem, size_t(h->mat_bytes)) != hipSuccess) {
            h->mat_mem = nullptr;
            rc = TN_ERR_ALLOC;
        }
        if (rc == TN_ERR_ALLOC) rc = drop_matrix(h, st);      // an order less, not a layer less
    }
    if (rc == TN_OK && (desc->flags & TN_FLAG_TRAINABLE)) {
        rc = prepare_matrix_grad(h, desc, st);
        if (rc == TN_OK) rc = write_operands(h, st);
        if (rc == TN_OK) rc = prepare_backward(h, desc, st);
    }
    if (rc != TN_OK) {
        (void)hipStreamSynchronize(st);
        free_handle(h);
        return rc;
    }
    // workspace: two ping-pong buffers, each chunk_tokens * max_intermediate elements, and the
    // partial-sum buffer of the split-K kernel; allocated here, or carved out of the caller's block
    int64_t per_token = h->plan.max_intermediate * h->elt;
    if (h->kron && h->kron_min_tokens <= 1) per_token = 0;      // every call runs the one-launch kernel: no intermediates
    if (h->pair && h->pair_min_tokens <= 1) per_token = 0;
    int64_t max_r = 1;
    for (const auto& s : h->steps) max_r = std::max(max_r, s.plan.R);
    const int64_t row_cap = ((int64_t(1) << 31) - 1024) / max_r;      // rows of a pass are indexed with 32 bits
    const bool split_ok = !(desc->flags & TN_FLAG_NO_SPLIT_K) && h->elt == 2;
    auto step_need = [&](const DevStep& s, int64_t chunk) {
        int64_t need = 0;
        for (int64_t t = 1; t <= chunk; ++t) {
            if (t * s.plan.R >= kGemmMinRows && gemm_fits(s) && s.cmode != 0) break;
            SplitCfg c = split_config(s, t * s.plan.R);
            if (!c.use) break;          // larger passes only add tiles
            need = std::max(need, c.partial_bytes);
        }
        // the matrix-product kernel takes as many K ranges as the buffer has room for: sized for row counts up to where
        // the tiles alone fill the chip
        if (gemm_fits(s))
            for (int64_t t = 1; t <= chunk && t * s.plan.R <= 8192; t += std::max<int64_t>(1, t / 8))
                if (t * s.plan.R >= kGemmMinRows) need = std::max(need, gemm_choice(h, s, t * s.plan.R, kMaxPartialBytes).partial_bytes);
        return need;
    };
    auto partial_need = [&](int64_t chunk) {
        int64_t need = 0;
        if (!split_ok) return need;
        // a backward pass runs its steps, both ways, with the same buffer
        for (size_t i = 0; h->trainable && i < h->steps.size(); ++i)
            need = std::max({need, step_need(h->steps[i], h->bwd_chunk), i > 0 ? step_need(h->bwd[i], h->bwd_chunk) : 0});
        if (h->matrix)
            for (int64_t t = h->mat_ranges.front().first; t <= std::min<int64_t>(h->max_tokens, 4096); t += std::max<int64_t>(1, t / 8))
                need = std::max(need, gemm_choice(h, h->mat_y, t, kMaxPartialBytes).partial_bytes);
        if (h->kron) {
            for (int64_t t = 1; t <= std::min<int64_t>(h->max_tokens, 4 * int64_t(h->num_cus)); ++t)
                need = std::max(need, kron_geometry(h, h->kron_dims, t, kMaxPartialBytes).partial_bytes);
            if (h->kron_min_tokens <= 1) return need;
        }
        if (h->pair) {
            for (int64_t t = h->pair_min_tokens; t <= std::min<int64_t>(h->max_tokens, 32 * int64_t(h->num_cus)); ++t)
                need = std::max(need, pair_geometry(h, t, kMaxPartialBytes).partial_bytes);
            if (h->pair_min_tokens <= 1) return need;
        }
        if (h->lazy)
            for (int64_t t = h->lazy_min_tokens; t <= std::min<int64_t>(h->max_tokens, 4 * int64_t(h->num_cus)); ++t)
                need = std::max(need, kron_geometry(h, h->lazy_dims, t, kMaxPartialBytes).partial_bytes);
        for (int64_t t = 1; h->direct && t <= std::min(h->max_tokens, kDirectMaxTokens); ++t)
            need = std::max(need, direct_geometry(h, t, kMaxPartialBytes).partial_bytes);
        if (!h->trainable || chunk > h->bwd_chunk)
            for (const auto& s : h->steps) need = std::max(need, step_need(s, chunk));
        return need;
    };
    // a lazily merged plan needs room for its slices: in the caller's block they share the space of the two
    // buffers (never in use at the same time), otherwise they get an allocation of their own
    if (h->lazy) {
        const int64_t room = desc->workspace
                                 ? desc->workspace_bytes - (split_ok ? std::min<int64_t>(kMaxPartialBytes, desc->workspace_bytes / 4) : 0) - 512
                                 : (desc->workspace_limit_bytes > 0 ? desc->workspace_limit_bytes : kDefaultWorkspaceBytes);
        if (room < h->lazy_slice_bytes) {
            // no room for the slices: every call runs the compact steps, and what the lazy plan kept goes away
            // (the kernels that wrote these buffers may still be running on the stream)
            if (hipStreamSynchronize(st) != hipSuccess) {
                free_handle(h);
                return TN_ERR_HIP;
            }
            h->lazy = h->direct = false;
            h->packed_bytes -= h->lazy_kept_bytes;
            h->lazy_kept_bytes = 0;
            for (void* v : h->lazy_sources) (void)hipFree(v);
            h->lazy_sources.clear();
            for (int w = 0; w < 2; ++w)
                if (h->lazy_gen_tables[w]) {
                    (void)hipFree(h->lazy_gen_tables[w]);
                    h->lazy_gen_tables[w] = nullptr;
                    h->lazy_mfma[w] = false;
                }
            if (h->lazy_tables) (void)hipFree(h->lazy_tables);
            h->lazy_tables = nullptr;
        }
    }
    // with the chained pair kernel or a lazily merged plan only calls below the token threshold use the buffers
    int64_t ws_tokens = h->pair ? std::min<int64_t>(h->max_tokens, h->pair_min_tokens - 1) : h->max_tokens;
    // (one token's buffers stay: calls that may not use the rebuilt plan - profiled steps, the entry point that
    // allocates nothing - run the compact steps token by token)
    if (h->lazy) ws_tokens = std::min<int64_t>(ws_tokens, std::max<int64_t>(1, h->lazy_min_tokens - 1));
    if (h->matrix) {
        // between the ranges a call runs in one launch (the pair or the Kronecker-sum kernel); a layer without one has no such gaps
        if (!h->pair && !h->kron && !h->lazy) h->mat_ranges = {{h->mat_ranges.back().first, kMatrixNoEnd}};
        ws_tokens = std::min<int64_t>(ws_tokens, std::max<int64_t>(1, h->mat_ranges.front().first - 1));
    }
    int64_t chunk = ws_tokens;
    if (desc->workspace) {
        // caller-owned block: [partial sums | buffer 0 | buffer 1], 256-byte aligned pieces
        h->owns_workspace = false;
        char* base = static_cast<char*>(desc->workspace);
        int64_t avail = desc->workspace_bytes;
        int64_t part = split_ok ? std::min<int64_t>(kMaxPartialBytes, avail / 4) & ~int64_t(255) : 0;
        int64_t half = ((avail - part) / 2) & ~int64_t(255);
        if (per_token > 0) {
            chunk = std::min<int64_t>(std::min<int64_t>(ws_tokens, half / per_token), row_cap);
            if (chunk < 1) {
                free_handle(h);
                return TN_ERR_INVALID_ARG;      // the block cannot hold one token's intermediates
            }
            h->ws[0] = base + part;
            h->ws[1] = base + part + half;
        } else {
            chunk = std::max<int64_t>(1, std::min<int64_t>(chunk, row_cap));
        }
        if (part > 0) {
            h->partial = base;
            h->partial_bytes = part;
        }
        if (h->lazy) h->lazy_slices = base + part;
        if (h->matrix) place_matrix(h, base + part);
        h->workspace_bytes = 0;
    } else {
        int64_t limit = desc->workspace_limit_bytes > 0 ? desc->workspace_limit_bytes : kDefaultWorkspaceBytes;
        if (h->matrix) {
            place_matrix(h, h->mat_mem);
            h->workspace_bytes += h->mat_bytes;
            limit -= h->mat_bytes;
        }
        if (per_token > 0) {
            chunk = std::max<int64_t>(1, std::min<int64_t>(ws_tokens, limit / (2 * per_token)));
            chunk = std::max<int64_t>(1, std::min<int64_t>(chunk, row_cap));
            for (int b = 0; b < 2; ++b) {
                if (hipMalloc(&h->ws[b], size_t(chunk * per_token)) != hipSuccess) {
                    free_handle(h);
                    return TN_ERR_ALLOC;
                }
            }
            h->workspace_bytes += 2 * chunk * per_token;
        } else {
            chunk = std::max<int64_t>(1, std::min<int64_t>(chunk, row_cap));
        }
        int64_t need = partial_need(chunk);
        if (need > 0) {
            if (hipMalloc(&h->partial, size_t(need)) != hipSuccess) {
                free_handle(h);
                return TN_ERR_ALLOC;
            }
            h->partial_bytes = need;
            h->workspace_bytes += need;
        }
        if (h->lazy) {
            if (hipMalloc(&h->lazy_slices, size_t(h->lazy_slice_bytes)) != hipSuccess) {
                free_handle(h);
                return TN_ERR_ALLOC;
            }
            h->workspace_bytes += h->lazy_slice_bytes;
        }
    }
    for (int w = 0; w < 2 && h->lazy; ++w) {
        h->lazy_gen[w].dst = static_cast<char*>(h->lazy_slices) + (w == 0 ? 0 : h->lazy_h1_offset);
        h->lazy_gen_mfma[w].dst = h->lazy_gen[w].dst;
        h->lazy_half[w].out = h->lazy_gen[w].dst;
    }
    h->chunk_tokens = chunk;
    if (h->lazy && h->owns_workspace) {
        // the handle's own workspace: nobody else writes the slices, so they are built here once and every call
        // finds them (a layer that shares a caller's block rebuilds them per call instead)
        rc = launch_lazy_generate(h, st);
        if (rc != TN_OK) {
            (void)hipStreamSynchronize(st);
            free_handle(h);
            return rc;
        }
        h->lazy_slices_kept = true;
    }
    price_direct(h);
    {
        std::vector<int> fuse(h->steps.size(), 0);
        for (size_t i = 0; i < h->steps.size(); ++i) fuse[i] = h->steps[i].fuse_next ? 1 : 0;
        h->schedule = tn::launch_schedule(h->steps.size(), fuse);
    }
    // everything create enqueued (repacking, table uploads) is done before the handle is handed out, so
    // that a forward on any stream may follow without further ordering
    if (hipStreamSynchronize(st) != hipSuccess) {
        free_handle(h);
        return TN_ERR_HIP;
    }
    for (void* v : h->create_temps) (void)hipFree(v);
    h->create_temps.clear();
    h->create_tables = {};
    h->create_sources = {};
    h->matrix_plans = {};
    *out = h;
    return TN_OK;
}

}  // extern "C"

namespace {

// Brackets one launch with a pair of HIP events when the handle is being profiled.
struct ProfScope {
    tn_linear_s* h;
    hipStream_t st;
    tn_linear_s::ProfRec rec;
    bool ok = true;
    ProfScope(tn_linear_s* handle, int step, hipStream_t stream) : h(handle), st(stream), rec{step, nullptr, nullptr} {
        if (!h->profiling) return;
        ok = hipEventCreate(&rec.start) == hipSuccess && hipEventCreate(&rec.stop) == hipSuccess;
        if (ok) (void)hipEventRecord(rec.start, st);
    }
    void done() {
        if (!h->profiling || !ok) return;
        (void)hipEventRecord(rec.stop, st);
        h->prof.push_back(rec);
    }
};

// One forward call in the workspace `w`. allow_lazy: calls large enough may run on the lazily merged plan,
// whose slices live in the handle's own workspace.
int forward_in(tn_linear_s* h, const Workspace& w, bool allow_lazy, const void* x, void* y, int64_t tokens,
               hipStream_t st) {
    const char* xb = static_cast<const char*>(x);
    char* yb = static_cast<char*>(y);
    if (h->small_chain && (h->elt == 4 || tokens <= kSmallChainMaxBf16Tokens)) {
        // every step in one launch, tensors and intermediates in LDS
        const int64_t pass = int64_t(1) << 24;
        for (int64_t t0 = 0; t0 < tokens; t0 += pass) {
            int64_t nt = std::min(pass, tokens - t0);
            ProfScope prof(h, 0, st);
            if (!prof.ok) return TN_ERR_HIP;
            int rc = launch_small_chain(h, xb + t0 * h->plan.N * h->elt, yb + t0 * h->plan.M * h->elt, nt, st);
            prof.done();
            if (rc != TN_OK) return rc;
        }
        return TN_OK;
    }
    if (allow_lazy && takes_matrix(h, tokens)) {
        int rc = launch_matrix_build(h, w.partial, w.partial_bytes, st);          // not part of the profiled launch
        const int64_t pass = int64_t(1) << 20;
        for (int64_t t0 = 0; t0 < tokens && rc == TN_OK; t0 += pass) {
            ProfScope prof(h, 0, st);
            if (!prof.ok) return TN_ERR_HIP;
            rc = launch_matrix_y(h, xb + t0 * h->plan.N * h->elt, yb + t0 * h->plan.M * h->elt, std::min(pass, tokens - t0), w.partial,
                                 w.partial_bytes, st);
            prof.done();
        }
        return rc;
    }
    const bool use_pair = h->pair && tokens >= h->pair_min_tokens;
    const bool use_kron = h->kron && tokens >= h->kron_min_tokens;
    const bool use_lazy = allow_lazy && h->lazy && tokens >= h->lazy_min_tokens;
    if (use_lazy && !use_pair && !use_kron && tokens <= kDirectMaxTokens && h->direct_geom[tokens].taken) {
        ProfScope prof(h, 0, st);
        if (!prof.ok) return TN_ERR_HIP;
        const int rc = launch_direct(h, w, h->direct_geom[tokens], x, y, tokens, st);
        prof.done();
        return rc;
    }
    if (use_pair || use_kron || use_lazy) {
        // both steps in one launch, no intermediate in memory; passes only bound the 32-bit token index
        // (and, for the Kronecker-sum kernel, keep a call's partial sums within their buffer)
        const int64_t pass = use_pair ? int64_t(1) << 24 : int64_t(1) << 20;
        if (!use_pair && !use_kron && !h->lazy_slices_kept) {
            // a caller's block is shared with other layers: whatever it held is gone
            int rc = launch_lazy_generate(h, st);          // not part of the profiled launch: a kernel of its own
            if (rc != TN_OK) return rc;
        }
        for (int64_t t0 = 0; t0 < tokens; t0 += pass) {
            int64_t nt = std::min(pass, tokens - t0);
            ProfScope prof(h, 0, st);
            if (!prof.ok) return TN_ERR_HIP;
            const void* xp = xb + t0 * h->plan.N * h->elt;
            void* yp = yb + t0 * h->plan.M * h->elt;
            int rc = use_pair ? launch_pair(h, w, xp, yp, nt, st)
                              : (use_kron ? launch_kron_eager(h, w, xp, yp, nt, st) : launch_kron_lazy(h, w, xp, yp, nt, st));
            prof.done();
            if (rc != TN_OK) return rc;
        }
        return TN_OK;
    }
    if (w.chunk_tokens < 1) return TN_ERR_INVALID_ARG;
    for (int64_t t0 = 0; t0 < tokens; t0 += w.chunk_tokens) {
        int64_t nt = std::min(w.chunk_tokens, tokens - t0);
        for (size_t li = 0; li < h->schedule.size(); ++li) {
            const tn::LaunchIO& l = h->schedule[li];
            const void* A = l.in == tn::kBufX ? static_cast<const void*>(xb + t0 * h->plan.N * h->elt) : w.ws[l.in];
            void* Out = l.out == tn::kBufY ? static_cast<void*>(yb + t0 * h->plan.M * h->elt) : w.ws[l.out];
            ProfScope prof(h, l.first, st);
            if (!prof.ok) return TN_ERR_HIP;
            const DevStep& s = h->steps[size_t(l.first)];
            int rc;
            if (l.steps == 2 && li + 1 < h->schedule.size() && h->schedule[li + 1].steps == 1 &&
                chain2_split_applies(h, s, h->steps[size_t(l.first) + 2], nt)) {
                // few tokens: the pair and the wide step after it in one launch, the pair's result in LDS
                const tn::LaunchIO& l2 = h->schedule[li + 1];
                void* Out2 = l2.out == tn::kBufY ? static_cast<void*>(yb + t0 * h->plan.M * h->elt) : w.ws[l2.out];
                const Chain2SplitArgs fa = chain2_split_args(s, h->steps[size_t(l.first) + 1], h->steps[size_t(l.first) + 2], A, Out2, nt);
                rc = launch_chain2_split(h, &fa, nullptr, st);
                ++li;
            } else {
                rc = l.steps == 2 ? launch_chain2(h, s, h->steps[size_t(l.first) + 1], A, Out, nt, st)
                                  : launch_step(h, w, s, A, Out, nt, st);
            }
            prof.done();
            if (rc != TN_OK) return rc;
        }
    }
    return TN_OK;
}

}  // namespace

extern "C" {

// the kernels read and write rows of activations in 16-byte pieces
static bool aligned16(const void* p) { return (reinterpret_cast<uintptr_t>(p) & 15) == 0; }

int tn_linear_forward(tn_linear_t h, const void* x, void* y, int64_t tokens, void* stream) {
    if (!h || tokens < 0) return TN_ERR_INVALID_ARG;
    if (tokens == 0) return TN_OK;
    if (!x || !y || !aligned16(x) || !aligned16(y)) return TN_ERR_INVALID_ARG;
    Workspace w;
    w.ws[0] = h->ws[0];
    w.ws[1] = h->ws[1];
    w.partial = h->partial;
    w.partial_bytes = h->partial_bytes;
    w.chunk_tokens = h->chunk_tokens;
    return forward_in(h, w, true, x, y, tokens, static_cast<hipStream_t>(stream));
}

int tn_linear_forward2(tn_linear_t ha, tn_linear_t hb, const void* x, void* ya, void* yb, int64_t tokens, void* stream) {
    if (!ha || !hb || tokens < 0) return TN_ERR_INVALID_ARG;
    if (ha->elt != hb->elt || ha->plan.N != hb->plan.N) return TN_ERR_INVALID_ARG;
    if (tokens == 0) return TN_OK;
    if (!x || !ya || !yb || !aligned16(x) || !aligned16(ya) || !aligned16(yb)) return TN_ERR_INVALID_ARG;
    hipStream_t st = static_cast<hipStream_t>(stream);
    // Launch by launch in step when the two layers have the same launch structure and the call is one pass of
    // the per-step path for both: where a launch of the decode-size kernels serves both layers, it does.
    auto per_step_path = [&](const tn_linear_s* h) {
        return !h->profiling && !(h->small_chain && (h->elt == 4 || tokens <= kSmallChainMaxBf16Tokens)) &&
               !(h->pair && tokens >= h->pair_min_tokens) && !(h->kron && tokens >= h->kron_min_tokens) &&
               !(h->lazy && tokens >= h->lazy_min_tokens) && !takes_matrix(h, tokens) && tokens <= h->chunk_tokens;
    };
    bool together = ha != hb && per_step_path(ha) && per_step_path(hb) && ha->schedule.size() == hb->schedule.size();
    for (size_t li = 0; together && li < ha->schedule.size(); ++li) {
        const tn::LaunchIO &la = ha->schedule[li], &lb = hb->schedule[li];
        if (la.first != lb.first || la.steps != lb.steps) together = false;
        else if (la.steps == 2 && (ha->steps[size_t(la.first)].chain_cfg != hb->steps[size_t(lb.first)].chain_cfg ||
                                   ha->steps[size_t(la.first)].chain_run_c1 != hb->steps[size_t(lb.first)].chain_run_c1))
            together = false;
    }
    if (!together) {
        int rc = tn_linear_forward(ha, x, ya, tokens, stream);
        return rc != TN_OK ? rc : tn_linear_forward(hb, x, yb, tokens, stream);
    }
    tn_linear_s* hs[2] = {ha, hb};
    void* ys[2] = {ya, yb};
    Workspace ws[2];
    for (int n = 0; n < 2; ++n) {
        ws[n].ws[0] = hs[n]->ws[0];
        ws[n].ws[1] = hs[n]->ws[1];
        ws[n].partial = hs[n]->partial;
        ws[n].partial_bytes = hs[n]->partial_bytes;
        ws[n].chunk_tokens = hs[n]->chunk_tokens;
    }
    auto buffer = [&](int n, int id) -> void* {
        return id == tn::kBufX ? const_cast<void*>(x) : (id == tn::kBufY ? ys[n] : ws[n].ws[id]);
    };
    // Each layer takes the launches tn_linear_forward would give it (so that its result has the same bits); where both
    // take the same decode-size kernel at the same point of the chain, one launch serves both.
    bool skip[2] = {false, false};                 // the layer's launch at this index ran inside its previous, fused one
    for (size_t li = 0; li < ha->schedule.size(); ++li) {
        const tn::LaunchIO& l = ha->schedule[li];
        const size_t f = size_t(l.first);
        const bool has_next = li + 1 < ha->schedule.size() && ha->schedule[li + 1].steps == 1;
        int rc = TN_OK;
        bool fuse[2];
        Chain2SplitArgs fa[2];
        for (int n = 0; n < 2; ++n) {
            fuse[n] = !skip[n] && l.steps == 2 && has_next &&
                      chain2_split_applies(hs[n], hs[n]->steps[f], hs[n]->steps[f + 2], tokens);
            if (fuse[n])
                fa[n] = chain2_split_args(hs[n]->steps[f], hs[n]->steps[f + 1], hs[n]->steps[f + 2],
                                          buffer(n, hs[n]->schedule[li].in), buffer(n, hs[n]->schedule[li + 1].out), tokens);
        }
        if (fuse[0] && fuse[1] && fa[0].kern == fa[1].kern) {
            rc = launch_chain2_split(ha, &fa[0], &fa[1], st);          // pair and wide step of both layers in one launch
            skip[0] = skip[1] = true;
        } else if (!skip[0] && !skip[1] && !fuse[0] && !fuse[1] && l.steps == 2 && factor_pair_applies(ha->steps[f], tokens) &&
                   factor_pair_applies(hb->steps[f], tokens) && ha->steps[f].pair_cfg == hb->steps[f].pair_cfg) {
            FactorPairArgs pa[2];
            for (int n = 0; n < 2; ++n)
                pa[n] = factor_pair_args(hs[n]->steps[f], hs[n]->steps[f + 1], buffer(n, hs[n]->schedule[li].in), buffer(n, hs[n]->schedule[li].out), tokens);
            rc = launch_factor_pair(ha, ha->steps[f].pair_cfg, pa[0], &pa[1], st);
        } else if (!skip[0] && !skip[1] && !fuse[0] && !fuse[1] && l.steps == 2 &&
                   chain2_small_applies(ha, ha->steps[f], tokens) && chain2_small_applies(hb, hb->steps[f], tokens)) {
            Chain2Args ca[2];
            for (int n = 0; n < 2; ++n)
                ca[n] = chain2_args(hs[n]->steps[f], hs[n]->steps[f + 1], buffer(n, hs[n]->schedule[li].in),
                                    buffer(n, hs[n]->schedule[li].out), tokens);
            rc = launch_chain2_small(ha->steps[f], ca[0], &ca[1], st);
        } else {
            for (int n = 0; n < 2 && rc == TN_OK; ++n) {
                if (skip[n]) {
                    skip[n] = false;
                    continue;
                }
                if (fuse[n]) {                     // e.g. only this layer qualifies, or only one streams its 4-bit form
                    rc = launch_chain2_split(hs[n], &fa[n], nullptr, st);
                    skip[n] = true;
                    continue;
                }
                const tn::LaunchIO& ln = hs[n]->schedule[li];
                const DevStep& s = hs[n]->steps[f];
                rc = ln.steps == 2 ? launch_chain2(hs[n], s, hs[n]->steps[f + 1], buffer(n, ln.in), buffer(n, ln.out), tokens, st)
                                   : launch_step(hs[n], ws[n], s, buffer(n, ln.in), buffer(n, ln.out), tokens, st);
            }
        }
        if (rc != TN_OK) return rc;
    }
    return TN_OK;
}

int tn_linear_param_gradients(tn_linear_t h, const void* x, const void* dy, void* const* grads, int64_t tokens,
                              void* stream) {
    if (!h || tokens < 0 || !grads || !h->trainable) return TN_ERR_INVALID_ARG;
    if (tokens == 0) return TN_OK;
    if (!x || !dy || !aligned16(x) || !aligned16(dy)) return TN_ERR_INVALID_ARG;
    hipStream_t st = static_cast<hipStream_t>(stream);
    if (h->mgrad && tokens >= h->mgrad_min_tokens) return matrix_gradients(h, x, dy, grads, tokens, st);
    const size_t n = h->steps.size();
    Workspace w;                                   // the forward workspace serves the split-K partial sums
    w.partial = h->partial;
    w.partial_bytes = h->partial_bytes;
    w.chunk_tokens = h->bwd_chunk;
    char* base = static_cast<char*>(h->bwd_ws);
    const int64_t dbuf = (h->plan.max_intermediate + 127) & ~int64_t(127);
    void* dbufs[2] = {base + h->bwd_chunk * h->bwd_saved_elems * h->elt,
                      base + h->bwd_chunk * (h->bwd_saved_elems + dbuf) * h->elt};
    auto saved = [&](size_t s) -> void* { return base + h->bwd_chunk * h->bwd_saved_off[s] * h->elt; };
    for (int64_t t0 = 0; t0 < tokens; t0 += h->bwd_chunk) {
        const int64_t nt = std::min(h->bwd_chunk, tokens - t0);
        const void* xc = static_cast<const char*>(x) + t0 * h->plan.N * h->elt;
        // forward, one launch per step, every step's input kept
        const void* cur = xc;
        for (size_t s = 0; s + 1 < n; ++s) {
            int rc = launch_step(h, w, h->steps[s], cur, saved(s + 1), nt, st);
            if (rc != TN_OK) return rc;
            cur = saved(s + 1);
        }
        // backward
        const void* dcur = static_cast<const char*>(dy) + t0 * h->plan.M * h->elt;
        int toggle = 0;
        for (size_t s = n; s-- > 0;) {
            const DevStep& fs = h->steps[s];
            const void* in_s = s == 0 ? xc : saved(s);
            void* g = grads[fs.plan.slot];
            if (g) {
                const int64_t elems = h->plan.tensors[size_t(fs.plan.tensor)].n_elems;
                int rc = launch_param_gradient(h, fs, dcur, in_s, static_cast<float*>(g), elems, nt, t0 > 0, st);
                if (rc != TN_OK) return rc;
            }
            if (s > 0) {
                int rc = launch_step(h, w, h->bwd[s], dcur, dbufs[toggle], nt, st);
                if (rc != TN_OK) return rc;
                dcur = dbufs[toggle];
                toggle ^= 1;
            }
        }
    }
    return TN_OK;
}

int tn_linear_quantized_tensor(tn_linear_t h, int32_t slot, void* codes, void* exponents, void* stream) {
    if (!h || slot < 0 || size_t(slot) >= h->quant_codes.size()) return TN_ERR_INVALID_ARG;
    hipStream_t st = static_cast<hipStream_t>(stream);
    const int64_t n = h->quant_elems[size_t(slot)];
    if (codes && hipMemcpyAsync(codes, h->quant_codes[size_t(slot)], size_t((n + 1) / 2), hipMemcpyDeviceToDevice, st) != hipSuccess)
        return TN_ERR_HIP;
    if (exponents &&
        hipMemcpyAsync(exponents, h->quant_exps[size_t(slot)], size_t((n + 31) / 32), hipMemcpyDeviceToDevice, st) != hipSuccess)
        return TN_ERR_HIP;
    return TN_OK;
}

int tn_linear_forward_scratch(tn_linear_t h, const void* x, void* y, int64_t tokens, void* stream) {
    if (!h || tokens < 0) return TN_ERR_INVALID_ARG;
    if (tokens == 0) return TN_OK;
    if (!x || !y || !aligned16(x) || !aligned16(y) || h->profiling) return TN_ERR_INVALID_ARG;       // profiling creates events, i.e. allocates
    void* base = (h->device >= 0 && h->device < 64) ? g_scratch_ptr[h->device] : nullptr;
    if (!base) return TN_ERR_UNSUPPORTED;
    Workspace w;
    const bool one_launch = h->small_chain && (h->elt == 4 || tokens <= kSmallChainMaxBf16Tokens);
    if (one_launch) {
        // nothing but x and y is touched
    } else if ((h->pair && tokens >= h->pair_min_tokens) || (h->kron && tokens >= h->kron_min_tokens)) {
        // only partial sums: the launch takes as many splits of the bond as fit
        w.partial = base;
        w.partial_bytes = kScratchBytes;
    } else {
        // the compact steps in one pass: [partial sums | buffer 0 | buffer 1], 256-byte aligned pieces
        int64_t max_r = 1;
        for (const auto& s : h->steps) max_r = std::max(max_r, s.plan.R);
        if (tokens > ((int64_t(1) << 31) - 1024) / max_r) return TN_ERR_SCRATCH;      // rows of a pass are indexed with 32 bits
        const int64_t per_token = h->plan.max_intermediate * h->elt;
        if (per_token > 0 && tokens > kScratchBytes / per_token) return TN_ERR_SCRATCH;
        const int64_t buf = (tokens * per_token + 255) & ~int64_t(255);
        // the split-K kernels' sums have to fit; the matrix-product kernel takes as many ranges of K as there is room for
        const int64_t room = kScratchBytes - 2 * buf - 256;
        int64_t part = 0;
        if (!(h->flags & TN_FLAG_NO_SPLIT_K) && h->elt == 2)
            for (const tn::LaunchIO& l : h->schedule)
                if (l.steps == 1) {
                    const DevStep& s = h->steps[size_t(l.first)];
                    if (tokens * s.plan.R >= kGemmMinRows && gemm_fits(s) && s.cmode != 0) {
                        part = std::max(part, gemm_choice(h, s, tokens * s.plan.R, std::max<int64_t>(0, std::min(kScratchBytes / 2, room))).partial_bytes);
                        continue;
                    }
                    const SplitCfg c = split_config(s, tokens * s.plan.R);
                    if (c.use) part = std::max(part, c.partial_bytes);
                }
        part = (part + 255) & ~int64_t(255);
        if (part + 2 * buf > kScratchBytes) return TN_ERR_SCRATCH;
        char* b = static_cast<char*>(base);
        w.partial = part > 0 ? b : nullptr;
        w.partial_bytes = part;
        w.ws[0] = b + part;
        w.ws[1] = b + part + buf;
        w.chunk_tokens = tokens;
    }
    return forward_in(h, w, false, x, y, tokens, static_cast<hipStream_t>(stream));
}

int tn_linear_profile(tn_linear_t h, int32_t enable) {
    if (!h) return TN_ERR_INVALID_ARG;
    if (enable) clear_profile(h);
    h->profiling = enable != 0;
    return TN_OK;
}

int tn_linear_profile_read(tn_linear_t h, int32_t step, double* total_ms, int64_t* launches) {
    if (!h || !total_ms || !launches || step < 0 || step >= int(h->steps.size())) return TN_ERR_INVALID_ARG;
    double ms = 0;
    int64_t n = 0;
    for (auto& r : h->prof) {
        if (r.step != step) continue;
        if (hipEventSynchronize(r.stop) != hipSuccess) return TN_ERR_HIP;
        float e = 0;
        if (hipEventElapsedTime(&e, r.start, r.stop) != hipSuccess) return TN_ERR_HIP;
        ms += e;
        ++n;
    }
    *total_ms = ms;
    *launches = n;
    return TN_OK;
}

int tn_linear_destroy(tn_linear_t h) {
    free_handle(h);
    return TN_OK;
}

int tn_linear_query(tn_linear_t h, int32_t what, int64_t* value) {
    if (!h || !value) return TN_ERR_INVALID_ARG;
    switch (what) {
        case TN_QUERY_PACKED_BYTES: *value = h->packed_bytes; return TN_OK;
        case TN_QUERY_WORKSPACE_BYTES: *value = h->workspace_bytes; return TN_OK;
        case TN_QUERY_CHUNK_TOKENS: *value = h->chunk_tokens; return TN_OK;
        case TN_QUERY_LAZY_MIN_TOKENS: *value = h->lazy ? h->lazy_min_tokens : 0; return TN_OK;
        case TN_QUERY_LAZY_FLOPS_PER_TOKEN: *value = h->lazy ? h->lazy_plan.flops : 0; return TN_OK;
        case TN_QUERY_MATRIX_MIN_TOKENS: *value = h->matrix ? h->mat_ranges.front().first : 0; return TN_OK;
        case TN_QUERY_MATRIX_BUILD_FLOPS: *value = h->matrix ? h->mat_flops : 0; return TN_OK;
        case TN_QUERY_GRADIENT_MATRIX_MIN_TOKENS: *value = h->mgrad ? h->mgrad_min_tokens : 0; return TN_OK;
        case TN_QUERY_GRADIENT_MATRIX_FLOPS: *value = h->mgrad ? h->mgrad_flops : 0; return TN_OK;
        case TN_QUERY_QUANT_BYTES: *value = h->quant_bytes; return TN_OK;
        case TN_QUERY_QUANT_STREAM_BYTES: *value = h->q4_stream_bytes; return TN_OK;
        case TN_QUERY_BACKWARD_CHUNK_TOKENS: *value = h->trainable ? (h->mgrad ? h->mgrad_chunk : h->bwd_chunk) : 0; return TN_OK;
        case TN_QUERY_BACKWARD_WORKSPACE_BYTES: *value = h->trainable ? h->bwd_ws_bytes + h->bwd_partial_bytes : 0; return TN_OK;
        default: break;
    }
    if (what >= TN_QUERY_MATRIX_TOKENS_BASE) {
        *value = takes_matrix(h, int64_t(what) - TN_QUERY_MATRIX_TOKENS_BASE) ? 1 : 0;
        return TN_OK;
    }
    if (what >= TN_QUERY_STEP_BASE && (what - TN_QUERY_STEP_BASE) % 10 == 5) {
        int s = (what - TN_QUERY_STEP_BASE) / 10;
        if (s >= int(h->steps.size())) return TN_ERR_INVALID_ARG;
        *value = h->steps[size_t(s)].variant;
        return TN_OK;
    }
    if (what >= TN_QUERY_STEP_BASE && (what - TN_QUERY_STEP_BASE) % 10 == 6) {
        int s = (what - TN_QUERY_STEP_BASE) / 10;
        if (s >= int(h->steps.size())) return TN_ERR_INVALID_ARG;
        *value = h->steps[size_t(s)].fuse_next ? 1 : ((h->pair && s == 0) ? 2 : ((h->kron && s == 0) ? 4 : 0));
        if (h->small_chain && size_t(s) + 1 < h->steps.size()) *value = 3;
        return TN_OK;
    }
    return plan_value(h->plan, what, value);
}

}  // extern "C"
