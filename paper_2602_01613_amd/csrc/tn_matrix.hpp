// Host-side planner (no GPU calls) of the order of contraction in which the parameter tensors of a train or a ring are
// contracted with each other first and with the activations last.
//
// A chain of tensors cut into two halves is a sum over the bond(s) between them, W[m, n] = sum_rho P[(m, n)_P, rho] *
// Q[(m, n)_Q, rho], where (m, n)_P are the modes of the first half. As matrix products:
//     half     P and Q from the one or two tensors each is made of,
//     w        W from P and Q,
//     y        Y = X W^T.
// For T tokens that is 2 M N (T + rho) operations, whatever the order of the tensors inside; the orders that carry the
// activations through the chain (tn_plan.hpp) take F T with F far above 2 M N at useful ranks (ring of rank 32, 5120 x
// 25600: F = 19 * 2 M N). So a call of many tokens is cheaper in this order, and one of a few tokens is not.
//
// Every product here is Out[row_off[r] + col_off[c]] = sum_k A[r][k] B[c][k]: the permutation from one product to the
// next happens in its stores, through two tables, as in the steps of tn_plan.hpp. An output is written either row-major
// or in the fragment-major packing of a B operand; both are sums of one offset per digit where the extents allow it,
// which is checked value by value.
#pragma once

#include <map>

#include "tn_plan.hpp"

namespace tn {

// Offset of element (c, k) of a packed operand with nks = Kp / 16 steps of k (see bfrag_offset in kernels/common.hpp),
// split into what c and what k contribute.
inline int64_t packed_col(int64_t c, int64_t nks) { return (c >> 5) * nks * 512 + (c & 31) * 8; }
inline int64_t packed_k(int64_t k) { return (k >> 4) * 512 + ((k >> 3) & 1) * 256 + (k & 7); }

struct SourceDim {
    int64_t extent;       // digits the operand is laid out for
    int64_t limit;        // digits the tensor has: zeros from there on
    int64_t stride;       // in elements of the caller's tensor
};

// An operand kept by the layer, written once from a caller's tensor: [rows][k], row-major or packed.
struct SourceOp {
    int slot = -1;
    std::vector<SourceDim> rows, ks;       // outer -> inner
    int64_t R = 1, K = 1;
};

struct Product {
    SourceOp a, b;                         // slot < 0: an intermediate
    int64_t R = 1, C = 1, K = 1, Kp = 64;  // Kp: K padded to whole tiles of 64
    std::vector<int32_t> row_off, col_off;
    int64_t out_elems = 0;
};

struct MatrixHalf {
    std::vector<int> tensors;              // network tensors: one (kept as an operand) or two (contracted per call)
    std::vector<int> mn;                   // ids of its modes, outer -> inner
    int64_t F = 1;                         // product of their extents
    Product build;                         // two tensors
    SourceOp keep;                         // one tensor
};

struct MatrixPlan {
    int64_t M = 0, N = 0;
    std::vector<int> bond;                 // ids shared by the halves, outer -> inner
    int64_t Kr = 1, Krp = 64;              // their extent, and padded to whole tiles of 64
    MatrixHalf half[2];                    // 0: rows of `w` (row-major), 1: its columns (packed)
    Product w;                             // out: W packed, columns m, k = n
    int64_t w_elems = 0;                   // with the columns padded to whole tiles
};

constexpr int64_t kMatrixMaxElems = int64_t(1) << 30;      // outputs are addressed with 31-bit byte offsets
constexpr int kMatrixColPad = 256;
constexpr int64_t kMatrixMaxDigits = int64_t(1) << 22;     // positions that a check value by value walks (64 MB of host memory)

namespace detail {

typedef std::map<int, std::vector<int64_t>> DigitOffsets;

// Offset that every digit of every id contributes to f(position over ids); false where f is not their sum.
template <typename F>
bool digit_offsets(const std::vector<int>& ids, const std::vector<int64_t>& ext, const F& f, DigitOffsets* out) {
    int64_t total = 1;
    std::vector<int64_t> weight(ids.size(), 1);
    for (size_t j = ids.size(); j-- > 0;) {
        weight[j] = total;
        total *= ext[size_t(ids[j])];
        if (total > kMatrixMaxDigits) return false;
    }
    // sums of every position, grown from the innermost id outwards
    std::vector<int64_t> sums(size_t(total), 0);
    for (size_t j = ids.size(); j-- > 0;) {
        std::vector<int64_t>& v = (*out)[ids[j]];
        v.resize(size_t(ext[size_t(ids[j])]));
        for (size_t d = v.size(); d-- > 0;) {
            v[d] = f(int64_t(d) * weight[j]);
            for (int64_t p = 0; p < weight[j]; ++p) sums[d * size_t(weight[j]) + size_t(p)] = sums[size_t(p)] + v[d];
        }
    }
    for (int64_t p = 0; p < total; ++p)
        if (sums[size_t(p)] != f(p)) return false;
    return true;
}

// The same where f is the position itself: a sum by construction, whatever its length.
inline void flat_offsets(const std::vector<int>& ids, const std::vector<int64_t>& ext, DigitOffsets* out) {
    int64_t weight = 1;
    for (size_t j = ids.size(); j-- > 0;) {
        std::vector<int64_t>& v = (*out)[ids[j]];
        v.clear();
        for (int64_t d = 0; d < ext[size_t(ids[j])]; ++d) v.push_back(d * weight);
        weight *= ext[size_t(ids[j])];
    }
}

// ids with the one whose neighbouring digits lie closest in the output innermost
inline void sort_by_offset(std::vector<int>* ids, const DigitOffsets& t) {
    auto key = [&](int i) {
        const std::vector<int64_t>& v = t.at(i);
        return v.size() > 1 ? v[1] : std::numeric_limits<int64_t>::max();
    };
    std::stable_sort(ids->begin(), ids->end(), [&](int x, int y) { return key(x) > key(y); });
}

inline std::vector<int32_t> digit_table(const std::vector<int>& ids, const std::vector<int64_t>& ext, const DigitOffsets& t) {
    std::vector<int32_t> tab(1, 0);
    for (int i : ids) {
        const std::vector<int64_t>& v = t.at(i);
        std::vector<int32_t> next(tab.size() * v.size());
        size_t at = 0;
        for (int32_t o : tab)
            for (int64_t d : v) next[at++] = o + int32_t(d);
        tab.swap(next);
    }
    return tab;
}

inline std::vector<int> shared_ids(const NetTensor& a, const NetTensor& b) {
    std::vector<int> s;
    for (int i : a.idx)
        if (contains(b.idx, i)) s.push_back(i);
    return s;
}

inline std::vector<int> without(const std::vector<int>& ids, const std::vector<int>& drop) {
    std::vector<int> s;
    for (int i : ids)
        if (!contains(drop, i)) s.push_back(i);
    return s;
}

inline SourceOp source_op(const Plan& p, const std::vector<int64_t>& ext, int tensor, const std::vector<int>& rows,
                          const std::vector<int>& ks) {
    const NetTensor& T = p.tensors[size_t(tensor)];
    SourceOp o;
    o.slot = T.slot;
    auto add = [&](const std::vector<int>& ids, std::vector<SourceDim>* dims, int64_t* n) {
        for (int i : ids) {
            int64_t stride = 0;
            for (size_t j = 0; j < T.idx.size(); ++j)
                if (T.idx[j] == i) stride = T.stride[j];
            dims->push_back({ext[size_t(i)], p.extent[size_t(i)], stride});
            *n *= ext[size_t(i)];
        }
    };
    add(rows, &o.rows, &o.R);
    add(ks, &o.ks, &o.K);
    return o;
}

inline int64_t round64(int64_t v) { return (v + 63) / 64 * 64; }

// The product of tensors ta and tb over the ids they share, stored through the digit offsets `t`; whichever of the two has
// stores in aligned runs of 8 columns supplies the columns. False if neither does, or the output is too large.
inline bool pair_product(const Plan& p, const std::vector<int64_t>& ext, int ta, int tb, const DigitOffsets& t, int64_t out_elems,
                         Product* out) {
    if (out_elems > kMatrixMaxElems) return false;
    for (int turn = 0; turn < 2; ++turn) {
        const int a = turn ? tb : ta, b = turn ? ta : tb;
        const NetTensor &A = p.tensors[size_t(a)], &B = p.tensors[size_t(b)];
        const std::vector<int> s = shared_ids(A, B);
        std::vector<int> rows = without(A.idx, s), cols = without(B.idx, s);
        if (s.empty() || rows.size() > size_t(kMaxGatherDims) || cols.size() > size_t(kMaxGatherDims)) return false;
        sort_by_offset(&rows, t);
        sort_by_offset(&cols, t);
        Product q;
        q.row_off = digit_table(rows, ext, t);
        q.col_off = digit_table(cols, ext, t);
        if (run_length(q.col_off, 8) != 8 || !all_multiple_of(q.row_off, 8)) continue;
        q.a = source_op(p, ext, a, rows, s);
        q.b = source_op(p, ext, b, cols, s);
        q.R = q.a.R;
        q.C = q.b.R;
        q.K = q.a.K;
        q.Kp = round64(q.K);
        q.out_elems = out_elems;
        *out = q;
        return true;
    }
    return false;
}

}  // namespace detail

// The plan for one cut of the network: the tensors of group[0] and of group[1], one or two each. `wt`: offsets of the modes' digits
// in the packed W.
inline bool matrix_plan_of_cut(const Plan& net, const std::vector<int> (&group)[2], const detail::DigitOffsets& wt, MatrixPlan* m) {
    using namespace detail;
    std::vector<int> open[2];              // ids of a group that its own tensors do not contract
    for (int g = 0; g < 2; ++g) {
        std::vector<int> inner;
        if (group[g].size() == 2) inner = shared_ids(net.tensors[size_t(group[g][0])], net.tensors[size_t(group[g][1])]);
        for (int t : group[g])
            for (int i : without(net.tensors[size_t(t)].idx, inner)) open[g].push_back(i);
    }
    int last_n = -1;                       // W is stored in runs along the last in-mode: the half that has it gives the columns
    for (int i : net.x_idx)
        if (net.extent[size_t(i)] > 1) last_n = i;
    const int q = contains(open[0], last_n) ? 0 : 1;
    if (last_n < 0 || !contains(open[q], last_n)) return false;
    *m = MatrixPlan();
    m->M = net.M;
    m->N = net.N;
    for (int i : open[1 - q])
        if (contains(open[q], i)) m->bond.push_back(i);
    if (m->bond.empty() || m->bond.size() > 2) return false;
    for (int i : m->bond) m->Kr *= net.extent[size_t(i)];
    m->Krp = round64(m->Kr);
    // a bond of one index may be laid out longer than it is (zeros); of two, it has to be whole tiles
    std::vector<int64_t> ext = net.extent;
    if (m->bond.size() == 1) ext[size_t(m->bond[0])] = m->Krp;
    else if (m->Kr != m->Krp) return false;
    m->w_elems = (m->M + kMatrixColPad - 1) / kMatrixColPad * kMatrixColPad * m->N;
    if (m->w_elems > kMatrixMaxElems) return false;
    for (int h = 0; h < 2; ++h) {
        const int g = h == 0 ? 1 - q : q;
        m->half[h].tensors = group[g];
        m->half[h].mn = without(open[g], m->bond);
        sort_by_offset(&m->half[h].mn, wt);
        m->half[h].F = prod_extents(m->half[h].mn, ext);
    }
    m->w.row_off = digit_table(m->half[0].mn, ext, wt);
    m->w.col_off = digit_table(m->half[1].mn, ext, wt);
    m->w.R = m->half[0].F;
    m->w.C = m->half[1].F;
    m->w.K = m->Kr;
    m->w.Kp = m->Krp;
    m->w.out_elems = m->w_elems;
    if (run_length(m->w.col_off, 8) != 8 || !all_multiple_of(m->w.row_off, 8)) return false;
    // the halves: [modes][bond], row-major for the rows of w and packed for its columns; of a bond of two indices, the one
    // whose digits can be stored in runs of 8 goes innermost
    for (int turn = 0; turn < int(m->bond.size()); ++turn) {
        if (turn) std::swap(m->bond[0], m->bond[1]);
        bool ok = true;
        for (int h = 0; h < 2 && ok; ++h) {
            MatrixHalf& H = m->half[h];
            if (H.tensors.size() == 1) {
                H.keep = source_op(net, ext, H.tensors[0], H.mn, m->bond);
                ok = H.F * m->Krp <= kMatrixMaxElems;
                continue;
            }
            DigitOffsets t;
            const int64_t krp = m->Krp;
            ok = digit_offsets(H.mn, ext, [&](int64_t c) { return h == 0 ? c * krp : packed_col(c, krp / 16); }, &t) &&
                 digit_offsets(m->bond, ext, [&](int64_t k) { return h == 0 ? k : packed_k(k); }, &t);
            const int64_t cols = h == 0 ? H.F : (H.F + kMatrixColPad - 1) / kMatrixColPad * kMatrixColPad;
            ok = ok && pair_product(net, ext, H.tensors[0], H.tensors[1], t, cols * krp, &H.build);
        }
        if (ok) return true;
    }
    return false;
}

// The cut of the network of `d` (a train or a ring of two to four tensors) over the smallest bond; false where the layer
// has no such plan.
inline bool make_matrix_plan(const tn_linear_desc* d, Plan* net, MatrixPlan* m) {
    if (d->dtype != TN_DTYPE_BF16 || (d->format != TN_FORMAT_TT && d->format != TN_FORMAT_TR)) return false;
    if (build_network(d, net) != TN_OK) return false;
    const int n = int(net->tensors.size());
    if (n < 2 || n > 4) return false;
    for (const NetTensor& T : net->tensors)
        if (T.trace_extent != 1) return false;
    if (net->N % 64 || net->M % 8 || net->N >= (int64_t(1) << 21)) return false;
    detail::DigitOffsets wt;
    const int64_t nks = net->N / 16;
    if (!detail::digit_offsets(net->y_idx, net->extent, [&](int64_t c) { return packed_col(c, nks); }, &wt) ||
        !detail::digit_offsets(net->x_idx, net->extent, packed_k, &wt))
        return false;
    // the cuts, smallest bond first: the first that has a plan is the one
    struct Cut {
        int64_t bond;
        std::vector<int> group[2];
    };
    std::vector<Cut> cuts;
    for (int first = 0; first < (d->format == TN_FORMAT_TR ? n : 1); ++first)
        for (int len = 1; len < n; ++len) {
            if (len > 2 || n - len > 2) continue;
            Cut c{1, {}};
            for (int j = 0; j < n; ++j) c.group[j < len ? 0 : 1].push_back((first + j) % n);
            std::vector<int> shared;
            for (int t : c.group[0])
                for (int u : c.group[1])
                    for (int i : detail::shared_ids(net->tensors[size_t(t)], net->tensors[size_t(u)])) shared.push_back(i);
            c.bond = detail::prod_extents(shared, net->extent);
            cuts.push_back(c);
        }
    std::stable_sort(cuts.begin(), cuts.end(), [](const Cut& x, const Cut& y) { return x.bond < y.bond; });
    for (const Cut& c : cuts)
        if (matrix_plan_of_cut(*net, c.group, wt, m)) return true;
    return false;
}

// ---- gradients of the parameter tensors on the same cut ----
// L = sum_{t, i} dY[t, i] Y[t, i] = sum_{m, n} dW[m, n] W[m, n] with dW = dY^T X, whatever W is made of. From there
//     dP[f, rho] = sum_g dW[f, g] Q[g, rho],   dQ[g, rho] = sum_f dW[f, g] P[f, rho]     (f, g: modes of the halves)
// and, where a half is two tensors contracted over s, H[f1, f2] = sum_s A[f1, s] B[f2, s],
//     dA[f1, s] = sum_f2 dH[f1, f2] B[f2, s],  dB[f2, s] = sum_f1 dH[f1, f2] A[f1, s].
// The modes of a half are laid out tensor by tensor here, those of each tensor as one number.
struct GradOut {                           // [R][C] -> the caller's tensor
    int slot = -1;
    std::vector<GatherDim> rows, cols;
};

struct MatrixGradHalf {
    bool pair = false;
    // the half as an operand of the other one's gradient: packed, columns bond (in the other half's order), k = its modes
    Product op;                            // pair
    SourceOp op_keep;                      // one tensor
    // its own gradient: rows its modes, columns the bond
    std::vector<int32_t> row_off, col_off; // pair: into dH [F1][F2]
    int64_t F1 = 1, F2 = 1;
    SourceOp a, b;                         // pair: A and B with rows s and k = f1, f2
    GradOut out_a, out_b;                  // pair: of dA [F1][S], dB [F2][S]; one tensor: out_a of [F][Kr]
};

struct MatrixGrad {
    std::vector<int32_t> dw_row, dw_col;   // dW [m][n] -> [F of half 0][F of half 1], or with
    bool tiled = false;                    // -> [F of half 1 / 32][F of half 0][32]
    MatrixGradHalf half[2];
};

namespace detail {

// One number for the modes of a tensor, in the order of its axes: an id of its own, with the ids it stands for.
struct Modes {
    std::vector<int64_t> ext;              // of every id, those of the numbers after the network's
    std::vector<std::vector<int>> parts;   // of the ids from first on
    int first = 0;
    int add(const std::vector<int>& ids) {
        int64_t e = 1;
        for (int i : ids) e *= ext[size_t(i)];
        ext.push_back(e);
        parts.push_back(ids);
        return int(ext.size()) - 1;
    }
    std::vector<int> spell(const std::vector<int>& ids) const {
        std::vector<int> r;
        for (int i : ids) {
            if (i < first) r.push_back(i);
            else r.insert(r.end(), parts[size_t(i - first)].begin(), parts[size_t(i - first)].end());
        }
        return r;
    }
};

inline std::vector<GatherDim> grad_dims(const Plan& p, int tensor, const std::vector<int>& ids) {
    const NetTensor& T = p.tensors[size_t(tensor)];
    std::vector<GatherDim> d;
    for (int i : ids)
        for (size_t j = 0; j < T.idx.size(); ++j)
            if (T.idx[j] == i) d.push_back({p.extent[size_t(i)], T.stride[j]});
    return d;
}

}  // namespace detail

// False where a layout does not come out in runs of 8 or in whole tiles of k.
inline bool make_matrix_grad(const Plan& net, const MatrixPlan& m, MatrixGrad* g, bool want_tiled = false) {
    using namespace detail;
    int last_n = -1;
    for (int i : net.x_idx)
        if (net.extent[size_t(i)] > 1) last_n = i;
    if (m.half[0].F % 64 || m.half[1].F % 64 || m.Kr % 8) return false;
    Modes md;
    md.ext = net.extent;
    md.first = int(net.extent.size());
    std::vector<int> order[2], number[2];              // of each half: tensors outer -> inner, and their numbers
    for (int h = 0; h < 2; ++h) {
        const MatrixHalf& H = m.half[h];
        order[h] = H.tensors;
        auto modes = [&](int t) {
            std::vector<int> ids;
            for (int i : net.tensors[size_t(t)].idx)
                if (contains(H.mn, i)) ids.push_back(i);
            // (m, n): the in-modes innermost
            std::stable_sort(ids.begin(), ids.end(), [&](int x, int y) { return !contains(net.x_idx, x) && contains(net.x_idx, y); });
            return ids;
        };
        auto extent_of = [&](int t) { return prod_extents(modes(t), net.extent); };
        if (order[h].size() == 2) {
            const bool swap = h == 1 ? !contains(modes(order[h][1]), last_n) : extent_of(order[h][1]) % 16 != 0;
            if (swap) std::swap(order[h][0], order[h][1]);
            if (extent_of(order[h][1]) % 16) return false;
        }
        for (int t : order[h]) number[h].push_back(md.add(modes(t)));
    }
    // dW: rows m, columns n, both in the caller's order
    DigitOffsets wt;
    for (int h = 0; h < 2; ++h) {
        int64_t weight = h == 0 ? m.half[1].F : 1;
        for (size_t j = number[h].size(); j-- > 0;) {
            const std::vector<int> ids = md.spell({number[h][j]});
            for (size_t i = ids.size(); i-- > 0;) {
                std::vector<int64_t>& v = wt[ids[i]];
                for (int64_t d = 0; d < net.extent[size_t(ids[i])]; ++d) v.push_back(d * weight);
                weight *= net.extent[size_t(ids[i])];
            }
        }
    }
    if (want_tiled) {
        // a sum of one offset per digit where the digits' parts below 32 never carry
        int64_t below = 0;
        std::vector<int> inner;
        for (int n : number[1])
            for (int i : md.spell({n})) inner.push_back(i);
        for (int i : inner) {
            int64_t most = 0;
            for (int64_t v : wt[i]) most = std::max(most, v % 32);
            below += most;
        }
        g->tiled = m.half[1].F % 32 == 0 && below < 32;
        if (g->tiled)
            for (auto& d : wt) {
                const bool in = contains(inner, d.first);
                for (int64_t& v : d.second) v = in ? v / 32 * m.half[0].F * 32 + v % 32 : v / m.half[1].F * 32;
            }
    }
    g->dw_row = digit_table(net.y_idx, net.extent, wt);
    g->dw_col = digit_table(net.x_idx, net.extent, wt);
    if (run_length(g->dw_col, 8) != 8 || !all_multiple_of(g->dw_row, 8)) return false;
    auto source = [&](int t, const std::vector<int>& rows, const std::vector<int>& ks) {
        return source_op(net, net.extent, t, md.spell(rows), md.spell(ks));
    };
    for (int h = 0; h < 2; ++h) {
        const MatrixHalf& H = m.half[h];
        MatrixGradHalf& G = g->half[h];
        G.pair = H.tensors.size() == 2;
        // order of the bond in its gradient's columns: for a pair, the tensor that has the innermost index is B
        std::vector<int> bond = m.bond;
        if (!G.pair) {
            std::vector<int> modes = md.spell(number[h]);
            G.out_a.slot = net.tensors[size_t(H.tensors[0])].slot;
            G.out_a.rows = grad_dims(net, H.tensors[0], modes);
            G.out_a.cols = grad_dims(net, H.tensors[0], bond);
        } else {
            const std::vector<int> s = shared_ids(net.tensors[size_t(H.tensors[0])], net.tensors[size_t(H.tensors[1])]);
            bool ok = false;
            for (int turn = 0; turn < 2 && !ok; ++turn) {
                bond = m.bond;
                if (turn && bond.size() == 2) std::swap(bond[0], bond[1]);
                if (net.extent[size_t(bond.back())] % 8) continue;
                const int ib = contains(net.tensors[size_t(order[h][0])].idx, bond.back()) ? 0 : 1;
                const int ta = order[h][size_t(1 - ib)], tb = order[h][size_t(ib)];
                std::vector<int> f1 = {number[h][size_t(1 - ib)]}, f2 = {number[h][size_t(ib)]};
                for (int i : bond) (contains(net.tensors[size_t(tb)].idx, i) ? f2 : f1).push_back(i);
                G.F1 = prod_extents(f1, md.ext);
                G.F2 = prod_extents(f2, md.ext);
                if (G.F2 % 64 || G.F1 > kMatrixMaxElems / G.F2) continue;
                DigitOffsets t;
                std::vector<int> all = f1;
                all.insert(all.end(), f2.begin(), f2.end());
                flat_offsets(all, md.ext, &t);
                G.row_off = digit_table(number[h], md.ext, t);
                G.col_off = digit_table(bond, md.ext, t);
                if (run_length(G.col_off, 8) != 8 || !all_multiple_of(G.row_off, 8)) continue;
                G.a = source(ta, s, f1);
                G.b = source(tb, s, f2);
                G.out_a.slot = net.tensors[size_t(ta)].slot;
                G.out_a.rows = grad_dims(net, ta, md.spell(f1));
                G.out_a.cols = grad_dims(net, ta, s);
                G.out_b.slot = net.tensors[size_t(tb)].slot;
                G.out_b.rows = grad_dims(net, tb, md.spell(f2));
                G.out_b.cols = grad_dims(net, tb, s);
                ok = true;
            }
            if (!ok) return false;
        }
        // the other half as the operand: columns in this bond order
        const int o = 1 - h;
        const MatrixHalf& O = m.half[o];
        MatrixGradHalf& P = g->half[o];
        if (O.tensors.size() == 1) {
            P.op_keep = source(O.tensors[0], bond, number[o]);
            continue;
        }
        DigitOffsets t;
        if (!digit_offsets(bond, md.ext, [&](int64_t c) { return packed_col(c, O.F / 16); }, &t) ||
            !digit_offsets(number[o], md.ext, packed_k, &t))
            return false;
        const NetTensor &A = net.tensors[size_t(order[o][0])], &B = net.tensors[size_t(order[o][1])];
        const std::vector<int> s = shared_ids(A, B);
        std::vector<int> rows = {number[o][0]}, cols = {number[o][1]};
        for (int i : bond) (contains(B.idx, i) ? cols : rows).push_back(i);
        sort_by_offset(&rows, t);
        sort_by_offset(&cols, t);
        Product& q = P.op;
        q.row_off = digit_table(rows, md.ext, t);
        q.col_off = digit_table(cols, md.ext, t);
        if (run_length(q.col_off, 8) != 8 || !all_multiple_of(q.row_off, 8)) return false;
        q.a = source(order[o][0], rows, s);
        q.b = source(order[o][1], cols, s);
        q.R = q.a.R;
        q.C = q.b.R;
        q.K = q.a.K;
        q.Kp = round64(q.K);
        q.out_elems = (m.Kr + kMatrixColPad - 1) / kMatrixColPad * kMatrixColPad * O.F;
        if (q.out_elems > kMatrixMaxElems) return false;
    }
    return true;
}

// ---- slices of the Kronecker-sum kernel as products ----
// The kernel (kernels/kronsum.hpp) reads, per value rho of the bond, two small matrices in fragment order: H0 with columns o1
// and k, H1 with columns o2 and a, where (o1, k) and (o2, a) are the modes of the halves. How it numbers o1, k, o2, a and rho
// is free, as long as the tables through which it reads x and writes y use the same numbers. The numbers are chosen such that
// both slice arrays are sums of one offset per digit: then each is one product of the two tensors of its half. k and a are
// padded with zeros to what the kernel's instantiation holds.
struct SlicePlan {
    Product half[2];
    std::vector<int32_t> xrow, xcol, yrow, ycol;       // where a and k sit in a token of x, o1 and o2 in one of y
    bool x_vec8 = true;                                 // 8 consecutive k of one a are one aligned piece of x
    int64_t h1_offset = 0, bytes = 0;                   // of the second array, and of both
};

// `q`: a plan of two steps whose tensors are merged from two of the caller's each; `net`: the network before the merges.
inline bool merged_tensors(const Plan& net, const Plan& q, int (&tensors)[2][2]) {
    const int nc = net.n_caller_tensors;
    for (int h = 0; h < 2; ++h) {
        const int mi = q.steps[size_t(h)].slot - nc;
        if (mi < 0 || mi >= int(q.merges.size()) || q.merges[size_t(mi)].p_slot >= nc || q.merges[size_t(mi)].q_slot >= nc) return false;
        tensors[h][0] = q.merges[size_t(mi)].p_slot;
        tensors[h][1] = q.merges[size_t(mi)].q_slot;
    }
    return true;
}

inline bool make_slice_plan(const Plan& net, const Plan& q, const KronDims& d, SlicePlan* out) {
    using namespace detail;
    const int *cfg = kKronConfig[d.cfg], at = cfg[0], ks0 = cfg[1], o2t = cfg[2], o1t = cfg[3];
    int tensors[2][2];
    if (!merged_tensors(net, q, tensors)) return false;
    if (d.A % 16 || d.K0 % 8) return false;
    std::vector<int64_t> ext = net.extent;
    const std::vector<int> bond = [&] {
        std::vector<int> b;
        for (int t : tensors[0])
            for (int i : net.tensors[size_t(t)].idx)
                for (int u : tensors[1])
                    if (contains(net.tensors[size_t(u)].idx, i) && !contains(b, i)) b.push_back(i);
        return b;
    }();
    if (prod_extents(bond, ext) != d.P) return false;
    // offsets of a mode's digits in a token of x or y
    auto strides = [&](const std::vector<int>& layout, const std::vector<int>& ids, const std::vector<int64_t>& e) {
        std::vector<int32_t> tab(1, 0);
        for (int i : ids) {
            int64_t st = 1;
            for (size_t j = layout.size(); j-- > 0 && layout[j] != i;) st *= net.extent[size_t(layout[j])];
            std::vector<int32_t> next;
            for (int32_t o : tab)
                for (int64_t v = 0; v < e[size_t(i)]; ++v) next.push_back(o + int32_t(v * st));
            tab.swap(next);
        }
        return tab;
    };
    const int64_t slice[2] = {int64_t(o1t) * ks0 * 512, int64_t(o2t) * 2 * at * 512};
    const int64_t chunks = (d.O1 + 32 * o1t - 1) / (32 * o1t);
    const int64_t elems[2] = {chunks * d.P * slice[0], d.P * slice[1]};
    for (int h = 0; h < 2; ++h) {
        std::vector<int> o, k;                          // out-modes and in-modes of the half
        for (int t : tensors[h])
            for (int i : net.tensors[size_t(t)].idx) {
                if (contains(net.y_idx, i)) o.push_back(i);
                if (contains(net.x_idx, i)) k.push_back(i);
            }
        if (prod_extents(o, ext) != (h == 0 ? d.O1 : d.C1) || prod_extents(k, ext) != (h == 0 ? d.K0 : d.A)) return false;
        const int64_t k_real = h == 0 ? d.K0 : d.A, k_pad = h == 0 ? 16 * int64_t(ks0) : 32 * int64_t(at), nks = h == 0 ? ks0 : 2 * at;
        // x's innermost mode first as the inner digit of k, then the others; both orders of the out-modes
        std::stable_sort(k.begin(), k.end(), [&](int a, int b) { return a < b; });
        bool ok = false;
        for (int turn = 0; turn < 4 && !ok; ++turn) {
            std::vector<int> oo = o, kk = k;
            if (turn & 1) std::reverse(oo.begin(), oo.end());
            if (turn & 2) std::reverse(kk.begin(), kk.end());
            std::vector<int64_t> e = ext;
            const int outer = kk[0];
            const int64_t inner = k_real / e[size_t(outer)];
            if (k_pad % inner || e[size_t(kk.back())] % 8) continue;
            e[size_t(outer)] = k_pad / inner;
            DigitOffsets t;
            const int64_t P = d.P;
            auto col = [&](int64_t c) {
                return h == 0 ? c / (32 * o1t) * P * slice[0] + c % (32 * o1t) / 32 * nks * 512 + c % 32 * 8 : c / 32 * nks * 512 + c % 32 * 8;
            };
            if (!digit_offsets(oo, e, col, &t) || !digit_offsets(kk, e, packed_k, &t) ||
                !digit_offsets(bond, e, [&](int64_t r) { return r * slice[h]; }, &t) ||
                !pair_product(net, e, tensors[h][0], tensors[h][1], t, elems[h], &out->half[h]))
                continue;
            const std::vector<int32_t> x_of = strides(net.x_idx, kk, net.extent);
            (h == 0 ? out->yrow : out->ycol) = strides(net.y_idx, oo, net.extent);
            if (h == 0) {
                out->xcol = x_of;
            } else {
                // the kernel's a in a block of 16 sits at 8 * ((a / 4) % 2) + 4 * ((a / 8) % 2) + a % 4
                out->xrow.resize(size_t(d.A));
                for (int64_t a = 0; a < d.A; ++a)
                    out->xrow[size_t(a)] = x_of[size_t((a & ~int64_t(15)) + 8 * ((a >> 2) & 1) + 4 * ((a >> 3) & 1) + (a & 3))];
            }
            ok = true;
        }
        if (!ok) return false;
    }
    out->x_vec8 = run_length(out->xcol, 8) == 8 && all_multiple_of(out->xrow, 8);
    out->h1_offset = (elems[0] * 2 + 255) & ~int64_t(255);
    out->bytes = out->h1_offset + ((elems[1] * 2 + 255) & ~int64_t(255));
    return true;
}

// ---- slices of the Kronecker-sum kernel made on chip ----
// kernels/krondirect.hpp: per value of the bond a workgroup makes both slices from slabs of the cores, for calls of a few
// tokens. A row of kDirectConfig is an instantiation:
//   AT tiles of 16 of a, KS steps of 32 of k; a wave has O1W tiles of 16 of o1 and O2W of o2, the four waves in W1 columns of o1;
//   per half, WS of the waves along the streamed core's tiles, F of its tiles and C of the resident one's to a wave;
//   whether the rows of the second half's product are the streamed core's (the first half's always are); resident cores in LDS.
constexpr int kDirectConfigs = 5;
constexpr int kDirectConfig[kDirectConfigs][13] = {
    {5, 2, 1, 8, 4, 4, 1, 4, 4, 1, 10, 1, 0},
    {5, 2, 1, 1, 2, 4, 1, 2, 2, 1, 3, 1, 0},
    {8, 2, 1, 5, 4, 4, 1, 4, 4, 1, 10, 1, 0},
    {4, 3, 3, 10, 4, 2, 3, 5, 4, 2, 5, 1, 0},
    {10, 5, 1, 5, 4, 4, 2, 5, 2, 3, 5, 0, 1}};
constexpr int kDirectMaxSteps = 3;                      // of 32, of the bond inside a half

struct DirectPlan {
    int cfg = -1, steps = 1;
    SourceOp src[2][2];                                 // per half: resident, streamed core; rows: its value of the bond, then its modes
    int64_t tiles[2][2] = {{0, 0}, {0, 0}};             // of 16 rows of a slab
    int64_t n_res = 1, n_str = 1;
    int64_t A = 0, K0 = 0, O1 = 0, C1 = 0;
    std::vector<int32_t> xrow, xcol, yrow, ycol;
    std::vector<uint16_t> unit[2];                      // [row tile][column tile][lane]: LDS position / 8 in the slice
    bool x_vec8 = false;
};

// Position in its slice, in bytes, of column o and contracted index k (w = 0), or a (w = 1: numbered within 32 as the
// accumulators of the first product come out).
inline int64_t direct_position(int w, int64_t o, int64_t k, int64_t steps) {
    const int64_t block = ((o / 16) * steps + k / 32) * 1024;
    return w == 0 ? block + ((k % 32) / 8 * 16 + o % 16) * 16 + (k % 8) * 2
                  : block + ((k % 16) / 4 * 16 + o % 16) * 16 + (k % 32) / 16 * 8 + (k % 4) * 2;
}

// `tensors`: the two of each half. False where no instantiation holds the shape.
inline bool make_direct_plan(const Plan& net, const int (&tensors)[2][2], DirectPlan* out) {
    using namespace detail;
    const std::vector<int64_t>& ext = net.extent;
    struct Core {
        int t = -1, m = -1, n = -1;
        int64_t M = 1, N = 1;
    };
    auto core_of = [&](int t, Core* c) {
        c->t = t;
        for (int i : net.tensors[size_t(t)].idx) {
            if (ext[size_t(i)] == 1) continue;
            if (contains(net.y_idx, i)) {
                if (c->m >= 0) return false;
                c->m = i;
            }
            if (contains(net.x_idx, i)) {
                if (c->n >= 0) return false;
                c->n = i;
            }
        }
        if (c->m < 0 || c->n < 0 || net.tensors[size_t(t)].trace_extent != 1) return false;
        c->M = ext[size_t(c->m)];
        c->N = ext[size_t(c->n)];
        return c->M * c->N % 16 == 0;
    };
    Core cores[2][2];
    int inner[2];                                       // the id contracted inside a half
    std::vector<int> bond;
    for (int h = 0; h < 2; ++h) {
        for (int i = 0; i < 2; ++i)
            if (!core_of(tensors[h][i], &cores[h][i])) return false;
        inner[h] = -1;
        for (int i : shared_ids(net.tensors[size_t(tensors[h][0])], net.tensors[size_t(tensors[h][1])])) {
            if (ext[size_t(i)] == 1) continue;
            if (inner[h] >= 0) return false;
            inner[h] = i;
        }
        if (inner[h] < 0) return false;
    }
    for (int t : tensors[0])
        for (int i : net.tensors[size_t(t)].idx)
            for (int u : tensors[1])
                if (ext[size_t(i)] > 1 && contains(net.tensors[size_t(u)].idx, i) && !contains(bond, i)) bond.push_back(i);
    if (bond.empty() || bond.size() > 2) return false;
    const int64_t longest = std::max(ext[size_t(inner[0])], ext[size_t(inner[1])]);
    const int steps = int((longest + 31) / 32);
    if (steps > kDirectMaxSteps) return false;
    // every id of a core is accounted for: its modes, the half's own bond, a value of the bond between the halves
    for (int h = 0; h < 2; ++h)
        for (const Core& c : cores[h])
            for (int i : net.tensors[size_t(c.t)].idx)
                if (ext[size_t(i)] > 1 && i != c.m && i != c.n && i != inner[h] && !contains(bond, i)) return false;
    auto x_stride = [&](const std::vector<int>& layout, int id) {
        int64_t st = 1;
        for (size_t j = layout.size(); j-- > 0 && layout[j] != id;) st *= ext[size_t(layout[j])];
        return st;
    };
    int64_t best = 0;
    struct Pick {
        int cfg, first, res;
    } pick{-1, 0, 0};
    auto of_half = [&](int first, int w) { return w == 0 ? first : 1 - first; };
    // the resident core of half h is the one that carries bond[res], the streamed one must not
    auto resident = [&](int h, int res) {
        const bool c0 = contains(net.tensors[size_t(cores[h][0].t)].idx, bond[size_t(res)]);
        const bool c1 = contains(net.tensors[size_t(cores[h][1].t)].idx, bond[size_t(res)]);
        return c0 == c1 ? -1 : c0 ? 0 : 1;
    };
    for (int first = 0; first < 2; ++first)
        for (int res = 0; res < int(bond.size()); ++res) {
            const int i0 = resident(of_half(first, 0), res), i1 = resident(of_half(first, 1), res);
            if (i0 < 0 || i1 < 0) continue;
            if (bond.size() == 2) {
                const int j0 = resident(of_half(first, 0), 1 - res), j1 = resident(of_half(first, 1), 1 - res);
                if (j0 != 1 - i0 || j1 != 1 - i1) continue;
            }
            const Core &R0 = cores[of_half(first, 0)][i0], &S0 = cores[of_half(first, 0)][1 - i0];
            const Core &R1 = cores[of_half(first, 1)][i1], &S1 = cores[of_half(first, 1)][1 - i1];
            const int64_t K0 = R0.N * S0.N, A = R1.N * S1.N, O1 = R0.M * S0.M, C1 = R1.M * S1.M;
            if (S0.N % 4 || K0 % 8 || A % 4) continue;
            const int64_t t[2][2] = {{R0.M * R0.N / 16, S0.M * S0.N / 16}, {R1.M * R1.N / 16, S1.M * S1.N / 16}};
            for (int c = 0; c < kDirectConfigs; ++c) {
                const int* g = kDirectConfig[c];
                const int at = g[0], ks = g[1], o1w = g[2], o2w = g[3], w1 = g[4], as = (at + 1) / 2;
                if ((g[11] ? S1.N : R1.N) % 4) continue;
                if (A > 16 * at || K0 > 32 * ks || O1 > 16 * o1w * w1 || C1 > 16 * o2w * (4 / w1)) continue;
                if (t[0][1] > g[5] * g[6] || t[0][0] > (4 / g[5]) * g[7] || t[1][1] > g[8] * g[9] || t[1][0] > (4 / g[8]) * g[10]) continue;
                const int64_t mfmas = 4 * (int64_t(steps) * (g[6] * g[7] + g[9] * g[10]) + o1w * (at * ks + o2w * as));
                // at least 35 % of it real, as in kron_shape
                const double real = double(longest) * double(O1 * K0 + C1 * A) + double(O1) * double(A) * double(K0 + C1);
                if (real < 0.35 * double(mfmas) * 8192.0) continue;
                if (pick.cfg < 0 || mfmas < best) {
                    pick = {c, first, res};
                    best = mfmas;
                }
            }
        }
    if (pick.cfg < 0) return false;
    const int* g = kDirectConfig[pick.cfg];
    *out = DirectPlan();
    out->cfg = pick.cfg;
    out->steps = steps;
    std::vector<int64_t> padded = ext;
    for (int w = 0; w < 2; ++w) padded[size_t(inner[w])] = 32 * steps;
    const int res_id = bond[size_t(pick.res)], str_id = bond.size() == 2 ? bond[size_t(1 - pick.res)] : -1;
    out->n_res = ext[size_t(res_id)];
    out->n_str = str_id >= 0 ? ext[size_t(str_id)] : 1;
    for (int w = 0; w < 2; ++w) {
        const int h = of_half(pick.first, w), i = resident(h, pick.res);
        const Core &R = cores[h][i], &Q = cores[h][1 - i];
        const bool rows_streamed = w == 0 || g[11];
        const Core &row = rows_streamed ? Q : R, &col = rows_streamed ? R : Q;
        for (int side = 0; side < 2; ++side) {
            const Core& c = side == 0 ? R : Q;
            std::vector<int> ids;
            const int id = side == 0 ? res_id : str_id;
            if (id >= 0) ids.push_back(id);
            if (c.t == row.t) {
                ids.push_back(c.m);
                ids.push_back(c.n);
            } else {
                ids.push_back(c.n);
                ids.push_back(c.m);
            }
            out->src[w][side] = source_op(net, padded, c.t, ids, {inner[h]});
            out->tiles[w][side] = c.M * c.N / 16;
            if (out->src[w][side].R > (int64_t(1) << 24)) return false;
        }
        // o = (rows' m, columns' m), k or a = (columns' n, rows' n)
        const int64_t O = row.M * col.M, K = row.N * col.N, k_steps = w == 0 ? g[1] : (g[0] + 1) / 2;
        std::vector<int32_t>&y = w == 0 ? out->yrow : out->ycol, &x = w == 0 ? out->xcol : out->xrow;
        std::vector<uint32_t> at_o, at_k;               // a position is o's share and k's
        const int64_t y_row = x_stride(net.y_idx, row.m), y_col = x_stride(net.y_idx, col.m), x_row = x_stride(net.x_idx, row.n), x_col = x_stride(net.x_idx, col.n);
        for (int64_t o = 0; o < O; ++o) {
            y.push_back(int32_t(o / col.M * y_row + o % col.M * y_col));
            at_o.push_back(uint32_t(direct_position(w, o, 0, k_steps) / 8));
        }
        for (int64_t k = 0; k < K; ++k) {
            x.push_back(int32_t(k / row.N * x_col + k % row.N * x_row));
            at_k.push_back(uint32_t(direct_position(w, 0, k, k_steps) / 8));      // (four k from a multiple of 4 on are 8 bytes)
        }
        const uint32_t rows = uint32_t(row.M * row.N), cols = uint32_t(col.M * col.N);
        std::vector<uint32_t> col_o, col_k;
        for (uint32_t n = 0; n < uint32_t(col.N); ++n)
            for (uint32_t m = 0; m < uint32_t(col.M); ++m) {
                col_o.push_back(m);
                col_k.push_back(n * uint32_t(row.N));
            }
        out->unit[w].resize(size_t(rows / 16) * (cols / 16) * 64);
        uint16_t* unit = out->unit[w].data();
        for (uint32_t r = 0; r < rows; r += 16)
            for (uint32_t c = 0; c < cols; c += 16)
                for (uint32_t fr = r; fr < r + 16; fr += 4) {
                    const uint32_t *o = &at_o[fr / uint32_t(row.N) * uint32_t(col.M)], *k = &at_k[fr % uint32_t(row.N)];
                    for (uint32_t fc = c; fc < c + 16; ++fc) *unit++ = uint16_t(o[col_o[fc]] + k[col_k[fc]]);
                }
        (w == 0 ? out->O1 : out->C1) = O;
        (w == 0 ? out->K0 : out->A) = K;
    }
    out->x_vec8 = run_length(out->xcol, 8) == 8 && all_multiple_of(out->xrow, 8);
    return true;
}

}  // namespace tn
