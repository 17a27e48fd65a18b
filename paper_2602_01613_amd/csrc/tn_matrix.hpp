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
        if (total > kMatrixMaxElems) return false;
    }
    std::vector<int64_t> sums(1, 0);       // of every position over the ids so far
    for (size_t j = 0; j < ids.size(); ++j) {
        std::vector<int64_t>& v = (*out)[ids[j]];
        v.clear();
        for (int64_t d = 0; d < ext[size_t(ids[j])]; ++d) v.push_back(f(d * weight[j]));
        std::vector<int64_t> next;
        next.reserve(sums.size() * v.size());
        for (int64_t s : sums)
            for (int64_t o : v) next.push_back(s + o);
        sums.swap(next);
    }
    for (int64_t p = 0; p < total; ++p)
        if (sums[size_t(p)] != f(p)) return false;
    return true;
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
        std::vector<int32_t> next;
        next.reserve(tab.size() * v.size());
        for (int32_t o : tab)
            for (int64_t d : v) next.push_back(o + int32_t(d));
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

// The plan for one cut of the network: the tensors of group[0] and of group[1], one or two each.
inline bool matrix_plan_of_cut(const Plan& net, const std::vector<int> (&group)[2], MatrixPlan* m) {
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
    if (m->N % 64 || m->M % 8 || m->N >= (int64_t(1) << 21)) return false;
    for (int i : open[1 - q])
        if (contains(open[q], i)) m->bond.push_back(i);
    if (m->bond.empty() || m->bond.size() > 2) return false;
    for (int i : m->bond) m->Kr *= net.extent[size_t(i)];
    m->Krp = round64(m->Kr);
    // a bond of one index may be laid out longer than it is (zeros); of two, it has to be whole tiles
    std::vector<int64_t> ext = net.extent;
    if (m->bond.size() == 1) ext[size_t(m->bond[0])] = m->Krp;
    else if (m->Kr != m->Krp) return false;
    DigitOffsets wt;
    const int64_t nks = m->N / 16;
    if (!digit_offsets(net.y_idx, ext, [&](int64_t c) { return packed_col(c, nks); }, &wt) || !digit_offsets(net.x_idx, ext, packed_k, &wt))
        return false;
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
    bool found = false;
    for (int first = 0; first < (d->format == TN_FORMAT_TR ? n : 1); ++first)
        for (int len = 1; len < n; ++len) {
            if (len > 2 || n - len > 2) continue;
            std::vector<int> group[2];
            for (int j = 0; j < n; ++j) group[j < len ? 0 : 1].push_back((first + j) % n);
            MatrixPlan c;
            if (matrix_plan_of_cut(*net, group, &c) && (!found || c.Kr < m->Kr)) {
                *m = c;
                found = true;
            }
        }
    return found;
}

}  // namespace tn
