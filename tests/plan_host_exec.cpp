// Test-only host executor of a contraction plan, in double precision.
//
// It walks the planner's steps exactly as the GPU kernels do - pack the
// parameter tensor as B[c][k] from the gather recipe, read A through the plain
// or table addressing, scatter the result through crow/ccol - so that the CPU
// test-suite can check the planner's order, layouts, tables and packing recipes
// against the oracle without a GPU. Never linked into the product library.
#include <cstdint>
#include <vector>

#include "../paper_2602_01613_amd/csrc/tn_matrix.hpp"

extern "C" int plan_host_forward(const tn_linear_desc* d, const double* const* tensors, const double* x,
                                 double* y, int64_t tokens) {
    tn::Plan p;
    int rc = tn::make_plan(d, &p);
    if (rc != TN_OK) return rc;
    // tensors merged at create time, in double
    std::vector<std::vector<double>> virt;
    auto source = [&](int slot) -> const double* {
        return slot < p.n_caller_tensors ? tensors[slot] : virt[size_t(slot - p.n_caller_tensors)].data();
    };
    auto offset_of = [](int64_t flat, const std::vector<tn::GatherDim>& dims) {
        int64_t off = 0;
        for (int j = int(dims.size()) - 1; j >= 0; --j) {
            off += (flat % dims[size_t(j)].extent) * dims[size_t(j)].stride;
            flat /= dims[size_t(j)].extent;
        }
        return off;
    };
    for (const tn::MergeOp& m : p.merges) {
        const double* P = source(m.p_slot);
        const double* Q = source(m.q_slot);
        std::vector<double> out(size_t(m.R * m.C), 0.0);
        for (int64_t r = 0; r < m.R; ++r)
            for (int64_t c = 0; c < m.C; ++c) {
                double acc = 0;
                for (int64_t k = 0; k < m.K; ++k)
                    acc += P[offset_of(r, m.rdims) + offset_of(k, m.kp)] * Q[offset_of(c, m.cdims) + offset_of(k, m.kq)];
                out[size_t(r * m.C + c)] = acc;
            }
        virt.push_back(std::move(out));
    }
    std::vector<double> cur(x, x + tokens * p.N), nxt;
    for (size_t s = 0; s < p.steps.size(); ++s) {
        const tn::Step& st = p.steps[s];
        std::vector<double> B(size_t(st.C * st.K), 0.0);
        for (int64_t c = 0; c < st.C; ++c)
            for (int64_t k = 0; k < st.K; ++k) {
                int64_t off = 0, rem = k;
                for (int j = int(st.kdims.size()) - 1; j >= 0; --j) {
                    off += (rem % st.kdims[j].extent) * st.kdims[j].stride;
                    rem /= st.kdims[j].extent;
                }
                rem = c;
                for (int j = int(st.cdims.size()) - 1; j >= 0; --j) {
                    off += (rem % st.cdims[j].extent) * st.cdims[j].stride;
                    rem /= st.cdims[j].extent;
                }
                double v = 0;
                for (int64_t a = 0; a < st.trace_extent; ++a) v += source(st.slot)[off + a * st.trace_stride];
                B[size_t(c * st.K + k)] = v;
            }
        nxt.assign(size_t(tokens * st.c_tok_stride), 0.0);
        // every output position must be written exactly once
        std::vector<char> hit(nxt.size(), 0);
        for (int64_t t = 0; t < tokens; ++t)
            for (int64_t r = 0; r < st.R; ++r)
                for (int64_t c = 0; c < st.C; ++c) {
                    double acc = 0;
                    for (int64_t k = 0; k < st.K; ++k) {
                        int64_t ao = t * st.a_tok_stride + (st.a_plain ? r * st.K + k : int64_t(st.arow[r]) + st.acol[k]);
                        acc += cur[size_t(ao)] * B[size_t(c * st.K + k)];
                    }
                    int64_t oo = t * st.c_tok_stride + st.crow[r] + st.ccol[c];
                    if (oo < 0 || oo >= int64_t(nxt.size()) || hit[size_t(oo)]) return -100 - int(s);
                    hit[size_t(oo)] = 1;
                    nxt[size_t(oo)] = acc;
                }
        for (char h : hit)
            if (!h) return -200 - int(s);
        cur.swap(nxt);
    }
    if (int64_t(cur.size()) != tokens * p.M) return -300;
    for (size_t i = 0; i < cur.size(); ++i) y[i] = cur[i];
    return 0;
}

// vectorisation hints of a step, for the tests: field 0 c_vec, 1 r_vec, 2 a_plain, 3 merges in the plan
extern "C" int plan_host_step_hint(const tn_linear_desc* d, int step, int field, int64_t* value) {
    tn::Plan p;
    int rc = tn::make_plan(d, &p);
    if (rc != TN_OK) return rc;
    if (step < 0 || step >= int(p.steps.size())) return TN_ERR_INVALID_ARG;
    const tn::Step& st = p.steps[size_t(step)];
    *value = field == 0 ? st.c_vec : field == 1 ? st.r_vec : field == 2 ? int64_t(st.a_plain) : int64_t(p.merges.size());
    return 0;
}

// Buffers of the launches of one pass (see tn::launch_schedule) with the chained factor pairs the plan
// allows: in_buf / out_buf receive one entry per launch (-1 = x, -2 = y, 0 / 1 = workspace buffers),
// steps the number of steps each launch covers. Returns the number of launches, or a negative status.
extern "C" int plan_host_launch_buffers(const tn_linear_desc* d, int cap, int* in_buf, int* out_buf, int* steps) {
    tn::Plan p;
    int rc = tn::make_plan(d, &p);
    if (rc != TN_OK) return rc;
    const std::vector<tn::LaunchIO> sched = tn::launch_schedule(p.steps.size(), tn::chain2_pairs(p));
    if (int(sched.size()) > cap) return TN_ERR_INVALID_ARG;
    for (size_t i = 0; i < sched.size(); ++i) {
        in_buf[i] = sched[i].in;
        out_buf[i] = sched[i].out;
        steps[i] = sched[i].steps;
    }
    return int(sched.size());
}

static double source_value(const double* const* tensors, const tn::SourceOp& o, int64_t r, int64_t k) {
    int64_t off = 0;
    auto walk = [&](const std::vector<tn::SourceDim>& dims, int64_t f) {
        for (size_t j = dims.size(); j-- > 0;) {
            const int64_t digit = f % dims[j].extent;
            if (digit >= dims[j].limit) return false;
            off += digit * dims[j].stride;
            f /= dims[j].extent;
        }
        return true;
    };
    return walk(o.rows, r) && walk(o.ks, k) ? tensors[o.slot][off] : 0.0;
}

// The order that contracts the parameter tensors with each other first (tn_matrix.hpp), in double: W [M][N] as the packed
// operand says it. Returns 1 when the layer has no such plan, negative when an output position is written twice or never
// or lies outside.
extern "C" int plan_host_matrix(const tn_linear_desc* d, const double* const* tensors, double* w_out) {
    tn::Plan net;
    tn::MatrixPlan m;
    if (!tn::make_matrix_plan(d, &net, &m)) return 1;
    auto operand = [&](const tn::SourceOp& o, int64_t r, int64_t k) { return source_value(tensors, o, r, k); };
    int bad = 0;
    auto store = [&](std::vector<double>* out, std::vector<char>* hit, const tn::Product& p, int64_t r, int64_t c, double v) {
        const int64_t o = int64_t(p.row_off[size_t(r)]) + p.col_off[size_t(c)];
        if (o < 0 || o >= int64_t(out->size()) || (*hit)[size_t(o)]) {
            bad = -1;
            return;
        }
        (*hit)[size_t(o)] = 1;
        (*out)[size_t(o)] = v;
    };
    std::vector<double> half[2];       // [modes][bond], in the half's own layout
    for (int h = 0; h < 2; ++h) {
        const tn::MatrixHalf& H = m.half[h];
        if (H.tensors.size() == 1) {
            half[h].assign(size_t((H.F + 255) / 256 * 256 * m.Krp), 0.0);
            for (int64_t f = 0; f < H.F; ++f)
                for (int64_t k = 0; k < H.keep.K; ++k)
                    half[h][size_t(h == 0 ? f * m.Krp + k : tn::packed_col(f, m.Krp / 16) + tn::packed_k(k))] = operand(H.keep, f, k);
            continue;
        }
        half[h].assign(size_t(H.build.out_elems), 0.0);
        std::vector<char> hit(half[h].size(), 0);
        for (int64_t r = 0; r < H.build.R; ++r)
            for (int64_t c = 0; c < H.build.C; ++c) {
                double acc = 0;
                for (int64_t k = 0; k < H.build.K; ++k) acc += operand(H.build.a, r, k) * operand(H.build.b, c, k);
                store(&half[h], &hit, H.build, r, c, acc);
            }
        int64_t n = 0;
        for (char v : hit) n += v;
        if (n != H.F * m.Krp) return -2;
    }
    std::vector<double> w(size_t(m.w_elems), 0.0);
    std::vector<char> hit(w.size(), 0);
    for (int64_t r = 0; r < m.w.R; ++r)
        for (int64_t c = 0; c < m.w.C; ++c) {
            double acc = 0;
            for (int64_t k = 0; k < m.Krp; ++k)
                acc += half[0][size_t(r * m.Krp + k)] * half[1][size_t(tn::packed_col(c, m.Krp / 16) + tn::packed_k(k))];
            store(&w, &hit, m.w, r, c, acc);
        }
    if (bad) return bad;
    for (int64_t i = 0; i < m.M; ++i)
        for (int64_t j = 0; j < m.N; ++j) {
            const size_t o = size_t(tn::packed_col(i, m.N / 16) + tn::packed_k(j));
            if (!hit[o]) return -3;
            w_out[i * m.N + j] = w[o];
        }
    return 0;
}

// Gradients of sum(dW * W) with respect to the parameter tensors on the same cut, in double. dw [M][N]; grads receives every
// tensor's gradient in the caller's layout. Returns 1 when the layer has no such plan.
extern "C" int plan_host_matrix_grad(const tn_linear_desc* d, const double* const* tensors, const double* dw, double* const* grads) {
    tn::Plan net;
    tn::MatrixPlan m;
    tn::MatrixGrad g;
    if (!tn::make_matrix_plan(d, &net, &m) || !tn::make_matrix_grad(net, m, &g)) return 1;
    const int64_t F[2] = {m.half[0].F, m.half[1].F};
    std::vector<double> D(size_t(m.M * m.N), 0.0);
    std::vector<char> hit(D.size(), 0);
    for (int64_t i = 0; i < m.M; ++i)
        for (int64_t j = 0; j < m.N; ++j) {
            const int64_t o = int64_t(g.dw_row[size_t(i)]) + g.dw_col[size_t(j)];
            if (o < 0 || o >= int64_t(D.size()) || hit[size_t(o)]) return -1;
            hit[size_t(o)] = 1;
            D[size_t(o)] = dw[i * m.N + j];
        }
    auto put = [&](const tn::GradOut& o, int64_t r, int64_t c, double v) {
        int64_t off = 0;
        for (size_t j = o.cols.size(); j-- > 0;) {
            off += c % o.cols[j].extent * o.cols[j].stride;
            c /= o.cols[j].extent;
        }
        for (size_t j = o.rows.size(); j-- > 0;) {
            off += r % o.rows[j].extent * o.rows[j].stride;
            r /= o.rows[j].extent;
        }
        grads[o.slot][off] = v;
    };
    for (int h = 0; h < 2; ++h) {
        const tn::MatrixGradHalf &G = g.half[h], &O = g.half[1 - h];
        // the other half: packed, columns bond, k = its modes
        std::vector<double> op(size_t((m.Kr + 255) / 256 * 256 * F[1 - h]), 0.0);
        if (O.pair) {
            std::vector<char> seen(op.size(), 0);
            for (int64_t r = 0; r < O.op.R; ++r)
                for (int64_t c = 0; c < O.op.C; ++c) {
                    double acc = 0;
                    for (int64_t k = 0; k < O.op.K; ++k) acc += source_value(tensors, O.op.a, r, k) * source_value(tensors, O.op.b, c, k);
                    const int64_t o = int64_t(O.op.row_off[size_t(r)]) + O.op.col_off[size_t(c)];
                    if (o < 0 || o >= int64_t(op.size()) || seen[size_t(o)]) return -2;
                    seen[size_t(o)] = 1;
                    op[size_t(o)] = acc;
                }
        } else {
            for (int64_t c = 0; c < m.Kr; ++c)
                for (int64_t k = 0; k < F[1 - h]; ++k)
                    op[size_t(tn::packed_col(c, F[1 - h] / 16) + tn::packed_k(k))] = source_value(tensors, O.op_keep, c, k);
        }
        std::vector<double> dh(size_t(F[h] * m.Kr), 0.0);
        std::vector<char> seen(dh.size(), 0);
        for (int64_t f = 0; f < F[h]; ++f)
            for (int64_t c = 0; c < m.Kr; ++c) {
                double acc = 0;
                for (int64_t k = 0; k < F[1 - h]; ++k)
                    acc += D[size_t(h == 0 ? f * F[1] + k : k * F[1] + f)] * op[size_t(tn::packed_col(c, F[1 - h] / 16) + tn::packed_k(k))];
                if (!G.pair) {
                    put(G.out_a, f, c, acc);
                    continue;
                }
                const int64_t o = int64_t(G.row_off[size_t(f)]) + G.col_off[size_t(c)];
                if (o < 0 || o >= int64_t(dh.size()) || seen[size_t(o)]) return -3;
                seen[size_t(o)] = 1;
                dh[size_t(o)] = acc;
            }
        if (!G.pair) continue;
        const int64_t S = G.a.R;
        for (int64_t c = 0; c < S; ++c) {
            for (int64_t f = 0; f < G.F1; ++f) {
                double acc = 0;
                for (int64_t k = 0; k < G.F2; ++k) acc += dh[size_t(f * G.F2 + k)] * source_value(tensors, G.b, c, k);
                put(G.out_a, f, c, acc);
            }
            for (int64_t f = 0; f < G.F2; ++f) {
                double acc = 0;
                for (int64_t k = 0; k < G.F1; ++k) acc += dh[size_t(k * G.F2 + f)] * source_value(tensors, G.a, c, k);
                put(G.out_b, f, c, acc);
            }
        }
    }
    return 0;
}

// The slices of the Kronecker-sum kernel as products of the cores, in double, put together to W [M][N] the way the kernel reads
// them. Returns 1 when the layer has no such plan.
extern "C" int plan_host_slices(const tn_linear_desc* d, const double* const* tensors, double* w_out) {
    tn_linear_desc halves = *d;
    halves.flags |= TN_FLAG_MERGE_HALVES | (20 << TN_FLAG_VARIANT_SHIFT);
    tn::Plan q, net;
    tn::KronDims k;
    tn::SlicePlan s;
    if (tn::make_plan(&halves, &q) != TN_OK || q.steps.size() != 2 || q.merges.size() != 2 || !tn::kron_shape(q, &k) ||
        tn::build_network(d, &net) != TN_OK || !tn::make_slice_plan(net, q, k, &s))
        return 1;
    const int *cfg = tn::kKronConfig[k.cfg], at = cfg[0], ks0 = cfg[1], o2t = cfg[2], o1t = cfg[3];
    std::vector<double> H[2];
    for (int h = 0; h < 2; ++h) {
        const tn::Product& p = s.half[h];
        H[h].assign(size_t(p.out_elems), 1e300);               // what is not written must not be used
        std::vector<char> hit(H[h].size(), 0);
        for (int64_t r = 0; r < p.R; ++r)
            for (int64_t c = 0; c < p.C; ++c) {
                double acc = 0;
                for (int64_t e = 0; e < p.K; ++e) acc += source_value(tensors, p.a, r, e) * source_value(tensors, p.b, c, e);
                const int64_t o = int64_t(p.row_off[size_t(r)]) + p.col_off[size_t(c)];
                if (o < 0 || o >= int64_t(H[h].size()) || hit[size_t(o)]) return -1;
                hit[size_t(o)] = 1;
                H[h][size_t(o)] = acc;
            }
    }
    auto h0 = [&](int64_t o1, int64_t rho, int64_t kk) {
        const int64_t chunk = o1 / (32 * o1t), t = o1 % (32 * o1t) / 32, l = o1 % 32 + 32 * (kk % 16 / 8);
        return H[0][size_t((((chunk * k.P + rho) * o1t + t) * ks0 + kk / 16) * 512 + l * 8 + kk % 8)];
    };
    auto h1 = [&](int64_t o2, int64_t rho, int64_t a) {
        const int64_t m = a % 16, e = m / 8 * 4 + m % 4, l = o2 % 32 + 32 * (m % 8 / 4);
        return H[1][size_t(((rho * o2t + o2 / 32) * 2 * at + a / 16) * 512 + l * 8 + e)];
    };
    // the kernel multiplies padded k and a by zeros of x: they have to hold numbers
    for (int64_t rho = 0; rho < k.P; ++rho) {
        for (int64_t o = 0; o < k.O1; ++o)
            for (int64_t kk = k.K0; kk < 16 * ks0; ++kk)
                if (h0(o, rho, kk) != 0.0) return -2;
        for (int64_t o = 0; o < k.C1; ++o)
            for (int64_t a = k.A; a < 32 * at; ++a)
                if (h1(o, rho, a) != 0.0) return -3;
    }
    for (int64_t o1 = 0; o1 < k.O1; ++o1)
        for (int64_t o2 = 0; o2 < k.C1; ++o2)
            for (int64_t a = 0; a < k.A; ++a)
                for (int64_t kk = 0; kk < k.K0; ++kk) {
                    double acc = 0;
                    for (int64_t rho = 0; rho < k.P; ++rho) acc += h0(o1, rho, kk) * h1(o2, rho, a);
                    w_out[(int64_t(s.yrow[size_t(o1)]) + s.ycol[size_t(o2)]) * q.N + s.xrow[size_t(a)] + s.xcol[size_t(kk)]] = acc;
                }
    return 0;
}

// One token through the plan with the slices made on chip, tile by tile as kernels/krondirect.hpp walks it. 0 or, with no such plan, 1;
// *cfg: the instantiation.
extern "C" int plan_host_direct(const tn_linear_desc* d, const double* const* tensors, const double* x, double* y, int* cfg) {
    tn_linear_desc halves = *d;
    halves.flags |= TN_FLAG_MERGE_HALVES;
    tn::Plan q, net;
    tn::DirectPlan s;
    int pairs[2][2];
    if (tn::make_plan(&halves, &q) != TN_OK || q.steps.size() != 2 || q.merges.size() != 2 || tn::build_network(d, &net) != TN_OK ||
        !tn::merged_tensors(net, q, pairs) || !tn::make_direct_plan(net, pairs, &s))
        return 1;
    const int* g = tn::kDirectConfig[s.cfg];
    *cfg = s.cfg;
    const int64_t steps[2] = {g[1], (g[0] + 1) / 2}, columns[2] = {s.O1, s.C1}, contracted[2] = {s.K0, s.A};
    for (int64_t m = 0; m < net.M; ++m) y[m] = 0;
    std::vector<double> D(size_t(s.A));
    for (int64_t rr = 0; rr < s.n_res; ++rr)
        for (int64_t rs = 0; rs < s.n_str; ++rs) {
            std::vector<double> L[2];
            for (int w = 0; w < 2; ++w) {
                const int rows = w == 0 || g[11] ? 1 : 0;          // the side (resident, streamed) of the rows
                const tn::SourceOp &R = s.src[w][rows], &C = s.src[w][1 - rows];
                const int64_t slab[2] = {rr, rs}, tr = s.tiles[w][rows], tc = s.tiles[w][1 - rows];
                if (int64_t(s.unit[w].size()) != tr * tc * 64) return -1;
                L[w].assign(size_t((columns[w] + 15) / 16 * steps[w] * 512), 0.0);
                std::vector<char> hit(L[w].size(), 0);
                for (int64_t r = 0; r < tr; ++r)
                    for (int64_t c = 0; c < tc; ++c)
                        for (int64_t l = 0; l < 64; ++l)
                            for (int64_t v = 0; v < 4; ++v) {
                                const int64_t fr = (slab[rows] * tr + r) * 16 + 4 * (l / 16) + v, fc = (slab[1 - rows] * tc + c) * 16 + l % 16;
                                double acc = 0;
                                for (int64_t e = 0; e < R.K; ++e) acc += source_value(tensors, R, fr, e) * source_value(tensors, C, fc, e);
                                const size_t at = size_t(s.unit[w][size_t((r * tc + c) * 64 + l)]) * 4 + size_t(v);
                                if (at >= L[w].size() || hit[at]) return -2;
                                hit[at] = 1;
                                L[w][at] = acc;
                            }
                int64_t n = 0;
                for (char h : hit) n += h;
                if (n != columns[w] * contracted[w]) return -3;
            }
            for (int64_t o1 = 0; o1 < s.O1; ++o1) {
                for (int64_t a = 0; a < s.A; ++a) {
                    D[size_t(a)] = 0;
                    for (int64_t k = 0; k < s.K0; ++k)
                        D[size_t(a)] += x[s.xrow[size_t(a)] + s.xcol[size_t(k)]] * L[0][size_t(tn::direct_position(0, o1, k, steps[0]) / 2)];
                }
                for (int64_t o2 = 0; o2 < s.C1; ++o2)
                    for (int64_t a = 0; a < s.A; ++a)
                        y[s.yrow[size_t(o1)] + s.ycol[size_t(o2)]] += D[size_t(a)] * L[1][size_t(tn::direct_position(1, o2, a, steps[1]) / 2)];
            }
        }
    return 0;
}

// The plan of the gradients alone: 0, or 1 when the layer has none.
extern "C" int plan_host_matrix_grad_plan(const tn_linear_desc* d) {
    tn::Plan net;
    tn::MatrixPlan m;
    tn::MatrixGrad g;
    return tn::make_matrix_plan(d, &net, &m) && tn::make_matrix_grad(net, m, &g) ? 0 : 1;
}
