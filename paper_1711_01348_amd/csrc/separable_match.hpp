// Recognition of sums of products of two functions (separable.hpp).  Host only; included by families.cpp.
#pragma once
#include <algorithm>
#include <cstring>

#include "plan.hpp"
#include "separable.hpp"

namespace tad {

namespace {

struct Factor {
    int node;
    bool inverse;
    uint32_t reads;   // operands
};

uint32_t operands_of(const Graph &g, const std::vector<int> &alias, int node) {
    const int t = alias[node];
    const Node &nd = g.nodes[t];
    if (nd.op == P_ARG) return 1u << nd.k;
    uint32_t m = 0;
    if (nd.a >= 0) m |= operands_of(g, alias, nd.a);
    if (nd.b >= 0) m |= operands_of(g, alias, nd.b);
    return m;
}

// The factors of a node: inputs of its products, quotients and negations.  False: more than a program can hold.
bool collect_factors(Graph &g, const std::vector<int> &alias, int node, bool inverse, std::vector<Factor> &out) {
    const int t = alias[node];
    const Node nd = g.nodes[t];
    if (out.size() > 16) return false;
    switch (nd.op) {
    case P_MUL: return collect_factors(g, alias, nd.a, inverse, out) && collect_factors(g, alias, nd.b, inverse, out);
    case P_DIV: return collect_factors(g, alias, nd.a, inverse, out) && collect_factors(g, alias, nd.b, !inverse, out);
    case P_NEG:
        if (!collect_factors(g, alias, nd.a, inverse, out)) return false;
        out.push_back(Factor{-1, false, 0});   // a sign
        return true;
    default: out.push_back(Factor{t, inverse, operands_of(g, alias, t)}); return true;
    }
}

// One expression from the factors of a side: (product of the numerators) / (product of the denominators).
int side_expression(Graph &g, const std::vector<Factor> &factors) {
    int num = -1, den = -1;
    bool negative = false;
    for (const Factor &f : factors) {
        if (f.node < 0) { negative = !negative; continue; }
        int &to = f.inverse ? den : num;
        to = to < 0 ? f.node : g.add(P_MUL, to, f.node);
    }
    if (num < 0) num = g.constant(1.0);
    const int q = den < 0 ? num : g.add(P_DIV, num, den);
    return negative ? g.add(P_NEG, q) : q;
}

// every pair of indices reads an element of its own, numbered alike
bool pairs_are_elements(const tad_plan &sub, int p) {
    if (sub.arg_count[p] != sub.f_count) return false;
    int64_t stride = 1;
    for (int d = sub.expr.n_f - 1; d >= 0; --d) {
        if (sub.expr.f_shape[d] != 1 && sub.fwd.off[p][d] != stride) return false;
        stride *= sub.expr.f_shape[d];
    }
    return true;
}

// Is the forward pass of the general kernels the faster one?  General / dense, M x N x K:
//   few long sums, a workgroup each there and three launches here: 16 x 16 x 3000 9.5 / 11.4 us (64 bits 9.5 / 13.2), as a program with
//   exp 12.1 / 14.3, 64 x 16 x 1100 in 64 bits 9.8 / 13.4; 33 x 65 x 5000 48 / 14, 16 x 16 x 5000 with exp 15.8 / 14.7, 16 x 16 x 1000, a
//   thread each there, 55 / 12;
//   tanh of short sums of many results (its program takes longer here), 64 bits 10000 x 33 x 16 11 / 16, 100000 x 17 x 9 24 / 55, x 129 x 9
//   140 / 243, 100000 x 16 x 17 31 / 54, 10000 x 129 x 33 45 / 32, 100000 x 33 x 33 109 / 104, 10000 x 17 x 16 9.8 / 10.1; 32 bits
//   10000 x 129 x 16 12.8 / 17.8, 100000 x 17 x 16 24 / 27, 100000 x 16 x 33 20 / 32, 100001 x 16 x 65 34 / 41, 10000 x 64 x 16 9.7 / 8.8,
//   100000 x 17 x 33 49 / 34.
bool forward_general(bool f64, bool tanh_dot, int64_t M, int64_t N, int64_t K) {
    if (K >= 1024 && M * N * K <= ((int64_t)1 << (tanh_dot ? 21 : 20))) return true;
    if (!tanh_dot || M * N < ((int64_t)1 << (f64 ? 18 : 20))) return false;
    const int64_t least = std::min(M, N);
    return K <= 16 || (f64 ? least <= 33 && K <= 28 : least <= 16 && K < 72);
}

}  // namespace

void match_separable(tad_plan &pl) {
    SepPlan &sp = pl.sep;
    sp = SepPlan{};
    const tad_expr &e = pl.expr;
    if (pl.flags & (TAD_PLAN_GENERIC_ONLY | TAD_PLAN_KEEP_PROGRAM)) return;
    if (pl.has_alias || e.n_constraints > 0 || e.n_sum < 1 || e.n_f < 2) return;
    const bool program = e.body == TAD_BODY_PROGRAM && pl.fwd_family == TAD_FAMILY_PROGRAM;
    if (!program && !(e.body == TAD_BODY_TANH_DOT && pl.fwd_family == TAD_FAMILY_GENERIC)) return;
    for (int s = 0; s < e.n_sum; ++s)
        if (e.sum_lo[s] != 0) return;
    const int n_ops = (int)pl.args.size();

    // ---- factors ---------------------------------------------------------------------------------------------------
    tad_expr text = e;
    if (!program) {
        std::vector<tad_op> in, out;
        if (!builtin_body_programs(e.body, in, out)) return;
        text.n_operands = n_ops;
        text.n_inner = (int)in.size();
        text.n_outer = (int)out.size();
        std::copy(in.begin(), in.end(), text.inner);
        std::copy(out.begin(), out.end(), text.outer);
        uint32_t wanted = 0;
        for (int p = 0; p < n_ops; ++p) wanted |= pl.args[p].needs_grad ? 1u << p : 0u;
        if (build_program_body(text, sp.prog, 0, wanted)) return;
    } else {
        sp.prog = pl.prog;
    }
    Graph g;
    const int root = parse_postfix(text.inner, text.n_inner, false, n_ops, g);
    if (root < 0) return;
    const std::vector<int> alias = simplify(g);
    std::vector<Factor> factors;
    if (!collect_factors(g, alias, root, false, factors)) return;

    // ---- function indices of the two sides ------------------------------------------------------------------------
    int64_t extent[TAD_MAX_EXT];
    for (int d = 0; d < pl.n_ext; ++d) extent[d] = pl.hi[d] - pl.lo[d] + 1;
    auto moves = [&](uint32_t reads, int d) {
        for (int p = 0; p < n_ops; ++p) {
            if (!((reads >> p) & 1u) || extent[d] == 1) continue;
            for (int r = 0; r < pl.args[p].rank; ++r)
                if (pl.args[p].index[r][d] != 0) return true;
        }
        return false;
    };
    std::vector<Factor> of[2];
    int lead = 0;
    for (int split = 1; split < e.n_f && !lead; ++split) {
        bool good = true;
        of[0].clear();
        of[1].clear();
        bool own[2] = {false, false};
        for (const Factor &f : factors) {
            bool in[2] = {false, false};
            for (int d = 0; d < e.n_f; ++d)
                if (moves(f.reads, d)) in[d < split ? 0 : 1] = true;
            good = good && !(in[0] && in[1]);
            own[0] = own[0] || in[0];
            own[1] = own[1] || in[1];
            of[in[1] ? 1 : 0].push_back(f);
        }
        if (good && own[0] && own[1]) lead = split;
    }
    if (!lead) return;
    int64_t M = 1, N = 1, K = 1;
    for (int d = 0; d < pl.n_ext; ++d) (d < lead ? M : d < e.n_f ? N : K) *= extent[d];
    if (M < kProductExtent || N < kProductExtent || K < kProductSum || K >= ((int64_t)1 << 30)) return;
    // Factors are evaluated in 64 bits: of 32-bit operands nothing overflows there that did not in 32 bits, in whatever order
    // the factors are multiplied.  With 64-bit operands the order of the operations has to stay as written: one product
    // of two functions.
    if (pl.dtype == TAD_F64 && (of[0].size() != 1 || of[1].size() != 1 || of[0][0].inverse || of[1][0].inverse)) return;
    sp.M = M; sp.N = N; sp.K = K;

    // ---- the sides ------------------------------------------------------------------------------------------------
    for (int q = 0; q < 2; ++q) {
        SepSide &s = sp.side[q];
        const int at = q == 0 ? 0 : lead, count = q == 0 ? lead : e.n_f - lead;
        s.X = q == 0 ? M : N;
        if (s.X * K > INT32_MAX - 255) return;   // pairs of indices are numbered in 32 bits, 256 per workgroup
        if (count + e.n_sum > TAD_MAX_EXT) return;
        const int node = side_expression(g, of[q]);
        const std::vector<int> simple = simplify(g);
        uint32_t reads = 0, wanted = 0;
        for (const Factor &f : of[q]) reads |= f.reads;
        for (int p = 0; p < n_ops; ++p)
            if (((reads >> p) & 1u) && pl.args[p].needs_grad) wanted |= 1u << p;
        const Node &top = g.nodes[simple[node]];
        int64_t sm = 0, sk = 0;
        if (top.op == P_ARG && product_group_stride(pl.fwd.off[top.k] + at, extent + at, count, sm) &&
            product_group_stride(pl.fwd.off[top.k] + e.n_f, extent + e.n_f, e.n_sum, sk)) {
            s.operand = top.k;
            const bool rows = sm == K && sk == 1, cols = sm == 1 && sk == s.X;
            s.fills = (rows || cols) && pl.arg_count[top.k] == s.X * K;
            s.k_major = !rows && cols;
        }
        if (s.operand < 0 || (!s.fills && wanted)) {
            // the order of the pairs: along the faster index of the first operand that moves along both
            if (s.operand < 0)
                for (int p = 0; p < n_ops; ++p) {
                    const int64_t *off = pl.fwd.off[p];
                    if (!((reads >> p) & 1u) || off[at + count - 1] == 0 || off[pl.n_ext - 1] == 0) continue;
                    const int64_t x = off[at + count - 1] < 0 ? -off[at + count - 1] : off[at + count - 1];
                    const int64_t k = off[pl.n_ext - 1] < 0 ? -off[pl.n_ext - 1] : off[pl.n_ext - 1];
                    s.k_major = x < k;
                    break;
                }
            tad_expr se;
            tad_arg sa[TAD_MAX_ARGS];
            std::memset(&se, 0, sizeof se);
            std::memset(sa, 0, sizeof sa);
            se.body = TAD_BODY_PROGRAM;
            int dims[TAD_MAX_EXT], n = 0;
            if (s.k_major)
                for (int k = 0; k < e.n_sum; ++k) dims[n++] = e.n_f + k;
            for (int d = 0; d < count; ++d) dims[n++] = at + d;
            if (!s.k_major)
                for (int k = 0; k < e.n_sum; ++k) dims[n++] = e.n_f + k;
            se.n_f = n;
            for (int d = 0; d < n; ++d) se.f_shape[d] = extent[dims[d]];
            std::vector<tad_op> ops;
            if (!emit_postfix(g, simple, node, ops, TAD_MAX_PROGRAM)) return;
            int index[TAD_MAX_ARGS];
            for (int p = 0; p < n_ops; ++p) {
                if (!((reads >> p) & 1u)) continue;
                index[p] = (int)s.operands.size();
                tad_arg &a = sa[index[p]];
                s.operands.push_back(p);
                a.rank = pl.args[p].rank;
                a.needs_grad = pl.args[p].needs_grad;
                for (int r = 0; r < a.rank; ++r) {
                    a.shape[r] = pl.args[p].shape[r];
                    for (int d = 0; d < n; ++d) a.index[r][d] = pl.args[p].index[r][dims[d]];
                }
            }
            for (size_t i = 0; i < ops.size(); ++i) {
                se.inner[i] = ops[i];
                if (ops[i].op == TAD_OP_ARG) se.inner[i].iarg = index[ops[i].iarg];
            }
            se.n_inner = (int)ops.size();
            se.outer[0].op = TAD_OP_SUM;
            se.n_outer = 1;
            se.n_operands = (int)s.operands.size();
            if (se.n_operands < 1) return;
            tad_plan *sub = nullptr;
            // KEEP_PROGRAM: the derivatives of the factor are read from its program
            if (derive_plan(&se, sa, se.n_operands, pl.dtype, TAD_PLAN_KEEP_PROGRAM, &sub)) return;
            s.sub.reset(sub);
            if (s.operand < 0 && wanted) {
                Graph gs;
                const int value = parse_postfix(se.inner, se.n_inner, false, se.n_operands, gs);
                std::vector<int> grads, roots{value}, place;
                reverse_accumulate(gs, value, se.n_operands, grads);
                for (int p = 0; p < se.n_operands; ++p)
                    if (sa[p].needs_grad) roots.push_back(grads[p]);
                s.joint_on = lower_joint(gs, roots, s.joint, place);
                size_t at_root = 0;
                s.joint_place[0] = s.joint_on ? place[at_root++] : -1;
                for (int p = 0; p < se.n_operands; ++p) s.joint_place[1 + p] = s.joint_on && sa[p].needs_grad ? place[at_root++] : -1;
            }
        }
        if (s.operand >= 0) {
            s.sm = sm;
            s.sk = sk;
        } else {
            s.sm = s.k_major ? 1 : K;
            s.sk = s.k_major ? s.X : 1;
        }
    }
    // ---- products -------------------------------------------------------------------------------------------------
    const bool f64 = pl.dtype == TAD_F64;
    for (int p = 0; p < n_ops; ++p) {
        if (!((sp.prog.outer_mask >> p) & 1u)) continue;
        sp.outer_linear = sp.outer_linear && product_group_stride(pl.fwd.off[p], extent, lead, sp.outer_r[p]) &&
                          product_group_stride(pl.fwd.off[p] + lead, extent + lead, e.n_f - lead, sp.outer_c[p]);
    }
    sp.identity = sp.prog.outer.n == 1 && sp.prog.outer.op[0] == P_SUM;
    const SepSide &A = sp.side[0], &B = sp.side[1];
    auto wide = [&](const SepSide &s) { return f64 || s.operand < 0; };
    ProductDesc &f = sp.set.forward;
    f.R = (int)M; f.C = (int)N; f.Q = (int)K;
    f.ar = A.sm; f.aq = A.sk; f.bq = B.sk; f.bc = B.sm;
    f.a64 = wide(A); f.b64 = wide(B);
    if (!sp.identity && sp.outer_linear && sp.prog.outer.n_regs >= 0) f.outer = f64 ? 2 : 4;   // ProgWidth
    if (!product_addressable(f)) return;
    for (int q = 0; q < 2; ++q) {
        SepSide &s = sp.side[q];
        const SepSide &o = sp.side[1 - q];
        const int64_t gx = q == 0 ? N : 1, gy = q == 0 ? 1 : N;   // strides of g along the side's own and the other function index
        ProductDesc &d = sp.set.grad[q];
        d.Q = (int)o.X;
        if (!s.k_major) { d.R = (int)s.X; d.C = (int)K; d.ar = gx; d.aq = gy; d.bq = o.sm; d.bc = o.sk; }
        else { d.R = (int)K; d.C = (int)s.X; d.ar = o.sk; d.aq = o.sm; d.bq = gy; d.bc = gx; }
        d.a64 = s.k_major ? wide(o) : f64;
        d.b64 = s.k_major ? f64 : wide(o);
        d.scaled = s.sub && s.operand < 0;
        if (!product_addressable(d)) return;
        if (!s.sub) continue;
        for (size_t p = 0; p < s.operands.size(); ++p) s.aligned.push_back(pairs_are_elements(*s.sub, (int)p));
    }
    for (int p = 0; p < n_ops; ++p) sp.term_is_g[p] = same_program(sp.prog.douter_arg[p], sp.prog.douter);
    // partial sums of the gathers
    size_t gather_part = 0;
    auto gathers = [&](const ArgPlan &ap, int64_t count, double pairs) {
        if (!ap.derived) return;
        const long long n = gather_launch_count(ap.dev, count);
        gather_part = std::max(gather_part, split_workspace_bytes(n, sum_shape(ap.dev, n, pairs).splits));
    };
    for (const SepSide &s : sp.side)
        if (s.sub)
            for (size_t p = 0; p < s.operands.size(); ++p) gathers(s.sub->ap[p], s.sub->arg_count[p], (double)(s.X * K));
    for (int p = 0; p < n_ops; ++p)
        if ((sp.prog.outer_mask >> p) & 1u) gathers(pl.ap_outer[p], pl.arg_count[p], (double)pl.f_count);
    // ... and those of the products, no more of them than `most` bytes
    auto shape = [&](ProductSet &set, size_t most) {
        size_t bytes = gather_part;
        for (ProductDesc *d : {&set.forward, &set.grad[0], &set.grad[1]}) {
            product_shape(*d, most);
            bytes = std::max(bytes, product_partial_bytes(*d));
        }
        product_pair(set.grad[0], set.grad[1]);
        return bytes;
    };
    size_t part = shape(sp.set, SIZE_MAX);
    // workspace.  reuse: the first of a side's terms go where the factor's values were, which the products before them read last
    // (512 x 384 x 200, softplus: 73.0 us apart, 74.0 in the same place)
    auto layout = [&](bool reuse) {
        size_t ws = 0;
        auto reserve = [&](size_t bytes) {
            const size_t at = ws;
            ws += align256(bytes);
            return at;
        };
        for (SepSide &s : sp.side) {
            const size_t matrix = (size_t)(s.X * K) * 8;
            if (s.operand < 0) s.value_offset = reserve(matrix);
            if (!s.sub) continue;
            s.d_offset = reserve(matrix);
            s.h_offset.assign(s.operands.size(), 0);
            bool free_values = reuse && s.operand < 0;
            for (size_t p = 0; p < s.operands.size(); ++p) {
                if (s.operand >= 0 || !s.sub->ap[p].derived || s.aligned[p]) continue;
                s.h_offset[p] = free_values ? s.value_offset : reserve(matrix);
                free_values = false;
            }
        }
        const size_t sums = (size_t)pl.f_count * (f64 ? 8 : 4);
        sp.s_offset = reserve(sums);
        sp.g_offset = reserve(sums);
        sp.h_offset = sp.prog.outer_mask ? reserve((size_t)pl.f_count * 8) : 0;
        sp.part_offset = reserve(part);
        sp.set.ws_bytes = ws;
    };
    double data = (double)pl.f_count;
    for (int p = 0; p < n_ops; ++p) data += (double)pl.arg_count[p];
    // (the partial sums come last)
    auto rest = [&] { return sp.set.ws_bytes - align256(part); };
    // partial sums of the products give way where they alone are what lifts the workspace above a limit
    auto fit = [&](double limit, bool reuse) {
        if ((double)sp.set.ws_bytes <= limit || (double)(rest() + align256(gather_part)) > limit) return;
        part = shape(sp.set, ((size_t)limit - rest()) & ~(size_t)255);
        layout(reuse);
    };
    const double limit = kSeparableWorkspace, elements = 4.0 * data * (f64 ? 8 : 4);
    layout(false);
    fit(limit, false);
    if ((double)sp.set.ws_bytes > limit) {
        layout(true);
        fit(limit + elements, true);
    }
    if ((double)sp.set.ws_bytes > limit + elements) {
        sp = SepPlan{};
        return;
    }
    const size_t array = TAD_STATIC_SCRATCH_BYTES;
    if (sp.set.ws_bytes > array && rest() + align256(gather_part) <= array) {
        sp.lean = sp.set;
        sp.lean.ws_bytes = rest() + align256(shape(sp.lean, (array - rest()) & ~(size_t)255));
        sp.lean_on = true;
    }
    sp.on = true;
    sp.forward_on = !forward_general(pl.dtype == TAD_F64, !program, M, N, K);
}

}  // namespace tad
