// Pattern recognition: which kernel family evaluates the forward pass and each gradient.
// Every plan can run on the plan-driven generic kernels; a specialised family is chosen only
// when body, index matrices, shapes and dtype match its template exactly, and the derived plan
// has the structure the family's kernels assume (which kernel coordinate collapses, which is a window).
#include <algorithm>

#include "plan.hpp"
#include "launch_geom.h"
#include "product_match.hpp"
#include "separable_match.hpp"
#include "mfma_split.h"
#include "split.h"
#include "window_match.hpp"

namespace tad {

// 24-bit safety of the loop-free form: every coefficient and every index extent below 2^23
static bool fits24(int64_t v) { return v > -(1 << 23) && v < (1 << 23); }
static bool extents_fit24(const GatherPlan &g) {
    for (int r = 0; r < g.rank; ++r)
        if (!fits24(g.shape[r])) return false;
    return true;
}

// Largest |y_c| a kernel can meet for gradient elements inside the shape: y = (U beta) / alpha.
static int64_t y_extent(const GatherPlan &g, int c) {
    int64_t v = 0;
    for (int d = 0; d < g.rank; ++d) v += (g.U[c][d] < 0 ? -(int64_t)g.U[c][d] : g.U[c][d]) * (g.shape[d] - 1);
    return v;   // dividing by alpha_c >= 1 only makes it smaller
}

bool flatten_level(const GatherPlan &g, int level, FlatLevel &out) {
    if (level < 0 || level >= g.kappa || g.R > kFlatY || !extents_fit24(g)) return false;
    const int nl = g.lo_end[level] - g.lo_begin[level], nh = g.hi_end[level] - g.hi_begin[level];
    if (nl > kFlatRows || nh > kFlatRows) return false;
    for (int r = 0; r < kFlatRows; ++r) {
        out.ls[r] = 1; out.lk0[r] = kFlatNeutralLo;   // neutral lower row
        out.hs[r] = 1; out.hk0[r] = kFlatNeutralHi;   // neutral upper row
        out.lrs[r] = out.hrs[r] = 1.f;
        for (int c = 0; c < kFlatY; ++c) out.lky[r][c] = out.hky[r][c] = 0;
    }
    for (int r = 0; r < nl + nh; ++r) {
        const GRow &row = g.rows[(r < nl ? g.lo_begin[level] : g.hi_begin[level] - nl) + r];
        for (int m = 0; m < kMaxKernel; ++m)
            if (row.kz[m] != 0) return false;
        for (int c = 0; c < g.R; ++c)
            if (!fits24(row.ky[c])) return false;
        // the loop-free division needs |k0 + ky . y| < 2^23 for every y the kernels can meet
        int64_t worst = row.k0 < 0 ? -(int64_t)row.k0 : row.k0;
        for (int c = 0; c < g.R; ++c) worst += (row.ky[c] < 0 ? -(int64_t)row.ky[c] : row.ky[c]) * y_extent(g, c);
        if (worst >= kFlatNeutralHi || !fits24(row.scale)) return false;
        if (r < nl) {
            out.ls[r] = row.scale; out.lk0[r] = row.k0; out.lrs[r] = 1.f / (float)row.scale;
            for (int c = 0; c < g.R; ++c) out.lky[r][c] = row.ky[c];
        } else {
            out.hs[r - nl] = row.scale; out.hk0[r - nl] = row.k0; out.hrs[r - nl] = 1.f / (float)row.scale;
            for (int c = 0; c < g.R; ++c) out.hky[r - nl][c] = row.ky[c];
        }
    }
    return true;
}

bool flatten_feas(const GatherPlan &g, FlatFeas &out) {
    if (g.nF > kFlatFeas || g.R > kFlatY || !extents_fit24(g)) return false;
    for (int r = 0; r < g.nF; ++r)
        for (int c = 0; c < g.R; ++c)
            if (!fits24(g.feas[r].ky[c])) return false;
    for (int r = 0; r < kFlatFeas; ++r) {
        out.k0[r] = -1;                               // neutral: always satisfied
        for (int c = 0; c < kFlatY; ++c) out.ky[r][c] = 0;
    }
    for (int r = 0; r < g.nF; ++r) {
        out.k0[r] = g.feas[r].k0;
        for (int c = 0; c < g.R; ++c) out.ky[r][c] = g.feas[r].ky[c];
    }
    return true;
}

bool y_is_beta(const GatherPlan &g) {
    if (g.nC != 0 || g.R != g.rank) return false;
    for (int r = 0; r < g.R; ++r) {
        if (g.diag[r] != 1) return false;
        for (int c = 0; c < g.rank; ++c)
            if (g.U[r][c] != (r == c ? 1 : 0)) return false;
    }
    return true;
}

static bool index_is(const tad_arg &a, int n_ext, std::initializer_list<std::initializer_list<int64_t>> m) {
    if ((size_t)a.rank != m.size()) return false;
    int r = 0;
    for (const auto &row : m) {
        if ((int)row.size() != n_ext) return false;
        int d = 0;
        for (int64_t v : row)
            if (a.index[r][d++] != v) return false;
        ++r;
    }
    return true;
}

static bool all_derived(const tad_plan &pl) {
    for (const auto &ap : pl.ap)
        if (!ap.derived) return false;
    return true;
}

// f_ij = exp(-sum_k((a_ik + b_jk)^2 c_ii + d_{i+k}^3)), extended index (i, j, k)
static bool worked_structure(tad_plan &pl) {
    const tad_expr &e = pl.expr;
    if (e.body != TAD_BODY_WORKED || e.n_f != 2 || e.n_sum != 1) return false;
    if (e.sum_lo[0] != 0 || !all_derived(pl)) return false;
    const int64_t I = e.f_shape[0], J = e.f_shape[1], K = e.sum_hi[0] + 1;
    const tad_arg &a = pl.args[0], &b = pl.args[1], &c = pl.args[2], &d = pl.args[3];
    if (!index_is(a, 3, {{1, 0, 0}, {0, 0, 1}}) || a.shape[0] != I || a.shape[1] != K) return false;
    if (!index_is(b, 3, {{0, 1, 0}, {0, 0, 1}}) || b.shape[0] != J || b.shape[1] != K) return false;
    if (!index_is(c, 3, {{1, 0, 0}, {1, 0, 0}})) return false;
    if (!index_is(d, 3, {{1, 0, 1}})) return false;
    // plan of d: one kernel coordinate must be the collapsed j, the other the clipped window moving i
    const ArgPlan &pd = pl.ap[3];
    if (pd.smith.R != 1 || pd.K.cols != 2 || pd.VR(1, 0) != 0) return false;
    int lvl_j = -1, lvl_w = -1;
    for (int m = 0; m < 2; ++m) {
        if (pd.K(0, m) == 0 && pd.K(1, m) == 1 && pd.K(2, m) == 0) lvl_j = m;
        else if (pd.K(1, m) == 0 && pd.K(0, m) != 0) lvl_w = m;
    }
    if (lvl_j < 0 || lvl_w < 0) return false;
    if (!y_is_beta(pd.dev) || !flatten_feas(pd.dev, pl.fast.feas) || !flatten_level(pd.dev, lvl_w, pl.fast.flat[0]))
        return false;
    pl.fast.I = I; pl.fast.J = J; pl.fast.K = K;
    pl.fast.c_ld = c.shape[1];
    pl.fast.dd_level = lvl_w;
    pl.fast.dd_iy = (int)pd.VR(0, 0);
    pl.fast.dd_iz = (int)pd.K(0, lvl_w);
    return true;
}

static bool match_worked(tad_plan &pl) {
    if (pl.dtype != TAD_F32 || !worked_structure(pl)) return false;
    const int64_t I = pl.fast.I, J = pl.fast.J, K = pl.fast.K;
    if (J % 4 != 0) return false;   // rows of f must start 16-byte aligned for the vector loads and stores
    if (K <= kWorkedMaxK) {
        pl.fwd_family = TAD_FAMILY_WORKED;
        for (auto &ap : pl.ap) ap.family = TAD_FAMILY_WORKED;
        pl.ws_bytes = worked_workspace_bytes(I, J, K);
        return true;
    }
    if (K % 32 == 0) {
        // long summed index: the contraction over k (and the collapsed j / i contractions of the gradients)
        // are dense matrix products and run on the matrix cores
        pl.fwd_family = TAD_FAMILY_WORKED_MFMA;
        for (auto &ap : pl.ap) ap.family = TAD_FAMILY_WORKED_MFMA;
        pl.ws_bytes = mfma_workspace_bytes(I, J, K);
        return true;
    }
    return false;
}

static bool unary_body(int body) {
    return body == TAD_BODY_SQ || body == TAD_BODY_CUBE || body == TAD_BODY_SIN || body == TAD_BODY_EXP;
}

// the three one-argument patterns of the introduction: f_ij = phi(x_i), f_i = phi(x_ii), f_ij = phi(x_{i+j})
static int pattern_of(tad_plan &pl) {
    const tad_expr &e = pl.expr;
    if (!unary_body(e.body) || e.n_sum != 0 || !all_derived(pl)) return TAD_FAMILY_GENERIC;
    const tad_arg &x = pl.args[0];
    const ArgPlan &px = pl.ap[0];
    int fam = TAD_FAMILY_GENERIC;
    if (e.n_f == 2 && index_is(x, 2, {{1, 0}})) {
        // kernel coordinate = j over its whole range, i = y_0
        if (px.smith.R != 1 || px.K.cols != 1) return fam;
        if (px.VR(0, 0) != 1 || px.VR(1, 0) != 0 || px.K(0, 0) != 0 || px.K(1, 0) * px.K(1, 0) != 1) return TAD_FAMILY_GENERIC;
        if (!y_is_beta(px.dev) || !flatten_feas(px.dev, pl.fast.feas)) return TAD_FAMILY_GENERIC;
        fam = TAD_FAMILY_ROW_REDUCE;
    } else if (e.n_f == 1 && index_is(x, 1, {{1}, {1}})) {
        if (px.smith.R != 1 || px.K.cols != 0 || px.VR(0, 0) != 1) return TAD_FAMILY_GENERIC;
        // transformed index y = first gradient index; one cokernel row +-(1, -1)
        const GatherPlan &g = px.dev;
        if (g.nC != 1 || g.C[0][0] + g.C[0][1] != 0 || g.C[0][0] * g.C[0][0] != 1) return TAD_FAMILY_GENERIC;
        if (g.diag[0] != 1 || g.U[0][0] != 1 || g.U[0][1] != 0 || !flatten_feas(g, pl.fast.feas)) return TAD_FAMILY_GENERIC;
        pl.fast.c_ld = x.shape[1];
        fam = TAD_FAMILY_DIAGONAL;
    } else if (e.n_f == 2 && index_is(x, 2, {{1, 1}})) {
        if (px.smith.R != 1 || px.K.cols != 1) return fam;
        if (px.K(0, 0) * px.K(0, 0) != 1 || px.K(1, 0) * px.K(1, 0) != 1) return TAD_FAMILY_GENERIC;
        if (!y_is_beta(px.dev) || !flatten_feas(px.dev, pl.fast.feas) || !flatten_level(px.dev, 0, pl.fast.flat[0]))
            return TAD_FAMILY_GENERIC;
        pl.fast.dd_iy = (int)px.VR(0, 0); pl.fast.dd_iz = (int)px.K(0, 0);
        pl.fast.jy = (int)px.VR(1, 0); pl.fast.jz = (int)px.K(1, 0);
        fam = TAD_FAMILY_ANTIDIAGONAL;
    } else {
        return TAD_FAMILY_GENERIC;
    }
    pl.fast.I = e.f_shape[0];
    pl.fast.J = e.n_f == 2 ? e.f_shape[1] : 1;
    return fam;
}

static bool match_patterns(tad_plan &pl) {
    const int fam = pl.dtype == TAD_F32 ? pattern_of(pl) : TAD_FAMILY_GENERIC;
    if (fam == TAD_FAMILY_GENERIC) return false;
    // rows must start 16-byte aligned for the vector loads and stores
    if ((fam == TAD_FAMILY_DIAGONAL ? pl.args[0].shape[1] : pl.expr.f_shape[1]) % 4 != 0) return false;
    if (fam == TAD_FAMILY_ANTIDIAGONAL) pl.ws_bytes = antidiag_workspace_bytes(pl.expr.f_shape[0], pl.expr.f_shape[1]);
    pl.fwd_family = fam;
    pl.ap[0].family = fam;
    return true;
}

// f_nij = tanh(sum_{u,v} x_{n, s i + u, s j + v} w_uv), extended index (n, i, j, u, v)
static bool match_strided(tad_plan &pl) {
    const tad_expr &e = pl.expr;
    if (e.body != TAD_BODY_TANH_DOT || pl.dtype != TAD_F32 || e.n_f != 3 || e.n_sum != 2) return false;
    if (e.sum_lo[0] != 0 || e.sum_lo[1] != 0 || !all_derived(pl)) return false;
    const tad_arg &x = pl.args[0], &w = pl.args[1];
    if (x.rank != 3 || w.rank != 2) return false;
    const int64_t s = x.index[1][1];
    if (s < 1) return false;
    if (!index_is(x, 5, {{1, 0, 0, 0, 0}, {0, s, 0, 1, 0}, {0, 0, s, 0, 1}})) return false;
    if (!index_is(w, 5, {{0, 0, 0, 1, 0}, {0, 0, 0, 0, 1}})) return false;
    const int64_t U = e.sum_hi[0] + 1, V = e.sum_hi[1] + 1;
    if (w.shape[0] != U || w.shape[1] != V || U * V > 49) return false;
    // x: two kernel coordinates with plan-driven ranges; w: the three function indices collapse completely
    const ArgPlan &px = pl.ap[0], &pw = pl.ap[1];
    if (px.K.cols != 2 || pw.K.cols != 3 || px.smith.R != 3) return false;
    // x: y = beta, and both ranges in the loop-free form (neither depends on the other kernel coordinate)
    if (!y_is_beta(px.dev) || !flatten_feas(px.dev, pl.fast.feas)) return false;
    if (!flatten_level(px.dev, 0, pl.fast.flat[0]) || !flatten_level(px.dev, 1, pl.fast.flat[1])) return false;
    pl.fast.N = e.f_shape[0]; pl.fast.I = e.f_shape[1]; pl.fast.J = e.f_shape[2];
    pl.fast.U = U; pl.fast.V = V; pl.fast.stride = s;
    pl.fast.P = x.shape[1]; pl.fast.Q = x.shape[2];
    pl.fwd_family = TAD_FAMILY_STRIDED;
    pl.ap[0].family = pl.ap[1].family = TAD_FAMILY_STRIDED;
    pl.ws_bytes = strided_workspace_bytes(e.f_shape[0], e.f_shape[1], e.f_shape[2], U, V, s, x.shape[2]);
    return true;
}

// f_ij = sum_k P(i, k) Q(k, j): both operands are matrices indexed by one function index and the summation index,
// their axes in either order, shapes exactly the index ranges.  Extended index (i, j, k).
// the body is the product of its two operands, summed: built in, or a program that says the same
static bool is_product_body(const tad_plan &pl) {
    if (pl.expr.body == TAD_BODY_MUL) return true;
    if (pl.expr.body != TAD_BODY_PROGRAM || pl.prog.n_operands != 2) return false;
    const DevProg &in = pl.prog.inner, &out = pl.prog.outer;
    return out.n == 1 && out.op[0] == P_SUM && in.n == 3 && in.result == 2 && in.op[0] == P_ARG &&
           in.op[1] == P_ARG && in.a[0] + in.a[1] == 1 && in.op[2] == P_MUL && in.a[2] + in.b[2] == 1;
}

static bool match_contraction(tad_plan &pl) {
    const tad_expr &e = pl.expr;
    if (!is_product_body(pl) || pl.dtype != TAD_F32 || e.n_f != 2 || e.n_sum != 1 || e.sum_lo[0] != 0) return false;
    if (!all_derived(pl)) return false;
    const int64_t ext[3] = {e.f_shape[0], e.f_shape[1], e.sum_hi[0] + 1};
    for (int d = 0; d < 3; ++d)
        if (ext[d] % 4 != 0 || ext[d] > (1 << 20)) return false;   // 16-byte rows; int32 addressing inside the kernel
    // axis_dim[p][r]: which extended index axis r of operand p follows (rows of the index matrix are unit vectors)
    int axis_dim[2][2];
    for (int p = 0; p < 2; ++p) {
        const tad_arg &a = pl.args[p];
        if (a.rank != 2) return false;
        for (int r = 0; r < 2; ++r) {
            int dim = -1;
            for (int d = 0; d < 3; ++d) {
                if (a.index[r][d] == 1 && dim < 0) dim = d;
                else if (a.index[r][d] != 0) return false;
            }
            if (dim < 0 || a.shape[r] != ext[dim]) return false;
            axis_dim[p][r] = dim;
        }
        if (axis_dim[p][0] == axis_dim[p][1]) return false;
    }
    auto has = [&](int p, int dim) { return axis_dim[p][0] == dim || axis_dim[p][1] == dim; };
    int P = -1, Q = -1;
    if (has(0, 0) && has(0, 2) && has(1, 1) && has(1, 2)) { P = 0; Q = 1; }
    else if (has(1, 0) && has(1, 2) && has(0, 1) && has(0, 2)) { P = 1; Q = 0; }
    else return false;
    // the derived plans must say what the kernels assume: y = beta, one kernel coordinate, and its range is the
    // whole collapsed dimension whatever beta is
    for (int p = 0; p < 2; ++p) {
        const ArgPlan &ap = pl.ap[p];
        const int gone = p == P ? 1 : 0;   // function index missing from the operand
        if (ap.smith.R != 2 || ap.K.cols != 1 || !y_is_beta(ap.dev)) return false;
        // no feasibility row may fail anywhere inside the operand's shape (no element is masked out)
        for (int r = 0; r < ap.dev.nF; ++r) {
            int64_t worst = ap.dev.feas[r].k0;
            for (int c = 0; c < 2; ++c) worst += std::max<int64_t>(0, (int64_t)ap.dev.feas[r].ky[c] * (ap.dev.shape[c] - 1));
            if (worst > 0) return false;
        }
        for (int d = 0; d < 3; ++d)
            if (ap.K(d, 0) * ap.K(d, 0) != (d == gone ? 1 : 0)) return false;
        FlatLevel fl;
        if (!flatten_level(ap.dev, 0, fl)) return false;
        for (int r = 0; r < kFlatRows; ++r)
            for (int c = 0; c < kFlatY; ++c)
                if (fl.lky[r][c] != 0 || fl.hky[r][c] != 0) return false;
        const int32_t y0[3] = {0, 0, 0};
        int32_t lo, hi;
        flat_bounds(fl, y0, lo, hi);
        if ((int64_t)hi - lo + 1 != ext[gone]) return false;
    }
    const int I = (int)ext[0], J = (int)ext[1], Kc = (int)ext[2];
    const bool p_ik = axis_dim[P][0] == 0;   // P stored [i][k]
    const bool q_kj = axis_dim[Q][0] == 2;   // Q stored [k][j]
    const int ldp = (int)pl.args[P].shape[1], ldq = (int)pl.args[Q].shape[1];
    GemmDesc *g = pl.fast.gemm;
    // f[i][j] = sum_k P(i,k) Q(k,j)
    g[0] = GemmDesc{I, J, Kc, P, Q, -1, ldp, ldq, !p_ik, !q_kj};
    // gradient of P in its own memory order
    if (p_ik) g[1] = GemmDesc{I, Kc, J, -1, Q, P, J, ldq, 0, q_kj};       // dP[i][k] = sum_j df[i][j] Q(k,j)
    else      g[1] = GemmDesc{Kc, I, J, Q, -1, P, ldq, J, !q_kj, 1};      // dP[k][i] = sum_j Q(k,j) df[i][j]
    // gradient of Q in its own memory order
    if (q_kj) g[2] = GemmDesc{Kc, J, I, P, -1, Q, ldp, J, p_ik, 0};       // dQ[k][j] = sum_i P(i,k) df[i][j]
    else      g[2] = GemmDesc{J, Kc, I, -1, P, Q, J, ldp, 1, !p_ik};      // dQ[j][k] = sum_i df[i][j] P(i,k)
    // A product with few output tiles and a long contraction index leaves most of the chip idle: cut the index
    // into pieces for separate workgroups (partial products in the workspace, added in a fixed order afterwards).
    // Tiles are counted as 128 x 128 whatever the kernel's are (k_contract_low has four times as many): the number of pieces decides how a sum is
    // rounded, and these are the sums the family has always had.
    size_t ws = 0;
    for (int q = 0; q < 3; ++q) {
        const long long tiles = (long long)((g[q].M + 127) / 128) * ((g[q].N + 127) / 128);
        int sp = 1;
        if (tiles < 256 && g[q].Kc >= 512) {
            sp = (int)std::min<long long>((512 + tiles - 1) / tiles, g[q].Kc / 256);
            sp = std::max(1, std::min(sp, 256));
        }
        g[q].splits = sp;
        if (sp > 1) ws = std::max(ws, align256((size_t)sp * g[q].M * g[q].N * sizeof(float)));
    }
    pl.ws_bytes = ws;
    pl.fwd_family = TAD_FAMILY_CONTRACTION;
    pl.ap[0].family = pl.ap[1].family = TAD_FAMILY_CONTRACTION;
    return true;
}

static void select_specialised(tad_plan &plan) {
    plan.fwd_family = TAD_FAMILY_GENERIC;
    for (auto &ap : plan.ap) ap.family = TAD_FAMILY_GENERIC;
    plan.ws_bytes = 0;
    if (plan.expr.body == TAD_BODY_PROGRAM) {
        // interpreter kernels; the backward pass keeps g = df * outer'(sum) for every function element
        plan.fwd_family = TAD_FAMILY_PROGRAM;
        for (auto &ap : plan.ap) ap.family = TAD_FAMILY_PROGRAM;
        // ... and, if the outer function reads operands, the sums themselves for the terms df * d outer / d x
        plan.ws_bytes = align256((size_t)plan.f_count * (plan.dtype == TAD_F64 ? 8 : 4)) * (plan.prog.outer_mask ? 2 : 1);
        // a plain product of two matrices (the form the derived expressions of a matrix product have) still
        // belongs on the matrix cores
        if (!(plan.flags & TAD_PLAN_GENERIC_ONLY) && !plan.has_alias && plan.expr.n_constraints == 0 &&
            match_contraction(plan)) {
            // the matcher has set the family and the workspace of the products
        }
        return;
    }
    if ((plan.flags & TAD_PLAN_GENERIC_ONLY) || plan.has_alias || plan.expr.n_constraints > 0) return;
    if (match_worked(plan)) return;
    if (match_patterns(plan)) return;
    if (match_strided(plan)) return;
    if (match_contraction(plan)) return;
}

static void reserve_partial_sums(tad_plan &plan);
static void select_split(tad_plan &plan);

void select_families(tad_plan &plan) {
    select_specialised(plan);
    reserve_partial_sums(plan);
    match_product(plan);
    plan.prod.ws_offset = align256(plan.ws_bytes);
    plan.ws_full = plan.prod.on && plan.prod.set.ws_bytes ? plan.prod.ws_offset + plan.prod.set.ws_bytes : plan.ws_bytes;
    if (plan.prod.on && plan.prod.lean_on) plan.ws_lean = plan.prod.ws_offset + plan.prod.lean.ws_bytes;
    select_split(plan);
    match_separable(plan);
    if (plan.sep.on) {   // one or the other
        plan.ws_full = std::max(plan.ws_bytes, plan.sep.set.ws_bytes);
        if (plan.sep.lean_on) plan.ws_lean = std::max(plan.ws_bytes, plan.sep.lean.ws_bytes);
    }
}

// The worked expression on the kernels with 64-bit sums; the reported family stays what it is without them.  They take the
// forms the fused 32-bit kernels have no code for, and those of fewer than 2^23 elements: the tiles of the 32-bit kernels
// (256 x 512) are made for a full chip.  Forward and gradients, 32-bit sums against 64-bit sums with one more column: 64 x 64 x 5
// 45 / 20 us, 1024 x 1024 x 5 44 / 24, 2048 x 2048 x 1 40 / 25, x 8 61 / 42, 4096 x 2048 x 5 58 / 57, 4096 x 4096 x 5 66 / 95 us.
constexpr int64_t kWideElements = (int64_t)1 << 23;

// Sums of a row that the 64-bit kernels leave to their finishing pass, (K + 2) for each of its tiles, up to which they are the
// faster ones: the pass adds them up in turn.  32-bit sums / 64-bit sums, I x J x K: 64 x 65536 x 1 (768) 42 / 36 us, 64 x 32768 x 5
// (896) 52 / 42, 16 x 32768 x 5 (896) 30 / 30; 256 x 28672 x 7 (1008) 66 / 71, 128 x 65532 x 2 (1024) 60 / 67, 256 x 16384 x 8 (1280)
// 65 / 74, 16 x 262144 x 5 (7168) 108 / 197.  (Against the general kernels the 64-bit ones are ahead at any length.)
constexpr int64_t kWideRowSums = 900;

static void select_worked_wide(tad_plan &plan) {
    const bool fused = plan.fwd_family == TAD_FAMILY_WORKED;
    if ((plan.fwd_family != TAD_FAMILY_GENERIC && !fused) || (fused && plan.f_count >= kWideElements)) return;
    if (!worked_structure(plan) || plan.fast.K > kWideMaxK) return;
    if (fused && (plan.fast.K + 2) * worked_wide_geom(plan.fast.I, plan.fast.J, plan.fast.K).n_jt > kWideRowSums) return;
    plan.worked_wide = true;
    plan.ws_full = std::max(plan.ws_bytes, worked_wide_geom(plan.fast.I, plan.fast.J, plan.fast.K).ws_bytes);
}

// Row reduce and antidiagonal patterns in a form their 32-bit kernels do not take; the family stays the general one, and the
// gradient too where that has the better layout for it.  General / streaming kernels, gradient of I x J:
//   row sums, one wavefront or workgroup per row.  Rows shorter than a wavefront, a thread each there: 65537 x 17 12.0 / 11.8 us,
//   100001 x 17 12 / 16, 1000001 x 3 26 / 171 (60001 x 65 12 / 12, 1000001 x 65 258 / 212).  Few rows so long that several workgroups share
//   one there: 65 x 65537 14 / 8, 65 x 98305 15 / 20, 16 x 131073 15 / 17, 3 x 1000001 14 / 203 (600 x 131073 58 / 54); 64 bits
//   1 x 65537 14 / 19, 2 x 100001 15 / 19.
//   antidiagonals of short rows in 32 bits, hardly longer than the chunks' sums: 200001 x 17 20 / 21, 1000001 x 17 73 / 101, x 33 351 / 119.
static bool wide_gradient(const tad_plan &plan, int fam, int64_t I, int64_t J, int64_t n_x) {
    if (fam == TAD_FAMILY_ROW_REDUCE) {
        if (J < 64) return n_x <= 65536;
        return J <= (n_x <= 16 && plan.dtype == TAD_F32 ? 131072 : 65536) || n_x >= 512;
    }
    return plan.dtype == TAD_F64 || J >= 20 || I <= 262144;
}

static void select_pattern_wide(tad_plan &plan) {
    if (plan.fwd_family != TAD_FAMILY_GENERIC) return;
    const int fam = pattern_of(plan);
    if (fam != TAD_FAMILY_ROW_REDUCE && fam != TAD_FAMILY_ANTIDIAGONAL) return;
    const bool gradient = wide_gradient(plan, fam, plan.fast.I, plan.fast.J, plan.arg_count[0]);
    if (fam == TAD_FAMILY_ANTIDIAGONAL) {
        // two launches backward: below, the one of the general kernels is as fast (40 x 41: 14.5 us against 16; 100 x 101: 19 against 15)
        if (plan.f_count < 4096) return;
        // the kernels address f as i * J + j with j = m - i
        if (plan.fast.dd_iy + plan.fast.jy != 1 || plan.fast.dd_iz + plan.fast.jz != 0) return;
        // short rows: the chunks' sums would be as large as f
        const size_t ws = antidiag_wide_workspace_bytes(plan.fast.I, plan.fast.J);
        if (plan.fast.J < 16 && ws > ((size_t)1 << 20)) return;
        if (gradient) plan.ws_full = std::max(plan.ws_bytes, ws);
    }
    plan.pattern_wide = fam;
    plan.pattern_wide_sums = gradient;
}

void select_wide(tad_plan &plan) {
    if ((plan.flags & TAD_PLAN_GENERIC_ONLY) || plan.has_alias) return;
    // its terms are listed, or the plan is to have its ranges walked
    if (!plan.term_list.empty() || ((plan.flags & TAD_PLAN_NO_TERM_LISTS) && small_expression(plan))) return;
    match_window(plan);
    if (plan.expr.n_constraints > 0) return;
    select_worked_wide(plan);
    select_pattern_wide(plan);
}

// Time of a choice: rounds of the `slots` workgroups that run at once, a stage of 32 terms and what a workgroup takes besides its stages, and 5 TB/s for
// the partial results.  No more pieces than the workspace holds: kMfmaSplit of either sum, and where one has fewer the other may have more.
// least_j, least_i: pieces that the sum over j, over i, has at least.
static MfmaPieces pieces_of_long_sums(int64_t I, int64_t J, int64_t K, bool cols, int tile, int slots, double stage, double besides, int64_t least_j, int64_t least_i) {
    MfmaPieces best{};
    best.time = -1;
    const int64_t columns = (K + 255) / 256, ti = (I + tile - 1) / tile * columns, tj = cols ? (J + tile - 1) / tile * columns : 0;
    const int64_t stages_j = (J + 31) / 32, stages_i = (I + 31) / 32, most_j = (stages_j + least_j - 1) / least_j, most_i = (stages_i + least_i - 1) / least_i;
    for (int64_t n = 1; n <= std::max(stages_i, stages_j); n += 1 + n / 16) {
        const int64_t in_j = std::min(n, most_j), in_i = std::min(n, most_i), nj = (stages_j + in_j - 1) / in_j, ni = cols ? (stages_i + in_i - 1) / in_i : 0;
        if (nj > kMfmaMostPieces || ni > kMfmaMostPieces || nj * I + ni * J > kMfmaSplit * (I + J) || 2 * nj * I + ni * J > kMfmaSplit * (2 * I + J)) continue;
        const int64_t rounds = (ti * nj + tj * ni + slots - 1) / slots;
        const double t = (double)rounds * ((double)std::max(in_j, cols ? in_i : 0) * stage + besides) + (double)(nj * I + ni * J) * (double)K * 8 / 5e6;
        if (best.time >= 0 && t >= best.time) continue;
        best = {(int)nj, (int)ni, (int)(32 * in_j), (int)(32 * in_i), false, t};
    }
    return best;
}

static void select_pieces(tad_plan &plan) {
    const int64_t I = plan.fast.I, J = plan.fast.J, K = plan.fast.K;
    for (int cols = 0; cols < 2; ++cols) {
        auto short_pieces = [&](const MfmaPieces &n) { return n.chunk_j <= mfma_chain((int)J) && (!cols || n.chunk_i <= mfma_chain((int)I)); };
        MfmaPieces &plain = plan.mfma_pieces[0][cols], &n = plan.mfma_pieces[1][cols];
        plain = pieces_of_long_sums(I, J, K, cols, 64, 512, 5.0, 5.0, 1, 1);
        plain.totals = !short_pieces(plain);
        if (!long_pays(I, J, K)) continue;
        if (K <= 128) {
            n = pieces_of_long_sums(I, J, K, cols, 128, K <= 64 ? 512 : 256, K <= 64 ? 2.5 : 2.2, 6.0, 1, 1);
            n.totals = !short_pieces(n);
            continue;
        }
        n = pieces_of_long_sums(I, J, K, cols, 128, 256, 3.6, 6.0, long_least_pieces(J), long_least_pieces(I));
        const MfmaPieces any = pieces_of_long_sums(I, J, K, cols, 128, 256, 3.9, 6.0, 1, 1);
        if (any.time >= n.time) continue;
        n = any;
        n.totals = !short_pieces(n);
    }
}

static void select_split(tad_plan &plan) {
    if (plan.fwd_family == TAD_FAMILY_WORKED_MFMA) {
        const int64_t I = plan.fast.I, J = plan.fast.J, K = plan.fast.K;
        select_pieces(plan);
        plan.mfma_split = long_pays(I, J, K) || long_forward_pays(I, J, K);
        if (plan.mfma_split) plan.ws_full = align256(plan.ws_bytes) + long_workspace_bytes(I, J, K);
    }
    if (plan.fwd_family != TAD_FAMILY_CONTRACTION) return;
    for (const GemmDesc &g : plan.fast.gemm)
        if (split_pays(g.M, g.N, g.Kc)) {
            plan.split = true;
            plan.ws_full = std::max(plan.ws_full, split_geom(g.M, g.N, g.Kc).bytes);
        }
}

static void reserve_partial_sums(tad_plan &plan) {
    // the fallback kernels share the elements of a gradient with few elements and long sums among several blocks:
    // room for their partial sums behind whatever the family keeps in the workspace
    bool fallback = true;
    for (const auto &ap : plan.ap) fallback = fallback && (ap.family == TAD_FAMILY_GENERIC || ap.family == TAD_FAMILY_PROGRAM);
    plan.split_ws_offset = plan.ws_bytes;
    if (!fallback) return;
    // ... and those of a forward sum with few function indices
    size_t most = cooperative_splits(plan.f_count, plan.terms_total) > 1
                      ? align256((size_t)plan.f_count * (size_t)cooperative_splits(plan.f_count, plan.terms_total) * 8)
                      : 0;
    for (size_t q = 0; q < plan.args.size(); ++q) {
        if (!plan.ap[q].derived) continue;   // no gradient planned for this operand
        const long long n = gather_launch_count(plan.ap[q].dev, plan.arg_count[(size_t)plan.root[q]]);
        most = std::max(most, split_workspace_bytes(n, gather_shape(plan.ap[q].dev, n, plan.terms_total).splits));
        if (plan.expr.body == TAD_BODY_PROGRAM && ((plan.prog.outer_mask >> q) & 1u)) {
            const long long no = gather_launch_count(plan.ap_outer[q].dev, plan.arg_count[(size_t)plan.root[q]]);
            most = std::max(most, split_workspace_bytes(no, cooperative_splits(no, (double)plan.f_count)));
        }
    }
    plan.ws_bytes += most;
}

}  // namespace tad
