// Sums of products of two functions as dense products (separable.hpp): the element-wise passes around the products.
//
//   forward    values of the factors that are functions of operands (64 bits), product, outer function
//   backward   the same values and sums again, g = df * d outer / d s; then per factor its derivative (a product) and per
//              operand of the factor dx_beta = sum over the pairs of indices that read x_beta of derivative * partial derivative:
//              in one pass where every pair reads an element of its own, else through the terms in the workspace and a
//              sum through the operand's plan
// What a factor or a partial derivative costs is paid once per pair of indices instead of once per term, which leaves
// the products as the bound (64-bit matrix instructions) and, below some 10^8 terms, the launches: 512 x 1024 x 768 with one
// interpreted term per thread 9895 us, 1.2 10^9 interpreted terms.
#include <hip/hip_runtime.h>

#include "gather_loop.h"
#include "launch.h"
#include "plan_dev.h"
#include "prog_eval.h"
#include "profile.h"
#include "separable.hpp"

namespace tad {

// Offsets of the operands at element `lin` of an expression without summation indices.
__device__ __forceinline__ void element_offsets(const ForwardPlan &P, int n_ops, int lin, int64_t *base) {
    // unrolled to the largest rank and cut short by tests of the uniform rank, so that every field of the plan comes from a
    // fixed place in the kernel arguments
    int32_t ext[kMaxExt];
    int t = lin;
#pragma unroll
    for (int d = kMaxExt - 1; d >= 1; --d) {
        ext[d] = 0;
        if (d < P.n_f) {
            const int s = P.f_shape[d], q = t / s;
            ext[d] = t - q * s;
            t = q;
        }
    }
    ext[0] = t;
#pragma unroll
    for (int p = 0; p < kMaxArgs; ++p) {
        if (p >= n_ops) continue;
        int64_t o = P.base0[p];
#pragma unroll
        for (int d = 0; d < kMaxExt; ++d)
            if (d < P.n_f) o += P.off[p][d] * (int64_t)ext[d];
        base[p] = o;
    }
}

// Values of the operands of `mask` at element `lin`, widened; the others are 0.
template <typename T, typename TV>
__device__ __forceinline__ void element_values(const ForwardPlan &P, int n_ops, uint32_t mask, const ArgPtrs &A, int lin, TV *v) {
    int64_t base[kMaxArgs];
    element_offsets(P, n_ops, lin, base);
#pragma unroll
    for (int p = 0; p < kMaxArgs; ++p) v[p] = p < n_ops && ((mask >> p) & 1u) ? (TV)static_cast<const T *>(A.p[p])[base[p]] : TV(0);
}

// A factor at every pair of indices, evaluated in 64 bits: of 32-bit operands nothing can overflow on the way there.
template <typename T, int FORM>
__global__ __launch_bounds__(256) void k_sep_factor(const ForwardPlan P, const DevProg inner, int n_ops, const ArgPtrs A,
                                                    double *__restrict__ out, int n) {
    const int lin = blockIdx.x * 256 + threadIdx.x;
    if (lin >= n) return;
    double v[kMaxArgs];
    element_values<T>(P, n_ops, ~0u, A, lin, v);
    out[lin] = prog_eval<double, FORM>(inner, v, 0.0);
}

// df == nullptr: out = prog(s, operands), else out = df * prog(s, operands); `out` may be `s`.  TO: T, or double for terms
// that are summed afterwards.
template <typename T, typename TO, int FORM>
__global__ __launch_bounds__(256) void k_sep_outer(const ForwardPlan P, const DevProg prog, int n_ops, uint32_t mask, const ArgPtrs A,
                                                   const T *s, const T *__restrict__ df, TO *out, int n) {
    const int lin = blockIdx.x * 256 + threadIdx.x;
    if (lin >= n) return;
    T v[kMaxArgs] = {};
    if (mask) element_values<T>(P, n_ops, mask, A, lin, v);
    const T o = prog_eval<T, FORM>(prog, v, s[lin]);
    out[lin] = df ? (TO)df[lin] * (TO)o : (TO)o;
}

// d * (partial derivative) at every pair of indices: into dx where pair number and element number are the same, else into h.
template <typename T, int FORM>
__global__ __launch_bounds__(256) void k_sep_terms(const ForwardPlan P, const DevProg dinner, int n_ops, const ArgPtrs A,
                                                   const double *__restrict__ d, T *__restrict__ dx, double *__restrict__ h, int n) {
    const int lin = blockIdx.x * 256 + threadIdx.x;
    if (lin >= n) return;
    double v[kMaxArgs];
    element_values<T>(P, n_ops, ~0u, A, lin, v);
    const double t = d[lin] * prog_eval<double, FORM>(dinner, v, 0.0);
    if (dx) dx[lin] = (T)t;
    else h[lin] = t;
}

// Sum of h over the pairs that read element `idx` (part of it, shared by parts threads of groups workgroups).
template <typename TI>
__device__ __forceinline__ bool sum_element(const GatherPlan &P, const TI *__restrict__ h, int idx, int *lin, int part, int parts,
                                            double *sum, int group, int groups) {
    int32_t y[kMaxRank] = {0, 0, 0, 0};
    *sum = 0.0;
    if (!gather_element_index(P, idx, lin, y)) return false;
    double acc = 0.0;
    gather_loops(P, y, part, parts, [&](const int32_t *z, int32_t n, int32_t step) {
        const TI *p = h + gather_offset(P, kSlotF, y, z);
        const int64_t st = P.offZ[kSlotF][0] * step;
        constexpr int U = 8;   // one wait for memory per batch
        int32_t it = 0;
        for (; it + U <= n; it += U) {
            TI v[U];
#pragma unroll
            for (int u = 0; u < U; ++u) { v[u] = *p; p += st; }
#pragma unroll
            for (int u = 0; u < U; ++u) acc += (double)v[u];
        }
        for (; it < n; ++it) { acc += (double)*p; p += st; }
    }, group, groups);
    *sum = acc;
    return true;
}

template <typename TI, typename T, int LAYOUT>
__global__ __launch_bounds__(LAYOUT == kSumColumns ? 1024 : 256) void k_sep_sum(const GatherPlan P, const TI *__restrict__ h,
                                                                               T *__restrict__ dx, int n, int accumulate,
                                                                               double *__restrict__ partial, int32_t *__restrict__ flag) {
    const int tid = threadIdx.x;
    int lin = -1;
    bool live = false;
    double total = 0.0;
    if constexpr (LAYOUT == kSumThread) {
        const int idx = blockIdx.x * 256 + tid;
        if (idx >= n) return;
        live = sum_element(P, h, idx, &lin, 0, 1, &total, 0, 1);
        store_element(dx, lin, live, total, accumulate);
    } else if constexpr (LAYOUT == kSumWave) {
        const int idx = blockIdx.x * 4 + (tid >> 6);
        if (idx >= n) return;   // the whole wavefront leaves together
        double mine;
        live = sum_element(P, h, idx, &lin, tid & 63, 64, &mine, 0, 1);
        total = wave_sum_all(mine);
        if ((tid & 63) == 0) store_element(dx, lin, live, total, accumulate);
    } else if constexpr (LAYOUT == kSumBlock) {
        __shared__ double red[4];
        const int idx = blockIdx.x;
        double mine;
        live = sum_element(P, h, idx, &lin, tid, 256, &mine, (int)blockIdx.y, (int)gridDim.y);
        total = block_sum_256(mine, red);
        if (tid != 0) return;
        if (partial) store_partial(partial, flag, idx, lin, live, total);
        else store_element(dx, lin, live, total, accumulate);
    } else {
        __shared__ double red[32][33];
        const int col = tid & 31, part = tid >> 5, idx = blockIdx.x * 32 + col;
        double mine = 0.0;
        if (idx < n) live = sum_element(P, h, idx, &lin, part, 32, &mine, (int)blockIdx.y, (int)gridDim.y);
        red[part][col] = mine;
        __syncthreads();
        if (part != 0 || idx >= n) return;
#pragma unroll
        for (int p = 0; p < 32; ++p) total += red[p][col];
        if (partial) store_partial(partial, flag, idx, lin, live, total);
        else store_element(dx, lin, live, total, accumulate);
    }
}

static int launched() { return hipGetLastError() == hipSuccess ? TAD_OK : TAD_EDEVICE; }

static ArgPtrs operand_pointers(const SepSide &side, const void *const *args) {
    ArgPtrs A{};
    for (size_t p = 0; p < side.operands.size(); ++p) A.p[p] = args[side.operands[p]];
    return A;
}

// the factors that are functions of operands
template <typename T>
static int evaluate_factors(const SepPlan &sp, const void *const *args, char *ws, hipStream_t s) {
    for (const SepSide &side : sp.side) {
        if (side.operand >= 0) continue;
        const tad_plan &sub = *side.sub;
        const int n = (int)sub.f_count;
        const ArgPtrs A = operand_pointers(side, args);
        double *const out = reinterpret_cast<double *>(ws + side.value_offset);
        const dim3 grid((n + 255) / 256), block(256);
        if (has_register_form(sub.prog.inner))
            TAD_LAUNCH("k_sep_factor", (k_sep_factor<T, 1>), grid, block, 0, s, sub.fwd, sub.prog.inner, (int)sub.args.size(), A, out, n);
        else
            TAD_LAUNCH("k_sep_factor", (k_sep_factor<T, 0>), grid, block, 0, s, sub.fwd, sub.prog.inner, (int)sub.args.size(), A, out, n);
        if (launched()) return TAD_EDEVICE;
    }
    return TAD_OK;
}

static const void *factor(const SepSide &side, const void *const *args, const char *ws) {
    return side.operand >= 0 ? args[side.operand] : ws + side.value_offset;
}

template <typename T>
static int sums(const tad_plan &pl, const void *const *args, void *out, char *ws, hipStream_t s) {
    const SepPlan &sp = pl.sep;
    const int rc = evaluate_factors<T>(sp, args, ws, s);
    if (rc) return rc;
    constexpr bool f64 = sizeof(T) == 8;
    const SepSide &a = sp.side[0], &b = sp.side[1];
    return product_run(sp.forward, factor(a, args, ws), f64 || a.operand < 0, factor(b, args, ws), f64 || b.operand < 0, out, f64,
                       ws + sp.part_offset, s);
}

template <typename T, typename TO>
static int apply_outer(const tad_plan &pl, const DevProg &prog, const void *const *args, const T *sum, const void *df, TO *out, hipStream_t s) {
    const int n = (int)pl.f_count;
    ArgPtrs A{};
    for (size_t q = 0; q < pl.args.size(); ++q) A.p[q] = args[q];
    const dim3 grid((n + 255) / 256), block(256);
    if (has_register_form(prog))
        TAD_LAUNCH("k_sep_outer", (k_sep_outer<T, TO, 1>), grid, block, 0, s, pl.fwd, prog, (int)pl.args.size(), pl.sep.prog.outer_mask, A,
                   sum, static_cast<const T *>(df), out, n);
    else
        TAD_LAUNCH("k_sep_outer", (k_sep_outer<T, TO, 0>), grid, block, 0, s, pl.fwd, prog, (int)pl.args.size(), pl.sep.prog.outer_mask, A,
                   sum, static_cast<const T *>(df), out, n);
    return launched();
}

template <typename TI, typename T>
static int sum_through_plan(const GatherPlan &g, int64_t count, double pairs, const TI *h, T *dx, int accumulate, char *part, hipStream_t s) {
    const int n = (int)gather_launch_count(g, count);
    if (g.live && !accumulate) {   // the launch visits the unmasked elements only
        TAD_LAUNCH("k_clear", (k_clear<T>), dim3(clear_blocks<T>(count)), dim3(256), 0, s, dx, (long long)count);
        if (launched()) return TAD_EDEVICE;
        accumulate = 1;
    }
    const GatherShape shape = sum_shape(g, n, pairs);
    double *const partial = shape.splits > 1 ? reinterpret_cast<double *>(part) : nullptr;
    int32_t *const flag = shape.splits > 1 ? reinterpret_cast<int32_t *>(part + align256((size_t)n * shape.splits * 8)) : nullptr;
    switch (shape.layout) {
    case kSumThread:
        TAD_LAUNCH("k_sep_sum", (k_sep_sum<TI, T, kSumThread>), dim3((n + 255) / 256), dim3(256), 0, s, g, h, dx, n, accumulate, partial, flag);
        break;
    case kSumWave:
        TAD_LAUNCH("k_sep_sum", (k_sep_sum<TI, T, kSumWave>), dim3((n + 3) / 4), dim3(256), 0, s, g, h, dx, n, accumulate, partial, flag);
        break;
    case kSumBlock:
        TAD_LAUNCH("k_sep_sum", (k_sep_sum<TI, T, kSumBlock>), dim3(n, shape.splits), dim3(256), 0, s, g, h, dx, n, accumulate, partial, flag);
        break;
    default:
        TAD_LAUNCH("k_sep_sum", (k_sep_sum<TI, T, kSumColumns>), dim3((n + 31) / 32, shape.splits), dim3(1024), 0, s, g, h, dx, n, accumulate,
                   partial, flag);
    }
    if (launched()) return TAD_EDEVICE;
    if (shape.splits > 1) {
        TAD_LAUNCH("k_split_finish", (k_split_finish<T>), dim3((n + 3) / 4), dim3(256), 0, s, (const double *)partial, (const int32_t *)flag,
                   shape.splits, dx, n, accumulate);
        return launched();
    }
    return TAD_OK;
}

template <typename T>
static int forward_t(const tad_plan &pl, const void *const *args, void *f, char *ws, hipStream_t s) {
    const SepPlan &sp = pl.sep;
    T *const sum = sp.identity ? static_cast<T *>(f) : reinterpret_cast<T *>(ws + sp.s_offset);
    const int rc = sums<T>(pl, args, sum, ws, s);
    if (rc || sp.identity) return rc;
    return apply_outer<T, T>(pl, sp.prog.outer, args, sum, nullptr, static_cast<T *>(f), s);
}

// every pair of indices reads an element of its own, numbered alike
static bool pairs_are_elements(const tad_plan &sub, int p) {
    if (sub.arg_count[p] != sub.f_count) return false;
    int64_t stride = 1;
    for (int d = sub.expr.n_f - 1; d >= 0; --d) {
        if (sub.expr.f_shape[d] != 1 && sub.fwd.off[p][d] != stride) return false;
        stride *= sub.expr.f_shape[d];
    }
    return true;
}

template <typename T>
static int backward_t(const tad_plan &pl, const void *const *args, const void *df, void *const *dx, char *ws, hipStream_t s) {
    const SepPlan &sp = pl.sep;
    constexpr bool f64 = sizeof(T) == 8;
    const int n_ops = (int)pl.args.size();
    char *const part = ws + sp.part_offset;
    T *const sum = reinterpret_cast<T *>(ws + sp.s_offset);
    const T *g = static_cast<const T *>(df);
    int rc;
    if (!sp.identity) {
        rc = sums<T>(pl, args, sum, ws, s);
        if (rc) return rc;
        T *const gw = reinterpret_cast<T *>(ws + sp.g_offset);
        rc = apply_outer<T, T>(pl, sp.prog.douter, args, sum, df, gw, s);
        if (rc) return rc;
        g = gw;
    } else {
        rc = evaluate_factors<T>(sp, args, ws, s);
        if (rc) return rc;
    }
    bool stored[kMaxArgs] = {};
    for (int q = 0; q < 2; ++q) {
        const SepSide &side = sp.side[q], &other = sp.side[1 - q];
        bool wanted = side.sub == nullptr && side.operand >= 0 && dx[side.operand];
        if (side.sub)
            for (int p : side.operands) wanted = wanted || dx[p];
        if (!wanted) continue;
        const void *o = factor(other, args, ws);
        const bool o64 = f64 || other.operand < 0;
        double *const d = reinterpret_cast<double *>(ws + sp.d_offset);
        void *const to = side.sub ? d : dx[side.operand];
        rc = side.k_major ? product_run(side.grad, o, o64, g, f64, to, f64 || side.sub, part, s)
                          : product_run(side.grad, g, f64, o, o64, to, f64 || side.sub, part, s);
        if (rc) return rc;
        if (!side.sub) {
            stored[side.operand] = true;
            continue;
        }
        const tad_plan &sub = *side.sub;
        const int n = (int)sub.f_count;
        const ArgPtrs A = operand_pointers(side, args);
        for (int p = 0; p < (int)side.operands.size(); ++p) {
            const int op = side.operands[p];
            if (!dx[op]) continue;
            const double *h = d;
            if (side.operand < 0) {
                const DevProg &prog = sub.prog.dinner[p];
                T *const direct = !stored[op] && pairs_are_elements(sub, p) ? static_cast<T *>(dx[op]) : nullptr;
                double *const terms = reinterpret_cast<double *>(ws + sp.h_offset);
                const dim3 grid((n + 255) / 256), block(256);
                if (has_register_form(prog))
                    TAD_LAUNCH("k_sep_terms", (k_sep_terms<T, 1>), grid, block, 0, s, sub.fwd, prog, (int)sub.args.size(), A, d, direct, terms, n);
                else
                    TAD_LAUNCH("k_sep_terms", (k_sep_terms<T, 0>), grid, block, 0, s, sub.fwd, prog, (int)sub.args.size(), A, d, direct, terms, n);
                if (launched()) return TAD_EDEVICE;
                h = direct ? nullptr : terms;
            }
            // (an operand may be read on both sides: the second one adds)
            if (h) rc = sum_through_plan(sub.ap[p].dev, pl.arg_count[op], (double)sub.f_count, h, static_cast<T *>(dx[op]), stored[op], part, s);
            if (rc) return rc;
            stored[op] = true;
        }
    }
    for (int q = 0; q < n_ops; ++q) {
        if (!dx[q]) continue;
        if (!((sp.prog.outer_mask >> q) & 1u)) {
            if (stored[q]) continue;
            TAD_LAUNCH("k_clear", (k_clear<T>), dim3(clear_blocks<T>(pl.arg_count[q])), dim3(256), 0, s, static_cast<T *>(dx[q]),
                       (long long)pl.arg_count[q]);   // nothing reads it
            if (launched()) return TAD_EDEVICE;
            continue;
        }
        // an operand of the outer function: the terms df * d outer / d x, which are g where the outer function adds it to the sum
        const DevProg &prog = sp.prog.douter_arg[q];
        const int add = stored[q] ? 1 : 0;
        if (sp.term_is_g[q]) {
            rc = sum_through_plan(pl.ap_outer[q].dev, pl.arg_count[q], (double)pl.f_count, g, static_cast<T *>(dx[q]), add, part, s);
        } else {
            double *const h = reinterpret_cast<double *>(ws + sp.h_offset);
            rc = apply_outer<T, double>(pl, prog, args, sum, df, h, s);
            if (rc) return rc;
            rc = sum_through_plan(pl.ap_outer[q].dev, pl.arg_count[q], (double)pl.f_count, (const double *)h, static_cast<T *>(dx[q]), add, part, s);
        }
        if (rc) return rc;
    }
    return TAD_OK;
}

int separable_forward(const tad_plan &pl, const void *const *args, void *f, void *ws, hipStream_t s) {
    return pl.dtype == TAD_F64 ? forward_t<double>(pl, args, f, static_cast<char *>(ws), s)
                               : forward_t<float>(pl, args, f, static_cast<char *>(ws), s);
}

int separable_backward(const tad_plan &pl, const void *const *args, const void *df, void *const *dx, void *ws, hipStream_t s) {
    return pl.dtype == TAD_F64 ? backward_t<double>(pl, args, df, dx, static_cast<char *>(ws), s)
                               : backward_t<float>(pl, args, df, dx, static_cast<char *>(ws), s);
}

}  // namespace tad
