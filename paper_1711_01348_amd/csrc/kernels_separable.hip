// Sums of products of two functions as dense products (separable.hpp): the element-wise passes around the products.
//
//   forward    values of the factors that are functions of operands (64 bits), product, outer function
//   backward   the same values and sums again, and with the values the partial derivatives of the factors; g = df * d outer / d s; then
//              per factor its derivative (a product) and per operand of the factor dx_beta = sum over the pairs of indices that
//              read x_beta of derivative * partial derivative: the product's results are multiplied where they leave it, and that is the
//              gradient where every pair reads an element of its own, else terms in the workspace that are summed through the
//              operand's plan
// What a factor or a partial derivative costs is paid once per pair of indices instead of once per term, which leaves
// the products as the bound (64-bit matrix instructions) and, below some 10^8 terms, the launches: 512 x 1024 x 768 with one
// interpreted term per thread 9895 us, 1.2 10^9 interpreted terms.
// The passes over pairs are bound by the interpreted operations and 64-bit functions.  Softplus 512 x 384 x 200, forward and gradients: partial
// derivatives in a pass of their own after the products 61.9 us (passes over pairs 7.9 and 13.2 us); in one launch with the values, the products
// scaled, 60.1 (17.7 us: as much work in a row); value and partial derivatives of a side as one program, which shares exp and cos, 53.5 (11.3 us); arguments
// asked for in one go, here and in the products, 44 (8.4 us).
#include <hip/hip_runtime.h>

#include <algorithm>

#include "element.h"
#include "fetch_args.h"
#include "gather_loop.h"
#include "launch.h"
#include "plan_dev.h"
#include "product_outer.h"
#include "prog_eval.h"
#include "profile.h"
#include "separable.hpp"

namespace tad {

// Passes over the pairs of indices of a factor, several in one launch (a launch costs as much as such a pass): workgroup b works
// on the task with first <= b < first of the next one.
// The kernel's arguments are read from memory, 850 cycles for whatever is asked for at once: what a thread needs first stands at the front.  With a
// plan that was walked index by index and a program read line by line, softplus 512 x 384 x 200 with its gradients took 52.9 us (a pass over
// pairs 8.0 and 11.3), so 47.8; 16 x 16 x 8 34.0 -> 26.3, of it 3.5 for the programs of all launches.
struct PairTask {
    int32_t n, n_ops;
    // the index map as two indices with 32-bit steps, where it comes down to that (inner > 0: the extent of the inner one): operand p is at
    // at[p][outer index * step[0][p] + inner index * step[1][p]], and what is not an operand is the first one's first element
    int32_t inner, step[2][kMaxArgs];
    const void *at[kMaxArgs];
    const double *d;       // null: out = prog, else out = d * prog
    double *out;           // 64-bit results, or null:
    void *dx;              // ... results of the operands' type
    double *results[3];    // a program of several results (all else null): where they go, null for those nobody wants
    DevProg prog;
    ForwardPlan plan;      // pairs of indices -> elements of the operands
    ArgPtrs args;
};
template <int N> struct PairTasks {
    int32_t count, first[N];
    PairTask task[N];
};
// Everything in 64 bits: of 32-bit operands nothing can overflow on the way to a product of factors.
template <typename T, int FORM, int N>
__global__ __launch_bounds__(256) void k_sep_pairs(const PairTasks<N> M) {
    int w = 0, first = 0;
#pragma unroll
    for (int i = 1; i < N; ++i)
        if (i < M.count && (int)blockIdx.x >= M.first[i]) { w = i; first = M.first[i]; }   // the same for the whole workgroup
    const PairTask &t = M.task[w];
    const int lin = ((int)blockIdx.x - first) * 256 + threadIdx.x, n = t.n, inner = t.inner;
    int32_t outer_step[kMaxArgs], inner_step[kMaxArgs];
    const T *at[kMaxArgs];
#pragma unroll
    for (int p = 0; p < kMaxArgs; ++p) {
        outer_step[p] = t.step[0][p];
        inner_step[p] = t.step[1][p];
        at[p] = static_cast<const T *>(t.at[p]);
    }
    // all of it in one go, and with it a word of every line of the program
    static_assert(kMaxArgs == 6 && kMaxProgOps == 64, "fields held here");
    asm volatile("" :: "s"(n), "s"(inner), "s"(outer_step[0]), "s"(outer_step[1]), "s"(outer_step[2]), "s"(outer_step[3]), "s"(outer_step[4]),
                 "s"(outer_step[5]), "s"(inner_step[0]), "s"(inner_step[1]), "s"(inner_step[2]), "s"(inner_step[3]), "s"(inner_step[4]),
                 "s"(inner_step[5]), "s"(at[0]), "s"(at[1]), "s"(at[2]), "s"(at[3]), "s"(at[4]), "s"(at[5]), "s"(t.prog.result),
                 "s"(t.prog.cst[0]), "s"(t.prog.n_words), "s"(t.prog.word[0]), "s"(t.prog.word[16]), "s"(t.prog.word[32]), "s"(t.prog.word[48]));
    if (lin >= n) return;
    double v[kMaxArgs];
    if (inner > 0) {
        const int32_t o = (int32_t)((uint32_t)lin / (uint32_t)inner), i = lin - o * inner;
        T x[kMaxArgs];
#pragma unroll
        for (int p = 0; p < kMaxArgs; ++p) x[p] = at[p][o * outer_step[p] + i * inner_step[p]];
#pragma unroll
        for (int p = 0; p < kMaxArgs; ++p) v[p] = (double)x[p];
    } else {
        element_values<T>(t.plan, t.n_ops, ~0u, t.args, lin, v);
    }
    const double o = prog_eval<double, FORM>(t.prog, v, 0.0, [&](int result, double value) {
        double *const to = result == 0 ? t.results[0] : result == 1 ? t.results[1] : t.results[2];
        if (to) to[lin] = value;
    });
    if (!t.out && !t.dx) return;
    const double r = t.d ? t.d[lin] * o : o;
    if (t.out) t.out[lin] = r;
    else static_cast<T *>(t.dx)[lin] = (T)r;
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
        if (it < n) {   // the rest is sent for together too
            TI v[U];
#pragma unroll
            for (int u = 0; u < U; ++u) v[u] = p[it + u < n ? u * st : 0];
#pragma unroll
            for (int u = 0; u < U; ++u)
                if (it + u < n) acc += (double)v[u];
        }
    }, group, groups);
    *sum = acc;
    return true;
}

template <typename TI, typename T, int LAYOUT>
__global__ __launch_bounds__(LAYOUT == kSumColumns ? 1024 : 256) void k_sep_sum(const GatherPlan P, const TI *__restrict__ h,
                                                                               T *__restrict__ dx, int n, int accumulate,
                                                                               double *__restrict__ partial, int32_t *__restrict__ flag) {
    const int tid = threadIdx.x;
    fetch_gather(P, kSlotF);
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

// ... of the sum alone, U elements per thread, 256 apart: fetching and decoding an operation costs more than carrying it out.
template <typename T, typename TO>
__global__ __launch_bounds__(256) void k_sep_outer_block(const DevProg prog, const T *s, const T *__restrict__ df, TO *out, int n) {
    constexpr int U = ProgWidth<T>::U;
    const int first = blockIdx.x * (256 * U) + threadIdx.x;
    T x[U], d[U], v[kMaxArgs][U] = {}, o[U];
#pragma unroll
    for (int u = 0; u < U; ++u) {
        const int at = min(first + 256 * u, n - 1);
        x[u] = s[at];
        d[u] = df ? df[at] : T(1);
    }
    fetch_program(prog);
    prog_eval_block<T, U, true>(prog, v, x, o);
#pragma unroll
    for (int u = 0; u < U; ++u)
        if (first + 256 * u < n) out[first + 256 * u] = df ? (TO)d[u] * (TO)o[u] : (TO)o[u];
}

static int launched() { return hipGetLastError() == hipSuccess ? TAD_OK : TAD_EDEVICE; }

static ArgPtrs operand_pointers(const SepSide &side, const void *const *args) {
    ArgPtrs A{};
    for (size_t p = 0; p < side.operands.size(); ++p) A.p[p] = args[side.operands[p]];
    return A;
}

// The index map of a pass as two indices: those of extent one fall away, and an index whose step is a whole turn of the one behind it, for every
// operand, is one with it.  No 32-bit form (three indices or more, far operands, no operand): inner = 0.
template <typename T>
static void two_indices(const ForwardPlan &P, PairTask &t) {
    int32_t count = 0, extent[kMaxExt];
    int64_t step[kMaxExt][kMaxArgs];   // from the innermost one
    t.inner = 0;
    for (int p = 0; p < kMaxArgs; ++p) {
        t.at[p] = nullptr;
        t.step[0][p] = t.step[1][p] = 0;
    }
    for (int d = P.n_f - 1; d >= 0; --d) {
        if (P.f_shape[d] == 1) continue;
        bool joins = count > 0;
        for (int p = 0; p < t.n_ops; ++p) joins = joins && P.off[p][d] == step[count - 1][p] * extent[count - 1];
        if (joins) {
            extent[count - 1] *= P.f_shape[d];   // (at most the pairs there are)
            continue;
        }
        extent[count] = P.f_shape[d];
        for (int p = 0; p < t.n_ops; ++p) step[count][p] = P.off[p][d];
        ++count;
    }
    if (count > 2 || t.n_ops < 1) return;
    for (int p = 0; p < t.n_ops; ++p) {
        int64_t reach = 0;
        for (int d = 0; d < count; ++d) {
            if (step[d][p] > INT32_MAX || step[d][p] < -INT32_MAX) return;
            reach += (step[d][p] < 0 ? -step[d][p] : step[d][p]) * (extent[d] - 1);
        }
        if (reach > INT32_MAX) return;
    }
    t.inner = count ? extent[0] : 1;
    for (int p = 0; p < kMaxArgs; ++p) {
        const int of = p < t.n_ops ? p : 0;
        t.at[p] = static_cast<const T *>(t.args.p[of]) + P.base0[of];
        for (int d = 0; d < count && p < t.n_ops; ++d) t.step[1 - d][p] = (int32_t)step[d][p];
    }
}

// passes over pairs of indices collected for one launch
template <typename T>
struct PairPass {
    PairTasks<6> tasks{};
    int blocks = 0;
    bool registers = true, joint = false;
    hipStream_t stream;
    explicit PairPass(hipStream_t s) : stream(s) {}
    int add(const SepSide &side, const void *const *args, const DevProg &prog, const double *d, double *out, void *dx,
            double *const *results = nullptr) {
        // a launch is of one form, and programs of several results are in registers
        if (tasks.count == 6 || (results && !registers) || (joint && !has_register_form(prog))) {
            const int rc = run();
            if (rc) return rc;
        }
        joint = joint || results;
        const tad_plan &sub = *side.sub;
        PairTask &t = tasks.task[tasks.count++];
        t.plan = sub.fwd;
        t.prog = prog;
        t.args = operand_pointers(side, args);
        t.d = d;
        t.out = out;
        t.dx = dx;
        for (int n = 0; n < 3; ++n) t.results[n] = results ? results[n] : nullptr;
        t.n_ops = (int)sub.args.size();
        t.n = (int)sub.f_count;
        two_indices<T>(sub.fwd, t);
        tasks.first[tasks.count - 1] = blocks;
        blocks += (t.n + 255) / 256;
        registers = registers && has_register_form(prog);
        return TAD_OK;
    }
    template <int N> int launch() {
        PairTasks<N> M;
        M.count = tasks.count;
        std::copy(tasks.first, tasks.first + N, M.first);
        std::copy(tasks.task, tasks.task + N, M.task);
        if (registers) TAD_LAUNCH("k_sep_pairs", (k_sep_pairs<T, 1, N>), dim3(blocks), dim3(256), 0, stream, M);
        else TAD_LAUNCH("k_sep_pairs", (k_sep_pairs<T, 0, N>), dim3(blocks), dim3(256), 0, stream, M);
        return launched();
    }
    int run() {
        if (tasks.count == 0) return TAD_OK;
        const int rc = tasks.count <= 2 ? launch<2>() : tasks.count == 3 ? launch<3>() : launch<6>();
        tasks.count = blocks = 0;
        registers = true;
        joint = false;
        return rc;
    }
};

// Where a gradient's partial derivative is kept for the product to scale its results by: an aligned operand's in the place of the
// factor's derivative, which is not stored then, another one's where its terms go.
static double *partial_place(const SepSide &side, int p, char *ws) {
    return reinterpret_cast<double *>(ws + (side.aligned[p] ? side.d_offset : side.h_offset[p]));
}

// a factor like exp(x) r: the partial derivative is the value
static bool partial_is_value(const SepSide &side, int p) { return same_program(side.sub->prog.inner, side.sub->prog.dinner[p]); }

// Is there one program for the value and the partial derivatives that are wanted?  (Derivatives of one node have one place: equal ones share
// it with the value only.)
static bool joint_side(const SepSide &side, const void *const *dx) {
    if (!side.joint_on) return false;
    uint32_t taken = 1u << side.joint_place[0];
    for (size_t p = 0; p < side.operands.size(); ++p) {
        const int place = side.joint_place[1 + p];
        if ((place >= 0) != (dx[side.operands[p]] != nullptr)) return false;
        if (place < 0) continue;
        if (place == side.joint_place[0]) {
            if (!partial_is_value(side, (int)p)) return false;
            continue;
        }
        if (place > 2 || (taken >> place & 1u)) return false;
        taken |= 1u << place;
    }
    return side.joint_place[0] <= 2;
}

// Can the product that yields a side's derivative multiply it by the partial derivatives?  (In a large workspace the terms of an operand take the
// place of the factor's values, which the products read.)
static bool scaled_side(const SepSide &side, const ProductDesc &d, const void *const *dx, bool one_of_two) {
    if (!side.sub || side.operand >= 0 || !product_scales(d, one_of_two)) return false;
    int wanted = 0, aligned = 0;
    for (size_t p = 0; p < side.operands.size(); ++p) {
        if (!dx[side.operands[p]]) continue;
        ++wanted;
        if (side.aligned[p]) ++aligned;
        else if (side.h_offset[p] == side.value_offset) return false;
    }
    return wanted >= 1 && wanted <= 2 && aligned <= 1;
}

// the factors that are functions of operands, and with them the partial derivatives (dx: the gradients wanted) of the sides that `scaled` says
template <typename T>
static int evaluate_factors(const SepPlan &sp, const void *const *args, char *ws, hipStream_t s, const bool *scaled = nullptr,
                            const void *const *dx = nullptr) {
    PairPass<T> pass(s);
    for (int q = 0; q < 2; ++q) {
        const SepSide &side = sp.side[q];
        if (side.operand >= 0) continue;
        double *const value = reinterpret_cast<double *>(ws + side.value_offset);
        int rc;
        if (scaled && scaled[q] && joint_side(side, dx)) {   // functions that value and partial derivatives share are evaluated once
            double *results[3] = {};
            for (size_t p = 0; p < side.operands.size(); ++p)
                if (dx[side.operands[p]]) results[side.joint_place[1 + p]] = partial_place(side, (int)p, ws);
            results[side.joint_place[0]] = value;
            rc = pass.add(side, args, side.joint, nullptr, nullptr, nullptr, results);
            if (rc) return rc;
            continue;
        }
        rc = pass.add(side, args, side.sub->prog.inner, nullptr, value, nullptr);
        for (int p = 0; !rc && scaled && scaled[q] && p < (int)side.operands.size(); ++p)
            if (dx[side.operands[p]] && !partial_is_value(side, p)) rc = pass.add(side, args, side.sub->prog.dinner[p], nullptr, partial_place(side, p, ws), nullptr);
        if (rc) return rc;
    }
    return pass.run();
}

static const void *factor(const SepSide &side, const void *const *args, const char *ws) {
    return side.operand >= 0 ? args[side.operand] : ws + side.value_offset;
}

template <typename T, typename TO>
static int apply_outer(const tad_plan &pl, const ProgramBody &pb, const DevProg &prog, const void *const *args, const T *sum, const void *df,
                       TO *out, hipStream_t s) {
    const int n = (int)pl.f_count;
    ArgPtrs A{};
    for (size_t q = 0; q < pl.args.size(); ++q) A.p[q] = args[pl.root[q]];
    const dim3 grid((n + 255) / 256), block(256);
    constexpr int U = ProgWidth<T>::U;
    // (dense layers with tanh, gradients, a thread per element with the walk through the plan / this: 16 x 16 x 16 8.6 / 7.0 us, 512 x 1024 x 768 44.2 / 40.7)
    if (has_register_form(prog) && !reads_operands(prog))
        TAD_LAUNCH("k_sep_outer", (k_sep_outer_block<T, TO>), dim3((n + 256 * U - 1) / (256 * U)), block, 0, s, prog, sum, static_cast<const T *>(df), out, n);
    else if (has_register_form(prog))
        TAD_LAUNCH("k_sep_outer", (k_sep_outer<T, TO, 1>), grid, block, 0, s, pl.fwd, prog, (int)pl.args.size(), pb.outer_mask, A,
                   sum, static_cast<const T *>(df), out, n);
    else
        TAD_LAUNCH("k_sep_outer", (k_sep_outer<T, TO, 0>), grid, block, 0, s, pl.fwd, prog, (int)pl.args.size(), pb.outer_mask, A,
                   sum, static_cast<const T *>(df), out, n);
    return launched();
}

// Sums through `prog` (null: stored as they are) into out; s_out (may be null): where the sums themselves are needed as well.
// df: see k_sep_outer.
template <typename T>
static int sums(const tad_plan &pl, const ProductSet &set, const DevProg *prog, const void *const *args, const void *df, void *out, T *s_out, char *ws, hipStream_t s,
                const bool *scaled = nullptr, const void *const *dx = nullptr) {
    const SepPlan &sp = pl.sep;
    int rc = evaluate_factors<T>(sp, args, ws, s, scaled, dx);
    if (rc) return rc;
    constexpr bool f64 = sizeof(T) == 8;
    const SepSide &a = sp.side[0], &b = sp.side[1];
    ProductJob j = {&set.forward, factor(a, args, ws), f64 || a.operand < 0, factor(b, args, ws), f64 || b.operand < 0, out, f64};
    if (prog && has_register_form(*prog) && sp.outer_linear && product_outer_fits(set.forward)) {
        ProductOuter o{};
        o.prog = *prog;
        for (size_t q = 0; q < pl.args.size(); ++q) {
            if (!((sp.prog.outer_mask >> q) & 1u)) continue;
            o.args.p[q] = args[q];
            o.off_r[q] = sp.outer_r[q];
            o.off_c[q] = sp.outer_c[q];
        }
        o.df = df;
        o.s_out = s_out;
        return product_run_outer(j, o, s);
    }
    T *const sum = s_out ? s_out : reinterpret_cast<T *>(ws + sp.s_offset);
    if (prog) j.c = sum;
    rc = product_run(j, ws + sp.part_offset, s);
    if (rc || !prog) return rc;
    return apply_outer<T, T>(pl, sp.prog, *prog, args, sum, df, static_cast<T *>(out), s);
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

// is the operand part of a factor (whose gradient is added to that of the outer function)?
static bool inner_reads(const SepPlan &sp, int operand) {
    for (const SepSide &side : sp.side) {
        if (side.operand == operand) return true;
        for (int p : side.operands)
            if (p == operand) return true;
    }
    return false;
}

template <typename T>
static int forward_t(const tad_plan &pl, const ProductSet &set, const void *const *args, void *f, char *ws, hipStream_t s) {
    return sums<T>(pl, set, pl.sep.identity ? nullptr : &pl.sep.prog.outer, args, nullptr, f, nullptr, ws, s);
}

template <typename T>
static int backward_t(const tad_plan &pl, const ProductSet &set, const void *const *args, const void *f, const void *df, void *const *dx, char *ws, hipStream_t s) {
    const SepPlan &sp = pl.sep;
    constexpr bool f64 = sizeof(T) == 8;
    const int n_ops = (int)pl.args.size();
    char *const part = ws + sp.part_offset;
    const T *g = static_cast<const T *>(df), *sum = nullptr;
    // the derivatives of the outer function are those of f where they can be: that saves the sums
    const bool from_f = outer_in_f(pl, sp.prog, dx);
    bool wanted[2] = {}, scaled[2];
    for (int q = 0; q < 2; ++q) {
        const SepSide &side = sp.side[q];
        if (side.sub)
            for (int p : side.operands) wanted[q] = wanted[q] || dx[p];
        else
            wanted[q] = dx[side.operand] != nullptr;
    }
    for (int q = 0; q < 2; ++q) scaled[q] = scaled_side(sp.side[q], set.grad[q], dx, wanted[0] && wanted[1]);
    int rc;
    if (sp.identity || from_f) {
        rc = evaluate_factors<T>(sp, args, ws, s, scaled, dx);
        if (!rc && !sp.identity) {
            T *const gw = reinterpret_cast<T *>(ws + sp.g_offset);
            sum = static_cast<const T *>(f);
            rc = apply_outer<T, T>(pl, sp.prog, sp.prog.douter_f, args, sum, df, gw, s);
            g = gw;
        }
    } else {
        T *s_out = nullptr;   // the sums themselves: for the terms of operands of the outer function that are not g
        for (int q = 0; q < n_ops; ++q)
            if (dx[q] && ((sp.prog.outer_mask >> q) & 1u) && !sp.term_is_g[q]) s_out = reinterpret_cast<T *>(ws + sp.s_offset);
        T *const gw = reinterpret_cast<T *>(ws + sp.g_offset);
        rc = sums<T>(pl, set, &sp.prog.douter, args, df, gw, s_out, ws, s, scaled, dx);
        g = gw;
        sum = s_out;
    }
    if (rc) return rc;
    // the derivatives of the factors
    bool stored[kMaxArgs] = {};
    ProductJob jobs[2];
    int n_jobs = 0;
    for (int q = 0; q < 2; ++q) {
        const SepSide &side = sp.side[q], &other = sp.side[1 - q];
        if (!wanted[q]) continue;
        const void *o = factor(other, args, ws);
        const bool o64 = f64 || other.operand < 0, wide = f64 || side.sub;
        void *const to = side.sub ? ws + side.d_offset : dx[side.operand];
        if (side.k_major) jobs[n_jobs++] = {&set.grad[q], o, o64, g, f64, to, wide};
        else jobs[n_jobs++] = {&set.grad[q], g, f64, o, o64, to, wide};
        if (!side.sub) stored[side.operand] = true;
        for (int p = 0; scaled[q] && p < (int)side.operands.size(); ++p) {
            void *const d = dx[side.operands[p]];
            if (!d) continue;
            ProductJob &j = jobs[n_jobs - 1];
            j.by[j.scaled] = partial_is_value(side, p) ? reinterpret_cast<const double *>(ws + side.value_offset) : partial_place(side, p, ws);
            j.to[j.scaled] = side.aligned[p] ? d : partial_place(side, p, ws);
            j.to64[j.scaled++] = f64 || !side.aligned[p];
        }
    }
    // the gradient of a bias along the trailing indices, the column sums of g, beside the first product: in a launch of its own it takes as long
    // as launches do (512 x 1024 x 768 6.7 us of 68).  Its 32 threads per column are not to outlast the product.  Gradients of M x N x K, beside / in a launch
    // of its own: 1000 x 16 x 16 16.4 / 25.0 us, 4000 x 16 x 16 21.6 / 26.7, 6000 x 16 x 16 25.6 / 27.8, x 512 x 512 167 / 176; 8000 x 16 x 16 28.4 / 27.7, x 512 x 512 194 / 194,
    // 16000 x 64 x 64 52 / 39.
    ProductColumns columns{};
    bool summed[kMaxArgs] = {};
    for (int q = 0; n_jobs && !columns.out && q < n_ops; ++q) {
        if (!dx[q] || !((sp.prog.outer_mask >> q) & 1u) || !sp.term_is_g[q] || stored[q] || !sp.outer_linear) continue;
        if (sp.outer_r[q] != 0 || sp.outer_c[q] != 1 || pl.arg_count[q] != sp.N || sp.M > 6144 || inner_reads(sp, q)) continue;
        columns = {g, dx[q], (int)sp.M, (int)sp.N, f64};
        summed[q] = true;
    }
    const ProductColumns *const beside = columns.out ? &columns : nullptr;
    rc = n_jobs == 2 ? product_run_two(jobs[0], jobs[1], part, s, beside) : n_jobs == 1 ? product_run(jobs[0], part, s, beside) : TAD_OK;
    if (rc) return rc;
    // derivative of the factor * derivative by its operand, at every pair of indices ...
    PairPass<T> pass(s);
    bool direct[2][kMaxArgs] = {};
    for (int q = 0; q < 2; ++q) {
        const SepSide &side = sp.side[q];
        if (!wanted[q] || !side.sub || side.operand >= 0) continue;
        for (int p = 0; p < (int)side.operands.size(); ++p) {
            const int op = side.operands[p];
            if (!dx[op]) continue;
            // an aligned operand moves along the side's function index: the other side does not read it
            direct[q][p] = side.aligned[p];
            if (direct[q][p]) stored[op] = true;
            if (scaled[q]) continue;
            rc = pass.add(side, args, side.sub->prog.dinner[p], reinterpret_cast<const double *>(ws + side.d_offset),
                          direct[q][p] ? nullptr : reinterpret_cast<double *>(ws + side.h_offset[p]), dx[op]);
            if (rc) return rc;
        }
    }
    rc = pass.run();
    if (rc) return rc;
    // ... and the sums of those that read the same element
    for (int q = 0; q < 2; ++q) {
        const SepSide &side = sp.side[q];
        if (!wanted[q] || !side.sub) continue;
        for (int p = 0; p < (int)side.operands.size(); ++p) {
            const int op = side.operands[p];
            if (!dx[op] || direct[q][p]) continue;
            const size_t at = side.operand >= 0 ? side.d_offset : side.h_offset[p];
            // (an operand may be read on both sides: the second one adds)
            rc = sum_through_plan(side.sub->ap[p].dev, pl.arg_count[op], (double)side.sub->f_count, reinterpret_cast<const double *>(ws + at),
                                  static_cast<T *>(dx[op]), stored[op], part, s);
            if (rc) return rc;
            stored[op] = true;
        }
    }
    for (int q = 0; q < n_ops; ++q) {
        if (!dx[q] || summed[q]) continue;
        if (!((sp.prog.outer_mask >> q) & 1u)) {
            if (stored[q]) continue;
            TAD_LAUNCH("k_clear", (k_clear<T>), dim3(clear_blocks<T>(pl.arg_count[q])), dim3(256), 0, s, static_cast<T *>(dx[q]),
                       (long long)pl.arg_count[q]);   // nothing reads it
            if (launched()) return TAD_EDEVICE;
            continue;
        }
        // an operand of the outer function: the terms df * d outer / d x, which are g where the outer function adds it to the sum
        const DevProg &prog = from_f ? sp.prog.douter_arg_f[q] : sp.prog.douter_arg[q];
        const int add = stored[q] ? 1 : 0;
        if (sp.term_is_g[q]) {
            rc = sum_through_plan(pl.ap_outer[q].dev, pl.arg_count[q], (double)pl.f_count, g, static_cast<T *>(dx[q]), add, part, s);
        } else {
            double *const h = reinterpret_cast<double *>(ws + sp.h_offset);
            rc = apply_outer<T, double>(pl, sp.prog, prog, args, sum, df, h, s);
            if (rc) return rc;
            rc = sum_through_plan(pl.ap_outer[q].dev, pl.arg_count[q], (double)pl.f_count, (const double *)h, static_cast<T *>(dx[q]), add, part, s);
        }
        if (rc) return rc;
    }
    return TAD_OK;
}

int separable_forward(const tad_plan &pl, const ProductSet &set, const void *const *args, void *f, void *ws, hipStream_t s) {
    return pl.dtype == TAD_F64 ? forward_t<double>(pl, set, args, f, static_cast<char *>(ws), s)
                               : forward_t<float>(pl, set, args, f, static_cast<char *>(ws), s);
}

int separable_backward(const tad_plan &pl, const ProductSet &set, const void *const *args, const void *f, const void *df, void *const *dx, void *ws, hipStream_t s) {
    return pl.dtype == TAD_F64 ? backward_t<double>(pl, set, args, f, df, dx, static_cast<char *>(ws), s)
                               : backward_t<float>(pl, set, args, f, df, dx, static_cast<char *>(ws), s);
}

int program_outer(const tad_plan &pl, const ProgramBody &pb, const DevProg &prog, const void *const *args, const void *s, const void *df,
                  void *out, hipStream_t stream) {
    return pl.dtype == TAD_F64
               ? apply_outer<double, double>(pl, pb, prog, args, static_cast<const double *>(s), df, static_cast<double *>(out), stream)
               : apply_outer<float, float>(pl, pb, prog, args, static_cast<const float *>(s), df, static_cast<float *>(out), stream);
}

bool outer_in_f(const tad_plan &pl, const ProgramBody &pb, void *const *dx) {
    uint32_t need = 1u << TAD_MAX_ARGS;
    for (size_t q = 0; q < pl.args.size(); ++q)
        if (dx[pl.root[q]] && ((pb.outer_mask >> q) & 1u)) need |= 1u << q;
    return (pb.in_f & need) == need;
}

}  // namespace tad
