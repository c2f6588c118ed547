// Interpreter of the scalar programs (program.hpp) on the device: shared by the plan-driven kernels and by the element-wise
// passes of sums that run as dense products.
#pragma once
#include <hip/hip_runtime.h>

#include <type_traits>

#include "plan_dev.h"

namespace tad {

// A program is read from the kernel's arguments line by line as it runs, 850 cycles a line that the scalar cache does not hold: a kernel that has
// something else to wait for first asks for a word of every line here.
__device__ __forceinline__ void fetch_program(const DevProg &P) {
    static_assert(kMaxProgOps == 64, "four lines of words");
    asm volatile("" :: "s"(P.result), "s"(P.cst[0]), "s"(P.n_words), "s"(P.word[0]), "s"(P.word[16]), "s"(P.word[32]), "s"(P.word[48]));
}

template <typename T> struct Fn;
template <> struct Fn<float> {
    static __device__ __forceinline__ float exp_(float x) { return expf(x); }
    static __device__ __forceinline__ float log_(float x) { return logf(x); }
    static __device__ __forceinline__ float sin_(float x) { return sinf(x); }
    static __device__ __forceinline__ float cos_(float x) { return cosf(x); }
    static __device__ __forceinline__ float tanh_(float x) { return tanhf(x); }
    static __device__ __forceinline__ float sqrt_(float x) { return sqrtf(x); }
};
template <> struct Fn<double> {
    static __device__ __forceinline__ double exp_(double x) { return exp(x); }
    static __device__ __forceinline__ double log_(double x) { return log(x); }
    static __device__ __forceinline__ double sin_(double x) { return sin(x); }
    static __device__ __forceinline__ double cos_(double x) { return cos(x); }
    static __device__ __forceinline__ double tanh_(double x) { return tanh(x); }
    static __device__ __forceinline__ double sqrt_(double x) { return sqrt(x); }
};

template <typename T>
__device__ __forceinline__ T prog_unary(int op, T x, int k) {
    switch (op) {
    case P_NEG: return -x;
    case P_EXP: return Fn<T>::exp_(x);
    case P_LOG: return Fn<T>::log_(x);
    case P_SIN: return Fn<T>::sin_(x);
    case P_COS: return Fn<T>::cos_(x);
    case P_TANH: return Fn<T>::tanh_(x);
    case P_SQRT: return Fn<T>::sqrt_(x);
    case P_POWI: {
        T r = x;
        for (int e = 1; e < k; ++e) r *= x;
        return r;
    }
    default: return T(0);
    }
}

// One pass over the operations of the form with one temporary per operation; the temporaries live in the
// thread's private memory (programs whose live values do not fit the register form).
template <typename T>
__device__ __forceinline__ T prog_eval_temporaries(const DevProg &P, const T *v, T s) {
    T t[kMaxProgOps];
    for (int i = 0; i < P.n; ++i) {
        const int a = P.a[i], b = P.b[i];
        T r;
        switch (P.op[i]) {
        case P_CONST: r = (T)P.cst[a]; break;
        case P_ARG: r = v[a]; break;
        case P_SUM: r = s; break;
        case P_ADD: r = t[a] + t[b]; break;
        case P_SUB: r = t[a] - t[b]; break;
        case P_MUL: r = t[a] * t[b]; break;
        case P_DIV: r = t[a] / t[b]; break;
        default: r = prog_unary<T>(P.op[i], t[a], P.k[i]);
        }
        t[i] = r;
    }
    return t[P.result];
}

// The register form, for U terms at once: kProgRegs values per term in vector registers, addressed by the
// wave-uniform register numbers of the operation words (every lane runs the same program, so the words are
// scalar loads from the kernel arguments; the next word is fetched while the current operation runs).  Fetching
// and decoding an operation costs more than carrying it out: U terms share that cost.  One array per term: an
// array of kProgRegs values indexed by a uniform number stays in registers, a two-dimensional one does not.
template <typename T> struct ProgWidth { static constexpr int U = sizeof(T) == 4 ? 4 : 2; };   // terms per pass

// REGS chooses the form at compile time: a kernel holds one of the two, so that the kernels of the register
// form need no private memory at all (the runtime sets private memory up per launch, and slowly once a kernel asks
// for much of it).  The kernels below are built in three forms (template parameter FORM): 0 one temporary per
// operation, one term per pass; 1 registers, one term per pass (elements with one or two terms: several terms per
// pass would only cost registers, i.e. waves per SIMD); 2 registers, ProgWidth<T>::U terms per pass.
// sink(n, value of the first term): results of a program of several (register form); nothing in all others.
struct NoSink {
    template <typename T> __device__ __forceinline__ void operator()(int, T) const {}
};
template <typename T, int U, bool REGS, typename SINK = NoSink>
__device__ __forceinline__ void prog_eval_block(const DevProg &P, const T (&v)[kMaxArgs][U], const T (&s)[U], T (&out)[U], SINK sink = SINK()) {
    static_assert(U >= 1 && U <= 4, "one register array per term below");
    if (P.result < 0) {
#pragma unroll
        for (int u = 0; u < U; ++u) out[u] = T(0);
        return;
    }
    if (!REGS) {
#pragma unroll
        for (int u = 0; u < U; ++u) {
            T col[kMaxArgs];
#pragma unroll
            for (int q = 0; q < kMaxArgs; ++q) col[q] = v[q][u];
            out[u] = prog_eval_temporaries<T>(P, col, s[u]);
        }
        return;
    }
    // not cleared: the allocation on the host writes every register before it is read
    T r0[kProgRegs], r1[kProgRegs], r2[kProgRegs], r3[kProgRegs];
    // DST[u] = EXPR for every term u; EXPR sees the term's register array as `r` and its number as `u`
#define TAD_EACH_TERM(DST, EXPR)                                                                    \
    {                                                                                               \
        { T(&r)[kProgRegs] = r0; constexpr int u = 0; (void)r; (void)u; DST[u] = EXPR; }            \
        if (U > 1) { T(&r)[kProgRegs] = r1; constexpr int u = U > 1 ? 1 : 0; (void)r; (void)u; DST[u] = EXPR; } \
        if (U > 2) { T(&r)[kProgRegs] = r2; constexpr int u = U > 2 ? 2 : 0; (void)r; (void)u; DST[u] = EXPR; } \
        if (U > 3) { T(&r)[kProgRegs] = r3; constexpr int u = U > 3 ? 3 : 0; (void)r; (void)u; DST[u] = EXPR; } \
    }
    // DST[u] = the operand with code CODE (wave-uniform): a register, a tensor operand, a constant or the sum.
    // The operand number selects code, not an address: v stays in registers.
#define TAD_FETCH(DST, CODE)                                                         \
    {                                                                                \
        static_assert(kMaxArgs == 6, "one case per operand");                        \
        const int code_ = (CODE);                                                    \
        if (code_ < kCodeArg) {                                                      \
            const int reg_ = code_ & (kProgRegs - 1);                                \
            TAD_EACH_TERM(DST, r[reg_])                                              \
        } else if (code_ < kCodeConst) {                                             \
            switch (code_ - kCodeArg) {                                              \
            case 0: TAD_EACH_TERM(DST, v[0][u]) break;                               \
            case 1: TAD_EACH_TERM(DST, v[1][u]) break;                               \
            case 2: TAD_EACH_TERM(DST, v[2][u]) break;                               \
            case 3: TAD_EACH_TERM(DST, v[3][u]) break;                               \
            case 4: TAD_EACH_TERM(DST, v[4][u]) break;                               \
            default: TAD_EACH_TERM(DST, v[5][u])                                     \
            }                                                                        \
        } else if (code_ < kCodeSum) {                                               \
            const T cst_ = (T)P.cst[(code_ - kCodeConst) & (kMaxProgConst - 1)];     \
            TAD_EACH_TERM(DST, cst_)                                                 \
        } else {                                                                     \
            TAD_EACH_TERM(DST, s[u])                                                 \
        }                                                                            \
    }
    uint32_t w = P.word[0];
    for (int i = 0; i < P.n_words; ++i) {
        const uint32_t next = P.word[(i + 1) & (kMaxProgOps - 1)];
        const int op = (int)(w & 0xff), first = (int)((w >> 8) & 0xff), second = (int)((w >> 16) & 0xff);
        const int dst = (int)(w >> 24) & (kProgRegs - 1);
        T x[U], y[U], o[U];
        TAD_FETCH(x, first)
        if (op >= P_ADD && op <= P_DIV) TAD_FETCH(y, second)
        switch (op) {
        case P_ADD:
#pragma unroll
            for (int u = 0; u < U; ++u) o[u] = x[u] + y[u];
            break;
        case P_SUB:
#pragma unroll
            for (int u = 0; u < U; ++u) o[u] = x[u] - y[u];
            break;
        case P_MUL:
#pragma unroll
            for (int u = 0; u < U; ++u) o[u] = x[u] * y[u];
            break;
        case P_DIV:
#pragma unroll
            for (int u = 0; u < U; ++u) o[u] = x[u] / y[u];
            break;
        default:
#pragma unroll
            for (int u = 0; u < U; ++u) o[u] = prog_unary<T>(op, x[u], second);
        }
        if constexpr (!std::is_same<SINK, NoSink>::value) {
            if (w >> 28) sink((int)(w >> 28) - 1, o[0]);   // the same for the whole wavefront
        }
        r0[dst] = o[0];
        if (U > 1) r1[dst] = o[U > 1 ? 1 : 0];
        if (U > 2) r2[dst] = o[U > 2 ? 2 : 0];
        if (U > 3) r3[dst] = o[U > 3 ? 3 : 0];
        w = next;
    }
    TAD_FETCH(out, P.result_code)
#undef TAD_FETCH
#undef TAD_EACH_TERM
}

// one term
template <typename T, int FORM, typename SINK = NoSink>
__device__ __forceinline__ T prog_eval(const DevProg &P, const T *v, T s, SINK sink = SINK()) {
    T vv[kMaxArgs][1], ss[1] = {s}, out[1];
#pragma unroll
    for (int q = 0; q < kMaxArgs; ++q) vv[q][0] = v[q];
    prog_eval_block<T, 1, (FORM > 0), SINK>(P, vv, ss, out, sink);
    return out[0];
}

// a program that is identically zero is never interpreted
inline bool has_register_form(const DevProg &P) { return P.result < 0 || P.n_regs >= 0; }

}  // namespace tad
