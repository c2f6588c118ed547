// The two streaming patterns of kernels_patterns.hip for the forms those do not take, rows of f that start anywhere (J not a
// multiple of four) and 64-bit tensors:
//
//   f_ij = phi(x_i)       dx_i = phi'(x_i) sum_j df_ij
//   f_ij = phi(x_{i+j})   dx_m = phi'(x_m) sum_{i in window(m)} df_{i,m-i}
//
// Bound by one write and one read of a tensor of f's size.  Forward, f is one run of elements, 16 bytes per thread whatever
// row they lie in.  The sums are in 64 bits, as those of the plan-driven kernels, which evaluate these forms otherwise (a
// wavefront per element, or one for 64 elements in turn; along an antidiagonal its lanes read a row apart: 4096 x 4095
// 223 us, 1000 x 1001 261 us, row sums of 1000 x 1001 220 us).  Antidiagonal sums: a wavefront takes 64 neighbouring m and the rows
// of one chunk, so that each of its loads is a contiguous piece of a row, and a second pass adds the chunks in the window.
#include <hip/hip_runtime.h>

#include "bodies.h"
#include "gather_loop.h"
#include "launch.h"
#include "launch_geom.h"
#include "plan_dev.h"
#include "profile.h"

namespace tad {

template <int BODY, typename T> __device__ __forceinline__ T phi(T x) { return body_outer<BODY, T>(x); }
template <int BODY, typename T> __device__ __forceinline__ T dphi(T x) {
    T v[1] = {x};
    return body_douter<BODY, T>(BODY == TAD_BODY_EXP ? phi<BODY, T>(x) : T(0), v);
}

// SUM: x is read at i + j, else at i.  `aligned`: f starts on a 16-byte boundary
template <int BODY, typename T, bool SUM>
__global__ __launch_bounds__(256) void k_pattern_wide_forward(const T *__restrict__ x, T *__restrict__ f, int n, int J, int aligned) {
    constexpr int V = 16 / (int)sizeof(T);
    typedef T vec __attribute__((ext_vector_type(V)));
    const long long e64 = ((long long)blockIdx.x * 256 + threadIdx.x) * V;
    if (e64 >= n) return;
    const int e = (int)e64, here = min(V, n - e);
    int i = e / J, j = e - i * J;
    vec o;
    if (j + V <= J) {   // within one row: a single load, or a single value
        T xv[V];
        if constexpr (SUM) {
            __builtin_memcpy(xv, x + (i + j), sizeof xv);
#pragma unroll
            for (int v = 0; v < V; ++v) o[v] = phi<BODY, T>(xv[v]);
        } else {
            const T p = phi<BODY, T>(x[i]);
#pragma unroll
            for (int v = 0; v < V; ++v) o[v] = p;
        }
    } else {
#pragma unroll
        for (int v = 0; v < V; ++v) {
            o[v] = v < here ? phi<BODY, T>(x[SUM ? i + j : i]) : T(0);
            if (++j == J) { j = 0; ++i; }
        }
    }
    if (aligned && here == V) {
        __builtin_nontemporal_store(o, reinterpret_cast<vec *>(f + e));
    } else {
#pragma unroll
        for (int v = 0; v < V; ++v)
            if (v < here) f[e + v] = o[v];
    }
}

// one wavefront (WAVES = 1, four rows per workgroup) or one workgroup of four per row
template <int BODY, typename T, int WAVES>
__global__ __launch_bounds__(256) void k_rowreduce_wide_backward(const FlatFeas feas, const T *__restrict__ x, const T *__restrict__ df,
                                                                 T *__restrict__ dx, int n_x, int J) {
    __shared__ double red[4];
    const int tid = threadIdx.x, lane = tid & 63, i = WAVES == 1 ? blockIdx.x * 4 + (tid >> 6) : blockIdx.x;
    if (WAVES == 1 && i >= n_x) return;
    const int32_t y[3] = {i, 0, 0};
    double s = 0.0;
    const bool live = flat_feasible(feas, y);   // elements of x beyond f's rows: no terms
    if (live) {
        constexpr int STEP = 64 * WAVES, U = 8;
        const T *p = df + (size_t)i * J;
        int j = WAVES == 1 ? lane : tid;
        for (; j + (U - 1) * STEP < J; j += U * STEP) {
            T v[U];
#pragma unroll
            for (int u = 0; u < U; ++u) v[u] = __builtin_nontemporal_load(p + j + u * STEP);
#pragma unroll
            for (int u = 0; u < U; ++u) s += (double)v[u];
        }
        for (; j < J; j += STEP) s += (double)p[j];
    }
    s = WAVES == 1 ? wave_sum_all(s) : block_sum_256(s, red);
    if ((WAVES == 1 ? lane : tid) == 0) dx[i] = live ? (T)((double)dphi<BODY, T>(x[i]) * s) : T(0);
}

// part[chunk][m - first row of the chunk]
template <typename T>
__global__ __launch_bounds__(256) void k_antidiag_wide_backward(const T *__restrict__ df, double *__restrict__ part, int I, int J,
                                                                int chunk_rows, int tiles) {
    const int chunk = blockIdx.x / tiles;
    const int i0 = chunk * chunk_rows, i1 = min(i0 + chunk_rows, I), W = J + chunk_rows;
    const int o = (int)(blockIdx.x - chunk * tiles) * 256 + threadIdx.x, o_first = o - (int)(threadIdx.x & 63);   // m = i0 + o
    if (o_first >= W) return;   // the whole wavefront
    double s = 0.0;
    const T *p = df + (size_t)i0 * J + o;   // element (i0, o): one row further down, one column to the left
    constexpr int U = 8;
    if (o_first - (i1 - 1 - i0) >= 0 && o_first + 63 < J) {   // every element of the wavefront's rows exists
        int r = 0;
        for (; r + U <= i1 - i0; r += U) {
            T v[U];
#pragma unroll
            for (int u = 0; u < U; ++u) v[u] = __builtin_nontemporal_load(p + (size_t)(r + u) * (J - 1));
#pragma unroll
            for (int u = 0; u < U; ++u) s += (double)v[u];
        }
        for (; r < i1 - i0; ++r) s += (double)p[(size_t)r * (J - 1)];
    } else {
        for (int r = 0; r < i1 - i0; r += U) {
            T v[U];
#pragma unroll
            for (int u = 0; u < U; ++u) {
                const int j = o - r - u;
                v[u] = r + u < i1 - i0 && j >= 0 && j < J ? df[(size_t)(i0 + r + u) * J + j] : T(0);
            }
#pragma unroll
            for (int u = 0; u < U; ++u) s += (double)v[u];
        }
    }
    if (o < W) part[(size_t)chunk * W + o] = s;
}

// 64 elements per workgroup; its four wavefronts take the chunks in the window in turn
template <int BODY, typename T>
__global__ __launch_bounds__(256) void k_antidiag_wide_finish(const FlatFeas feas, const FlatLevel win, int iy, int iz, const T *__restrict__ x,
                                                              const double *__restrict__ part, T *__restrict__ dx, int n_x, int J,
                                                              int chunk_rows) {
    __shared__ double red[4][64];
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, m = blockIdx.x * 64 + lane, W = J + chunk_rows;
    double s = 0.0;
    bool live = false;
    if (m < n_x) {
        const int32_t y[3] = {m, 0, 0};   // the transformed index is the gradient index (checked on the host)
        int32_t lo = 0, hi = -1;
        if (flat_feasible(feas, y)) flat_bounds(win, y, lo, hi);
        if (lo <= hi) {
            live = true;
            const int ia = iy * m + iz * lo, ib = iy * m + iz * hi;
            const int first = min(ia, ib) / chunk_rows, last = max(ia, ib) / chunk_rows;
            for (int c = first + wave; c <= last; c += 4) s += part[(size_t)c * W + (m - c * chunk_rows)];
        }
    }
    red[wave][lane] = s;
    __syncthreads();
    if (wave != 0 || m >= n_x) return;
    s = (red[0][lane] + red[1][lane]) + (red[2][lane] + red[3][lane]);
    dx[m] = live ? (T)((double)dphi<BODY, T>(x[m]) * s) : T(0);
}

#define TAD_UNARY_SWITCH(body, CALL)                                   \
    switch (body) {                                                    \
    case TAD_BODY_SQ: { constexpr int B_ = TAD_BODY_SQ; CALL; break; }       \
    case TAD_BODY_CUBE: { constexpr int B_ = TAD_BODY_CUBE; CALL; break; }   \
    case TAD_BODY_SIN: { constexpr int B_ = TAD_BODY_SIN; CALL; break; }     \
    case TAD_BODY_EXP: { constexpr int B_ = TAD_BODY_EXP; CALL; break; }     \
    default: return TAD_EUNSUPPORTED;                                  \
    }

template <typename T>
static int forward_t(const tad_plan &pl, const T *x, T *f, hipStream_t s) {
    const int n = (int)pl.f_count, J = (int)pl.fast.J, aligned = (reinterpret_cast<uintptr_t>(f) & 15) == 0;
    const dim3 grid((unsigned)((n + 256ll * (16 / (int)sizeof(T)) - 1) / (256 * (16 / (int)sizeof(T)))));
    if (pl.pattern_wide == TAD_FAMILY_ANTIDIAGONAL)
        TAD_UNARY_SWITCH(pl.expr.body, TAD_LAUNCH("k_pattern_wide_forward", (k_pattern_wide_forward<B_, T, true>), grid, dim3(256), 0, s, x, f, n, J, aligned))
    else
        TAD_UNARY_SWITCH(pl.expr.body, TAD_LAUNCH("k_pattern_wide_forward", (k_pattern_wide_forward<B_, T, false>), grid, dim3(256), 0, s, x, f, n, J, aligned))
    return hipGetLastError() == hipSuccess ? TAD_OK : TAD_EDEVICE;
}

template <typename T>
static int backward_t(const tad_plan &pl, const T *x, const T *df, T *dx, void *ws, hipStream_t s) {
    const int I = (int)pl.fast.I, J = (int)pl.fast.J, n_x = (int)pl.arg_count[0];
    if (pl.pattern_wide == TAD_FAMILY_ROW_REDUCE) {
        // a row long enough for four wavefronts, or too few rows for one each
        if (J >= 4096 || (J >= 512 && n_x < 2048))
            TAD_UNARY_SWITCH(pl.expr.body, TAD_LAUNCH("k_rowreduce_wide_backward", (k_rowreduce_wide_backward<B_, T, 4>), dim3(n_x), dim3(256), 0, s,
                                                      pl.fast.feas, x, df, dx, n_x, J))
        else
            TAD_UNARY_SWITCH(pl.expr.body, TAD_LAUNCH("k_rowreduce_wide_backward", (k_rowreduce_wide_backward<B_, T, 1>), dim3((n_x + 3) / 4), dim3(256),
                                                      0, s, pl.fast.feas, x, df, dx, n_x, J))
        return hipGetLastError() == hipSuccess ? TAD_OK : TAD_EDEVICE;
    }
    const int rows = antidiag_wide_rows(I, J), chunks = (I + rows - 1) / rows, tiles = (J + rows + 255) / 256;
    double *const part = static_cast<double *>(ws);
    TAD_LAUNCH("k_antidiag_wide_backward", (k_antidiag_wide_backward<T>), dim3((unsigned)tiles * (unsigned)chunks), dim3(256), 0, s, df, part, I, J,
               rows, tiles);
    if (hipGetLastError() != hipSuccess) return TAD_EDEVICE;
    TAD_UNARY_SWITCH(pl.expr.body, TAD_LAUNCH("k_antidiag_wide_finish", (k_antidiag_wide_finish<B_, T>), dim3((n_x + 63) / 64), dim3(256), 0, s,
                                              pl.fast.feas, pl.fast.flat[0], pl.fast.dd_iy, pl.fast.dd_iz, x, (const double *)part, dx, n_x, J, rows))
    return hipGetLastError() == hipSuccess ? TAD_OK : TAD_EDEVICE;
}

int pattern_wide_forward(const tad_plan &pl, const void *const *args, void *f, hipStream_t s) {
    return pl.dtype == TAD_F64 ? forward_t(pl, (const double *)args[0], (double *)f, s) : forward_t(pl, (const float *)args[0], (float *)f, s);
}

int pattern_wide_backward(const tad_plan &pl, const void *const *args, const void *df, void *const *dx, void *ws, hipStream_t s) {
    if (!dx[0]) return TAD_OK;
    return pl.dtype == TAD_F64 ? backward_t(pl, (const double *)args[0], (const double *)df, (double *)dx[0], ws, s)
                               : backward_t(pl, (const float *)args[0], (const float *)df, (float *)dx[0], ws, s);
}

}  // namespace tad
