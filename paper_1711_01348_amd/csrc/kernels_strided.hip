// Specialised fp32 kernels for a strided (non-unimodular looking) index map,
//
//     f_nij = tanh( sum_{u<U, v<V} x_{n, s i + u, s j + v} w_uv ),
//
// extended index (n, i, j, u, v).  With t_nij = df_nij (1 - f_nij^2):
//     dx_npq = sum over the plan's two kernel coordinates of t * w      (at most ceil(U/s) ceil(V/s) terms; the ranges, rational
//              bounds rounded exactly and clipped at the border, are the i, j with p - s i and q - s j among the taps)
//     dw_uv  = sum_{n,i,j} t_nij x_{n, s i + u, s j + v}                  (all three kernel coordinates collapse:
//              block-level reduction to per-block partials, finished in fixed order)
//
// Gradients of 32 x 128 x 128, 3 x 3, stride 2 (21 MB in the caches, bound by latency): wavefronts that evaluated the plan's range rows beside
// others for dw 19.0 us; one pass over pairs (i, j) for both 12.0; dx by pairs and dw in workgroups of their own 10.0.  Forward and gradients of 8 x 33 x 61,
// 7 x 7, stride 1: 89 / 22 / 18 us.  The pass for both was slower where a filter has many taps or the stride is large: dw of 32 x 128 x 128, 7 x 7, stride 1
// 16.8 / 20.7 / 16.1 us, both of 64 x 64 x 64, 7 x 7, stride 4 26.5 / 30.2 / 19.0, 3 x 3, stride 9 56 / 126 / 34, 256 x 14 x 14, 3 x 3, stride 16 39 / 64 / 21.
#include <hip/hip_runtime.h>

#include <algorithm>

#include "launch.h"
#include "plan_dev.h"
#include "profile.h"
#include "launch_geom.h"

namespace tad {

constexpr int kMaxTaps = 49;   // U*V <= 7*7

struct StridedGeom {
    int N, I, J, U, V, s, P, Q;   // x is N x P x Q
};

struct StridedRows {   // rows of `width` elements over 256 threads
    int width, magic, step_row, step_col;
    int hu, hv;        // gradients: rows and columns of t in front of a pair's own that its taps read
};

template <int CTRL, int ROW_MASK>
__device__ __forceinline__ float dpp_add_s(float v) {
    int t = __builtin_amdgcn_update_dpp(0, __float_as_int(v), CTRL, ROW_MASK, 0xf, ROW_MASK == 0xf);
    return v + __int_as_float(t);
}
__device__ __forceinline__ float wave_sum63s(float v) {
    v = dpp_add_s<0x111, 0xf>(v);
    v = dpp_add_s<0x112, 0xf>(v);
    v = dpp_add_s<0x114, 0xf>(v);
    v = dpp_add_s<0x118, 0xf>(v);
    v = dpp_add_s<0x142, 0xa>(v);
    v = dpp_add_s<0x143, 0xc>(v);
    return v;
}

__global__ __launch_bounds__(256) void k_strided_forward_direct(const StridedGeom g, const float *__restrict__ x,
                                                         const float *__restrict__ w, float *__restrict__ f,
                                                         int nf) {
    __shared__ float ws[kMaxTaps];
    if (threadIdx.x < g.U * g.V) ws[threadIdx.x] = w[threadIdx.x];
    __syncthreads();
    const int lin = blockIdx.x * 256 + threadIdx.x;
    if (lin >= nf) return;
    const int j = lin % g.J, i = (lin / g.J) % g.I, n = lin / (g.J * g.I);
    const float *xp = x + ((size_t)n * g.P + (size_t)g.s * i) * g.Q + (size_t)g.s * j;
    float acc = 0.f;
    for (int u = 0; u < g.U; ++u)
        for (int v = 0; v < g.V; ++v) acc = fmaf(xp[(size_t)u * g.Q + v], ws[u * g.V + v], acc);
    f[lin] = tanhf(acc);
}

// ------------------------------------------------------------------------------------------------
// Tiled kernels.  The index maps of this family make whole-row pieces of the tensors contiguous: the rows of x that
// a few rows i of f read, and the rows of f that the gradient of a few rows p of x sums over.  A block stages such a
// slice in LDS once, with 16-byte loads, and every term is then an LDS read.
//
// These kernels run a few microseconds, in which a wavefront mostly waits: for the one round of loads, for LDS, and for
// instructions that are new to its compute unit.  Everything that repeats is a loop that is not unrolled, and nothing is
// specialised that a loop bound can express.
// ------------------------------------------------------------------------------------------------

typedef float float4s __attribute__((ext_vector_type(4)));
typedef float float4a __attribute__((ext_vector_type(4), aligned(4)));   // 16 bytes from any element on

// Floats [first, first + count) of a tensor -> lds[0 ..], by 256 threads: four vectors per thread in flight.  The loads are unconditional
// (a load under a condition is waited for before the next one goes out) from wherever the slice starts.
__device__ __forceinline__ void slice_to_lds(const float *__restrict__ base, int first, int count, float *lds, int tid) {
    const float *p = base + first;
    const int nvec = count >> 2;
TAD_NOUNROLL
    for (int v0 = tid; v0 < nvec; v0 += 4 * 256) {
        float4a val[4];
#pragma unroll
        for (int h = 0; h < 4; ++h) val[h] = *reinterpret_cast<const float4a *>(p + 4 * min(v0 + h * 256, nvec - 1));
#pragma unroll
        for (int h = 0; h < 4; ++h)
            if (v0 + h * 256 < nvec) *reinterpret_cast<float4s *>(lds + 4 * (v0 + h * 256)) = val[h];
    }
    const int rest = 4 * nvec + tid;
    if (rest < count) lds[rest] = p[rest];
}

// A workgroup's elements are numbered row by row, `width` to a row; thread tid owns tid, tid + 256, ...: their rows and
// columns without a division each.
struct RowWalk {
    int row, col, width, step_row, step_col;
    __device__ __forceinline__ RowWalk(int tid, const StridedRows &w) : width(w.width), step_row(w.step_row), step_col(w.step_col) {
        row = (int)(((unsigned)tid * w.magic) >> 16);
        col = tid - row * width;
    }
    __device__ __forceinline__ void next() {
        row += step_row;
        col += step_col;
        if (col >= width) { col -= width; ++row; }
    }
};

// forward: block = `ti` rows i of one n; the rows s*i0 .. s*(i0+rows-1)+U-1 of x[n] are one contiguous slice.  A thread carries
// its E results through the taps together, so that it waits for LDS once per tap (32 x 128 x 128: 6.8 -> 5.1 us).
template <int E>
__global__ __launch_bounds__(256) void k_strided_forward(const StridedGeom g, const StridedRows W, int ti, const float *__restrict__ x,
                                                         const float *__restrict__ w, float *__restrict__ f) {
    extern __shared__ float4s dyn4[];
    float *xs = reinterpret_cast<float *>(dyn4);
    __shared__ float ws[kMaxTaps];
    const int tid = threadIdx.x;
    const int n = blockIdx.y, i0 = blockIdx.x * ti;
    const int rows = min(ti, g.I - i0);
    if (tid < g.U * g.V) ws[tid] = w[tid];
    slice_to_lds(x, (n * g.P + g.s * i0) * g.Q, (g.s * (rows - 1) + g.U) * g.Q, xs, tid);
    RowWalk at(tid, W);
    const int ne = rows * g.J;
    int xo[E];
    float acc[E];
#pragma unroll
    for (int k = 0; k < E; ++k) {
        xo[k] = tid + 256 * k < ne ? g.s * (at.row * g.Q + at.col) : 0;
        acc[k] = 0.f;
        at.next();
    }
    __syncthreads();
    const float *wp = ws;
TAD_NOUNROLL
    for (int u = 0; u < g.U; ++u) {
        const float *xp = xs + u * g.Q;
TAD_NOUNROLL
        for (int v = 0; v < g.V; ++v, ++xp, ++wp) {
            const float wv = *wp;
#pragma unroll
            for (int k = 0; k < E; ++k) acc[k] = fmaf(xp[xo[k]], wv, acc[k]);
        }
    }
    float *out = f + ((size_t)n * g.I + i0) * g.J;
#pragma unroll
    for (int k = 0; k < E; ++k)
        if (tid + 256 * k < ne) out[tid + 256 * k] = tanhf(acc[k]);
}

// The gradients: one launch in which some workgroups sum dw and the others write dx (the few that sum come first: they run longest).
struct StridedBackward {
    StridedGeom g;
    const float *x, *w, *f, *df;
    float *dx, *part;
    int blocks_dw, dw_ti;          // workgroups of dw, and their rows i (0: elements of f in memory order)
    int n_i;                       // steps of the stride along p
    unsigned n_dx;                 // by columns: threads
    StridedRows W;                 // by pairs
    int ti, blocks;                // ... steps of a workgroup, workgroups per n
};

// dw over a few function elements into part[blk][taps]: every tap has its sum in a register, and all are added over the wavefront at the end.
// dw_ti > 0: that many rows i of one n, up to kStridedMaxPerThread elements per thread, the slice of x in LDS; else kStridedDwElems elements, x
// from memory.
template <int TAPS>
__device__ __forceinline__ void strided_dw(const StridedBackward &A, int blk, float *xs) {
    __shared__ float red[4][TAPS];
    __shared__ int tapoff[TAPS];
    constexpr int E = kStridedMaxPerThread;
    static_assert(E * 256 == kStridedDwElems, "elements of a thread");
    const StridedGeom &g = A.g;
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, taps = g.U * g.V;
    if (tid < taps) tapoff[tid] = (tid / g.V) * g.Q + (tid % g.V);
    float acc[TAPS];
#pragma unroll
    for (int q = 0; q < TAPS; ++q) acc[q] = 0.f;
    if (A.dw_ti > 0) {
        const int n_it = (g.I + A.dw_ti - 1) / A.dw_ti, n = blk / n_it, i0 = (blk % n_it) * A.dw_ti, rows = min(A.dw_ti, g.I - i0), ne = rows * g.J;
        const size_t first = ((size_t)n * g.I + i0) * g.J;
        float fv[E], dv[E];
#pragma unroll
        for (int k = 0; k < E; ++k) {
            const int e = min(tid + 256 * k, ne - 1);
            fv[k] = A.f[first + e];
            dv[k] = A.df[first + e];
        }
        slice_to_lds(A.x, (n * g.P + g.s * i0) * g.Q, (g.s * (rows - 1) + g.U) * g.Q, xs, tid);
        __syncthreads();
        int il = 0, j = tid;
#pragma unroll
        for (int k = 0; k < E; ++k) {
            if (tid + 256 * k < ne) {
                while (j >= g.J) { j -= g.J; ++il; }
                const float t = dv[k] * (1.f - fv[k] * fv[k]), *xp = xs + g.s * (il * g.Q + j);
#pragma unroll
                for (int q = 0; q < TAPS; ++q)
                    if (q < taps) acc[q] = fmaf(t, xp[tapoff[q]], acc[q]);
                j += 256;
            }
        }
    } else {
        __syncthreads();
        const int nf = g.N * g.I * g.J;
#pragma unroll
        for (int k = 0; k < E; ++k) {
            const int lin = blk * kStridedDwElems + k * 256 + tid;
            if (lin < nf) {
                const int j = lin % g.J, i = (lin / g.J) % g.I, n = lin / (g.J * g.I);
                const float fv = A.f[lin], t = A.df[lin] * (1.f - fv * fv);
                const float *xp = A.x + ((size_t)n * g.P + (size_t)g.s * i) * g.Q + (size_t)g.s * j;
#pragma unroll
                for (int q = 0; q < TAPS; ++q)
                    if (q < taps) acc[q] = fmaf(t, xp[tapoff[q]], acc[q]);
            }
        }
    }
#pragma unroll
    for (int q = 0; q < TAPS; ++q) {
        const float sum = wave_sum63s(acc[q]);
        if (lane == 63) red[wave][q] = sum;
    }
    __syncthreads();
    if (tid < taps) A.part[(size_t)blk * taps + tid] = (float)(((double)red[0][tid] + (double)red[1][tid]) + ((double)red[2][tid] + (double)red[3][tid]));
}

// dx by columns: a thread per (n, i, q) writes the elements (s i + a, q), a < s, so that a wavefront stores 64 neighbouring columns.  Their taps
// are u = a + s u', v = q % s + s v' with t_{i - u', j - v'}, j = q / s.  NEAR: u' and v' are at most 1, the four t are read once for all a.
template <bool NEAR>
__device__ __forceinline__ void strided_dx_columns(const StridedBackward &A, unsigned e, const float *ws) {
    const StridedGeom &g = A.g;
    if (e >= A.n_dx) return;
    const int q = (int)(e % (unsigned)g.Q), r = (int)(e / (unsigned)g.Q), taps = g.U * g.V;
    const int i = r % A.n_i, n = r / A.n_i, j = q / g.s, b = q - j * g.s;
    const int p0 = g.s * i, rows = min(g.s, g.P - p0);
    const float *f = A.f + (size_t)n * g.I * g.J, *df = A.df + (size_t)n * g.I * g.J;
    float *out = A.dx + ((size_t)n * g.P + p0) * g.Q + q;
    if constexpr (NEAR) {
        float t[2][2];
        bool on[2][2];
#pragma unroll
        for (int y = 0; y < 2; ++y)
#pragma unroll
            for (int z = 0; z < 2; ++z) {
                const int ii = i - y, jj = j - z;
                on[y][z] = (unsigned)ii < (unsigned)g.I && (unsigned)jj < (unsigned)g.J && b + z * g.s < g.V && y * g.s < g.U;
                const int o = on[y][z] ? ii * g.J + jj : 0;
                const float fv = f[o], dv = df[o];
                t[y][z] = dv * (1.f - fv * fv);
            }
TAD_NOUNROLL
        for (int a = 0; a < rows; ++a, out += g.Q) {
            float acc = 0.f;
#pragma unroll
            for (int y = 0; y < 2; ++y) {
                const int u = a + y * g.s;   // the same for the whole workgroup
                if (u >= g.U) break;
#pragma unroll
                for (int z = 0; z < 2; ++z) acc = on[y][z] ? fmaf(t[y][z], ws[min(u * g.V + b + z * g.s, taps - 1)], acc) : acc;
            }
            *out = acc;
        }
    } else {
        // the terms of a thread in one loop, several of whose loads go out together
        const int n_v = b < g.V ? min((g.V - 1 - b) / g.s, j) + 1 : 0, v_skip = max(j - (g.J - 1), 0);   // v' from v_skip to n_v - 1
TAD_NOUNROLL
        for (int a = 0; a < rows; ++a, out += g.Q) {
            const int n_u = a < g.U ? min((g.U - 1 - a) / g.s, i) + 1 : 0, u_skip = max(i - (g.I - 1), 0);
            const int width = max(n_v - v_skip, 0), terms = width * max(n_u - u_skip, 0);
            float acc = 0.f;
            int o = (i - u_skip) * g.J + j - v_skip, k = (a + u_skip * g.s) * g.V + b + v_skip * g.s, c = 0;
#pragma unroll 4
            for (int m = 0; m < terms; ++m) {
                const float fv = f[o];
                acc = fmaf(df[o] * (1.f - fv * fv), ws[k], acc);
                --o;
                k += g.s;
                if (++c == width) {
                    c = 0;
                    o += width - g.J;
                    k += (g.V - width) * g.s;
                }
            }
            *out = acc;
        }
    }
}

// dx by pairs: `ti` steps of the stride in p of one n.  A thread owns E pairs (i, j) and writes the s x s elements of dx at (s i, s j).  With
// u = a + s u', v = b + s v':
//     dx_{n, s i + a, s j + b} = sum_{u', v'} t_{n, i - u', j - v'} w_uv
// so that the taps (u, v) of one (a, b) serve an element of dx, every tap once.  t is 0 in LDS outside the function indices, where the terms do not
// exist.  Indices run over i < ceil(P / s), j < ceil(Q / s) (rows and columns of x behind the last term: zeros), rows of t start with the
// (V - 1) / s columns in front of j = 0, so that a term is at the same distance in LDS for every element.
template <int E>
__device__ __forceinline__ void strided_dx_pairs(const StridedBackward &A, int blk, const float *ws, float *lds) {
    // a thread without a pair (in front of j = 0) reaches hv floats in front of t
    const StridedGeom &g = A.g;
    const StridedRows &W = A.W;
    const int tid = threadIdx.x, s = g.s, width = W.width, hu = W.hu, hv = W.hv;
    const int n = blk / A.blocks, i0 = (blk - n * A.blocks) * A.ti, rows = min(A.ti, A.n_i - i0);
    float *ts = lds + hv;
    // t on rows i0 - hu .. i0 + rows - 1
    const int nt = (hu + rows) * width;
    {
        RowWalk at(tid, W);
        const int f0 = n * g.I * g.J;
TAD_NOUNROLL
        for (int m0 = tid; m0 < nt; m0 += 4 * 256) {
            float fv[4], dv[4];
            bool in[4];
#pragma unroll
            for (int k = 0; k < 4; ++k) {
                const int i = i0 - hu + at.row, j = at.col - hv;
                in[k] = (unsigned)i < (unsigned)g.I && (unsigned)j < (unsigned)g.J;
                const int o = in[k] ? f0 + i * g.J + j : f0;
                fv[k] = A.f[o];
                dv[k] = A.df[o];
                at.next();
            }
#pragma unroll
            for (int k = 0; k < 4; ++k) {
                const float t = in[k] ? dv[k] * (1.f - fv[k] * fv[k]) : 0.f;
                if (m0 + 256 * k < nt) ts[m0 + 256 * k] = t;
            }
        }
    }
    __syncthreads();
    const float *const mine = ts + tid + hu * width;   // t of pair k: mine[256 k]
    int pi[E], pj[E];
    {
        RowWalk at(tid, W);
#pragma unroll
        for (int k = 0; k < E; ++k) {
            const int j = at.col - hv;
            pi[k] = at.row < rows && j >= 0 ? i0 + at.row : A.n_i;   // no element of dx has a row from s n_i on
            pj[k] = j;
            at.next();
        }
    }
    float *const out = A.dx + (size_t)n * g.P * g.Q;
    int a = 0, b = 0;
TAD_NOUNROLL
    for (;;) {
        float acc[E];
#pragma unroll
        for (int k = 0; k < E; ++k) acc[k] = 0.f;
        const float *t_row = mine;
        int du = 0;
TAD_NOUNROLL
        for (int u = a; u < g.U; u += s, t_row -= width, ++du) {
            const float *tp = t_row, *wp = ws + u * g.V + b;
            int dv = 0;
TAD_NOUNROLL
            for (int v = b; v < g.V; v += s, --tp, wp += s, ++dv) {
                const float wv = __int_as_float(__builtin_amdgcn_readfirstlane(__float_as_int(*wp)));
                float tv[E];
#pragma unroll
                for (int k = 0; k < E; ++k) tv[k] = tp[256 * k];
                if (__builtin_isfinite(wv)) {
#pragma unroll
                    for (int k = 0; k < E; ++k) acc[k] = fmaf(tv[k], wv, acc[k]);
                } else {   // a term that does not exist is left out, not multiplied by zero
#pragma unroll
                    for (int k = 0; k < E; ++k)
                        if ((unsigned)(pi[k] - du) < (unsigned)g.I && (unsigned)(pj[k] - dv) < (unsigned)g.J) acc[k] = fmaf(tv[k], wv, acc[k]);
                }
            }
        }
#pragma unroll
        for (int k = 0; k < E; ++k) {
            const int p = s * pi[k] + a, q = s * pj[k] + b;
            if (p < g.P && q < g.Q) out[p * g.Q + q] = acc[k];
        }
        if (++b < s) continue;
        b = 0;
        if (++a == s) break;
    }
}

// E: pairs per thread, or 0 by columns, -1 by columns that are NEAR
template <int TAPS, int E>
__global__ __launch_bounds__(256) void k_strided_backward(const StridedBackward A) {
    extern __shared__ float4s dyn4[];
    float *const lds = reinterpret_cast<float *>(dyn4);
    if ((int)blockIdx.x < A.blocks_dw) {
        strided_dw<TAPS>(A, (int)blockIdx.x, lds);
        return;
    }
    __shared__ float ws[kMaxTaps];
    if (threadIdx.x < A.g.U * A.g.V) ws[threadIdx.x] = A.w[threadIdx.x];
    const unsigned blk = blockIdx.x - (unsigned)A.blocks_dw;
    if constexpr (E > 0) {
        strided_dx_pairs<E>(A, (int)blk, ws, lds);
    } else {
        __syncthreads();
        strided_dx_columns<E != 0>(A, blk * 256u + threadIdx.x, ws);
    }
}

// dw_q = sum over the per-block partials, fixed order; one block of four waves per tap
__global__ __launch_bounds__(256) void k_strided_finish(const float *__restrict__ part, int n_part, int taps,
                                                        float *__restrict__ dw) {
    __shared__ double red[4];
    const int q = blockIdx.x, lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    double s = 0.0;
    for (int b = threadIdx.x; b < n_part; b += 256) s += (double)part[(size_t)b * taps + q];
    for (int m = 32; m >= 1; m >>= 1) s += __shfl_xor(s, m, 64);
    if (lane == 0) red[wave] = s;
    __syncthreads();
    if (threadIdx.x == 0) dw[q] = (float)((red[0] + red[1]) + (red[2] + red[3]));
}

static StridedGeom geom(const tad_plan &pl) {
    StridedGeom g;
    g.N = (int)pl.fast.N; g.I = (int)pl.fast.I; g.J = (int)pl.fast.J; g.U = (int)pl.fast.U; g.V = (int)pl.fast.V;
    g.s = (int)pl.fast.stride; g.P = (int)pl.fast.P; g.Q = (int)pl.fast.Q;
    return g;
}

// (tid * magic) >> 16 is tid / width for tid < 256: the error of magic, below width,
// times tid stays below 2^16 for width <= 256, and beyond that the quotient is 0.
static StridedRows row_walk(int width, int hu, int hv) {
    return {width, (65536 + width - 1) / width, 256 / width, 256 % width, hu, hv};
}

int strided_forward(const tad_plan &pl, const void *const *args, void *f, hipStream_t s) {
    const int nf = (int)pl.f_count;
    const StridedTiling t = strided_tiling(pl.fast.N, pl.fast.I, pl.fast.J, pl.fast.U, pl.fast.stride, pl.fast.Q);
    const float *x = (const float *)args[0], *w = (const float *)args[1];
    if (t.ti && pl.fast.N <= 65535) {   // N along the second axis of the grid
        const dim3 grid((unsigned)((pl.fast.I + t.ti - 1) / t.ti), (unsigned)pl.fast.N), block(256);
        const size_t lds = (size_t)t.x_slice * 4;
        const StridedRows rows = row_walk((int)pl.fast.J, 0, 0);
        const int64_t each = (t.ti * pl.fast.J + 255) / 256;
        if (each <= 1) TAD_LAUNCH("k_strided_forward", (k_strided_forward<1>), grid, block, lds, s, geom(pl), rows, t.ti, x, w, (float *)f);
        else if (each <= 2) TAD_LAUNCH("k_strided_forward", (k_strided_forward<2>), grid, block, lds, s, geom(pl), rows, t.ti, x, w, (float *)f);
        else TAD_LAUNCH("k_strided_forward", (k_strided_forward<4>), grid, block, lds, s, geom(pl), rows, t.ti, x, w, (float *)f);
    } else {
        TAD_LAUNCH("k_strided_forward_direct", k_strided_forward_direct, dim3((nf + 255) / 256), dim3(256), 0, s, geom(pl), x, w, (float *)f, nf);
    }
    return hipGetLastError() == hipSuccess ? TAD_OK : TAD_EDEVICE;
}

template <int TAPS>
static void launch_backward(const StridedBackward &A, int each, unsigned blocks, size_t lds, hipStream_t s) {
    const dim3 grid(blocks), block(256);
#define TAD_STRIDED_BACKWARD(E) TAD_LAUNCH("k_strided_backward", (k_strided_backward<TAPS, E>), grid, block, lds, s, A)
    switch (each) {
    case 1: TAD_STRIDED_BACKWARD(1); break;
    case 2: TAD_STRIDED_BACKWARD(2); break;
    case 4: TAD_STRIDED_BACKWARD(4); break;
    case 8: TAD_STRIDED_BACKWARD(8); break;
    case 0: TAD_STRIDED_BACKWARD(0); break;
    default: TAD_STRIDED_BACKWARD(-1);
    }
#undef TAD_STRIDED_BACKWARD
}

#define TAD_TAPS_SWITCH(taps, CALL)                                   \
    do {                                                              \
        if (taps <= 4) { constexpr int T_ = 4; CALL; }                \
        else if (taps <= 9) { constexpr int T_ = 9; CALL; }           \
        else if (taps <= 16) { constexpr int T_ = 16; CALL; }         \
        else if (taps <= 25) { constexpr int T_ = 25; CALL; }         \
        else { constexpr int T_ = kMaxTaps; CALL; }                   \
    } while (0)

int strided_backward(const tad_plan &pl, const void *const *args, const void *f, const void *df,
                     void *const *dx, void *ws, hipStream_t s) {
    if (!dx[0] && !dx[1]) return TAD_OK;
    StridedBackward A{};
    A.g = geom(pl);
    A.x = (const float *)args[0]; A.w = (const float *)args[1]; A.f = (const float *)f; A.df = (const float *)df;
    A.dx = (float *)dx[0]; A.part = (float *)ws;
    const StridedGeom &g = A.g;
    const int taps = g.U * g.V;
    size_t lds = 0;
    if (dx[1]) {
        const StridedTiling t = strided_dw_tiling(g.N, g.I, g.J, g.U, g.V, g.s, g.P, g.Q);
        A.dw_ti = t.ti;
        A.blocks_dw = (int)(t.ti ? (int64_t)g.N * ((g.I + t.ti - 1) / t.ti) : (pl.f_count + kStridedDwElems - 1) / kStridedDwElems);
        lds = (size_t)t.x_slice * 4;
    }
    A.n_i = (g.P + g.s - 1) / g.s;
    int each = 0;
    unsigned blocks_dx = 0;
    if (dx[0]) {
        const StridedPairs t = strided_pairs(g.N, g.U, g.V, g.s, g.P, g.Q);
        each = t.each;
        if (each) {
            A.W = row_walk(t.width, t.hu, t.hv);
            A.ti = t.ti;
            A.blocks = t.blocks;
            blocks_dx = (unsigned)(t.blocks * g.N);
            lds = std::max(lds, (size_t)t.t_floats * 4);
        } else {
            A.n_dx = (unsigned)g.N * A.n_i * g.Q;
            blocks_dx = (A.n_dx + 255) / 256;
            if ((g.U - 1) / g.s <= 1 && (g.V - 1) / g.s <= 1) each = -1;
        }
    }
    TAD_TAPS_SWITCH(taps, (launch_backward<T_>(A, each, (unsigned)A.blocks_dw + blocks_dx, lds, s)));
    if (hipGetLastError() != hipSuccess) return TAD_EDEVICE;
    if (dx[1]) {
        TAD_LAUNCH("k_strided_finish", k_strided_finish, dim3(taps), dim3(256), 0, s, (const float *)ws, A.blocks_dw,
                   taps, (float *)dx[1]);
        if (hipGetLastError() != hipSuccess) return TAD_EDEVICE;
    }
    return TAD_OK;
}

}  // namespace tad
