// Specialised fp32 kernels for a strided (non-unimodular looking) index map,
//
//     f_nij = tanh( sum_{u<U, v<V} x_{n, s i + u, s j + v} w_uv ),
//
// extended index (n, i, j, u, v).  With t_nij = df_nij (1 - f_nij^2):
//     dx_npq = sum over the plan's two kernel coordinates of t * w      (at most ceil(U/s) ceil(V/s) terms; the ranges, rational
//              bounds rounded exactly and clipped at the border, are the i, j with p - s i and q - s j among the taps)
//     dw_uv  = sum_{n,i,j} t_nij x_{n, s i + u, s j + v}                  (all three kernel coordinates collapse:
//              block-level reduction to per-block partials, finished in fixed order)
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
    int n_i, hu, hv;   // gradients: steps of the stride along p, rows and columns of t in front of a pair's own that its taps read
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

// Everything the dx role needs from the plan of x, in loop-free form (y = beta for this family).
struct StridedDx {
    FlatFeas feas;
    FlatLevel lvl[2];
    int32_t fY[3], fZ[2];   // element offset of f / df:  fY . beta + fZ . z
    int32_t wY[3], wZ[2];   // element offset of w
};

// Block roles in one launch.
//  * blocks [blocks_dw, ...): one thread per gradient element (n, p, q) of x.  Masks and both ranges come from
//    the plan (feasibility rows, rational range rows rounded exactly); the two ranges do not depend on each other.
//  * blocks [0, blocks_dw) reduce dw over kStridedDwElems function elements each into part[block][taps].
template <int TAPS>
__global__ __launch_bounds__(256) void k_strided_backward_direct(const StridedGeom g, const StridedDx D,
                                                          const float *__restrict__ x, const float *__restrict__ w,
                                                          const float *__restrict__ f, const float *__restrict__ df,
                                                          float *__restrict__ dx, float *__restrict__ part, int n_x,
                                                          int nf, int blocks_dw) {
    __shared__ float ws[kMaxTaps];
    __shared__ float red[4][TAPS];
    __shared__ int tapoff[TAPS];
    const int taps = g.U * g.V;
    // the few long-running dw blocks come first in launch order so that they overlap the dx stream
    if ((int)blockIdx.x >= blocks_dw) {
        const int lin = ((int)blockIdx.x - blocks_dw) * 256 + threadIdx.x;
        const bool inside = lin < n_x;
        const int q = lin % g.Q, t = lin / g.Q;
        const int32_t y[3] = {t / g.P, t % g.P, q};
        int32_t lo1 = 0, hi1 = -1, lo0 = 0, hi0 = -1;
        if (inside && flat_feasible(D.feas, y)) {
            flat_bounds(D.lvl[1], y, lo1, hi1);
            flat_bounds(D.lvl[0], y, lo0, hi0);
        }
        const int base_f = D.fY[0] * y[0] + D.fY[1] * y[1] + D.fY[2] * y[2];
        const int base_w = D.wY[0] * y[0] + D.wY[1] * y[1] + D.wY[2] * y[2];
        const int n1 = hi1 - lo1 + 1, n0 = hi0 - lo0 + 1;
        // Up to two values per coordinate (a stride of two or more under a 3 x 3 filter, ...): the loads of all
        // terms are issued together, before the filter taps are staged, so that the wavefront waits for memory
        // once instead of once per term.  Terms are added in the order of the loops below.
        const bool few = n1 <= 2 && n0 <= 2;
        float fv[2][2], dv[2][2];
        if (few) {
#pragma unroll
            for (int a = 0; a < 2; ++a)
#pragma unroll
                for (int b = 0; b < 2; ++b) {
                    const bool on = a < n1 && b < n0;
                    const int of = base_f + D.fZ[1] * (lo1 + a) + D.fZ[0] * (lo0 + b);
                    fv[a][b] = on ? f[of] : 0.f;
                    dv[a][b] = on ? df[of] : 0.f;
                }
        }
        if (threadIdx.x < taps) ws[threadIdx.x] = w[threadIdx.x];
        __syncthreads();
        if (!inside) return;
        float acc = 0.f;
        if (few) {
#pragma unroll
            for (int a = 0; a < 2; ++a)
#pragma unroll
                for (int b = 0; b < 2; ++b)
                    if (a < n1 && b < n0)
                        acc = fmaf(dv[a][b] * (1.f - fv[a][b] * fv[a][b]),
                                   ws[base_w + D.wZ[1] * (lo1 + a) + D.wZ[0] * (lo0 + b)], acc);
        } else {
            for (int32_t z1 = lo1; z1 <= hi1; ++z1) {
                int of = base_f + D.fZ[1] * z1 + D.fZ[0] * lo0;
                int ow = base_w + D.wZ[1] * z1 + D.wZ[0] * lo0;
                for (int32_t z0 = lo0; z0 <= hi0; ++z0) {
                    const float fval = f[of];
                    acc = fmaf(df[of] * (1.f - fval * fval), ws[ow], acc);
                    of += D.fZ[0];
                    ow += D.wZ[0];
                }
            }
        }
        dx[lin] = acc;
        return;
    }
    if (threadIdx.x < taps) tapoff[threadIdx.x] = (threadIdx.x / g.V) * g.Q + (threadIdx.x % g.V);
    __syncthreads();
    const int blk = blockIdx.x;
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    float acc[TAPS];
#pragma unroll
    for (int q = 0; q < TAPS; ++q) acc[q] = 0.f;
#pragma unroll
    for (int e = 0; e < kStridedDwElems / 256; ++e) {
        const int lin = blk * kStridedDwElems + e * 256 + threadIdx.x;
        if (lin < nf) {
            const int j = lin % g.J, i = (lin / g.J) % g.I, n = lin / (g.J * g.I);
            const float fv = f[lin];
            const float t = df[lin] * (1.f - fv * fv);
            const float *xp = x + ((size_t)n * g.P + (size_t)g.s * i) * g.Q + (size_t)g.s * j;
#pragma unroll
            for (int q = 0; q < TAPS; ++q)
                if (q < taps) acc[q] = fmaf(t, xp[tapoff[q]], acc[q]);
        }
    }
#pragma unroll
    for (int q = 0; q < TAPS; ++q) {
        const float sum = wave_sum63s(acc[q]);
        if (lane == 63) red[wave][q] = sum;
    }
    __syncthreads();
    if (threadIdx.x < taps)
        part[(size_t)blk * taps + threadIdx.x] =
            (red[0][threadIdx.x] + red[1][threadIdx.x]) + (red[2][threadIdx.x] + red[3][threadIdx.x]);
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

// Both gradients of `ti` steps of the stride in p of one n: a thread owns E pairs (i, j), reads each f_ij and df_ij once for
// everything, and writes the s x s elements of dx at (s i, s j).  With u = a + s u', v = b + s v':
//     dx_{n, s i + a, s j + b} = sum_{u', v'} t_{n, i - u', j - v'} w_uv,   dw_uv += t_nij x_{n, s i + u, s j + v}
// so that the taps (u, v) of one (a, b) serve an element of dx, every tap once.  The ranges of u', v' are the plan's (there is a
// single i for given p and u, if any); t is 0 in LDS outside the function indices, where the terms do not exist.  Indices run
// over i < ceil(P / s), j < ceil(Q / s) (rows and columns of x behind the last term: zeros), rows of t start with the
// (V - 1) / s columns in front of j = 0, so that a term is at the same distance in LDS for every element.
// Bound by latency (21 MB of traffic in the caches for 32 x 128 x 128, 3 x 3, stride 2): everything is loaded up front, a
// tap is 2 E independent LDS reads, and the code is short.  dx by wavefronts of their own that evaluated the plan's range rows, dw by
// others: 16.4 us in the trace; this kernel 10.3, of which dx alone takes 8.4 and dw alone 8.3.  Over the range (N x I x J, taps, stride;
// forward and gradients): 32 x 128 x 128, 3 x 3, 2: 24.2 -> 18.0 us; 4 x 60 x 60, 3 x 3, 1: 37.2 -> 16.9; 16 x 100 x 100, 7 x 7, 2:
// 52.7 -> 26.4; 8 x 33 x 61, 7 x 7, 1: 89.3 -> 22.1.
template <int E>
__global__ __launch_bounds__(256) void k_strided_backward(const StridedGeom g, const StridedRows W, int ti, int t_floats,
                                                          const float *__restrict__ x, const float *__restrict__ w,
                                                          const float *__restrict__ f, const float *__restrict__ df,
                                                          float *__restrict__ dx, float *__restrict__ part) {
    extern __shared__ float4s dyn4[];
    // a thread without a pair (in front of j = 0) reaches hv floats in front of t
    const int tid = threadIdx.x, s = g.s, taps = g.U * g.V, width = W.width, hu = W.hu, hv = W.hv;
    float *ts = reinterpret_cast<float *>(dyn4) + hv, *xs = reinterpret_cast<float *>(dyn4) + t_floats;
    __shared__ float ws[kMaxTaps];
    __shared__ float red[4][kMaxTaps];
    const int n = blockIdx.y, i0 = blockIdx.x * ti;
    const int rows = min(ti, W.n_i - i0), f_rows = min(rows, g.I - i0);   // f_rows <= 0: behind the last row of f
    const bool want_dw = part != nullptr;
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
                fv[k] = f[o];
                dv[k] = df[o];
                at.next();
            }
#pragma unroll
            for (int k = 0; k < 4; ++k) {
                const float t = in[k] ? dv[k] * (1.f - fv[k] * fv[k]) : 0.f;
                if (m0 + 256 * k < nt) ts[m0 + 256 * k] = t;
            }
        }
    }
    if (tid < taps) ws[tid] = w[tid];
    if (want_dw && f_rows > 0) slice_to_lds(x, (n * g.P + s * i0) * g.Q, (s * (f_rows - 1) + g.U) * g.Q, xs, tid);
    __syncthreads();
    const float *const mine = ts + tid + hu * width;   // t of pair k: mine[256 k]
    int pi[E], pj[E], xo[E];
    float t[E];
    bool live[E];
    {
        RowWalk at(tid, W);
#pragma unroll
        for (int k = 0; k < E; ++k) {
            const int j = at.col - hv;
            const bool pair = at.row < rows && j >= 0;
            live[k] = pair && at.row < f_rows && j < g.J;
            xo[k] = live[k] ? s * (at.row * g.Q + j) : 0;
            t[k] = live[k] ? mine[256 * k] : 0.f;
            pi[k] = pair ? i0 + at.row : W.n_i;        // no element of dx has a row from s n_i on
            pj[k] = j;
            at.next();
        }
    }
    float *const out = dx ? dx + (size_t)n * g.P * g.Q : nullptr;
    const int wave = tid >> 6;
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
            const float *tp = t_row, *xp = xs + u * g.Q + b, *wp = ws + u * g.V + b;
            int dv = 0;
TAD_NOUNROLL
            for (int v = b; v < g.V; v += s, --tp, xp += s, wp += s, ++dv) {
                const float wv = __int_as_float(__builtin_amdgcn_readfirstlane(__float_as_int(*wp)));
                float tv[E], xv[E];
#pragma unroll
                for (int k = 0; k < E; ++k) tv[k] = tp[256 * k];
                if (want_dw) {
#pragma unroll
                    for (int k = 0; k < E; ++k) xv[k] = xp[xo[k]];
                }
                if (__builtin_isfinite(wv)) {
#pragma unroll
                    for (int k = 0; k < E; ++k) acc[k] = fmaf(tv[k], wv, acc[k]);
                } else {   // a term that does not exist is left out, not multiplied by zero
#pragma unroll
                    for (int k = 0; k < E; ++k)
                        if ((unsigned)(pi[k] - du) < (unsigned)g.I && (unsigned)(pj[k] - dv) < (unsigned)g.J) acc[k] = fmaf(tv[k], wv, acc[k]);
                }
                if (want_dw) {
                    float sum = 0.f;
#pragma unroll
                    for (int k = 0; k < E; ++k) sum = fmaf(t[k], live[k] ? xv[k] : 0.f, sum);
                    sum = wave_sum63s(sum);
                    if ((tid & 63) == 63) red[wave][wp - ws] = sum;
                }
            }
        }
        if (out) {
#pragma unroll
            for (int k = 0; k < E; ++k) {
                const int p = s * pi[k] + a, q = s * pj[k] + b;
                if (p < g.P && q < g.Q) out[p * g.Q + q] = acc[k];
            }
        }
        if (++b < s) continue;
        b = 0;
        if (++a == s) break;
    }
    if (!want_dw) return;
    __syncthreads();
    if (tid < taps) part[(size_t)(blockIdx.y * gridDim.x + blockIdx.x) * taps + tid] = (red[0][tid] + red[1][tid]) + (red[2][tid] + red[3][tid]);
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
static StridedRows row_walk(int width, int n_i, int hu, int hv) {
    return {width, (65536 + width - 1) / width, 256 / width, 256 % width, n_i, hu, hv};
}

int strided_forward(const tad_plan &pl, const void *const *args, void *f, hipStream_t s) {
    const int nf = (int)pl.f_count;
    const StridedTiling t = strided_tiling(pl.fast.N, pl.fast.I, pl.fast.J, pl.fast.U, pl.fast.stride, pl.fast.Q);
    const float *x = (const float *)args[0], *w = (const float *)args[1];
    if (t.ti) {
        const dim3 grid((unsigned)((pl.fast.I + t.ti - 1) / t.ti), (unsigned)pl.fast.N), block(256);
        const size_t lds = (size_t)t.x_slice * 4;
        const StridedRows rows = row_walk((int)pl.fast.J, 0, 0, 0);
        const int64_t each = (t.ti * pl.fast.J + 255) / 256;
        if (each <= 1) TAD_LAUNCH("k_strided_forward", (k_strided_forward<1>), grid, block, lds, s, geom(pl), rows, t.ti, x, w, (float *)f);
        else if (each <= 2) TAD_LAUNCH("k_strided_forward", (k_strided_forward<2>), grid, block, lds, s, geom(pl), rows, t.ti, x, w, (float *)f);
        else TAD_LAUNCH("k_strided_forward", (k_strided_forward<4>), grid, block, lds, s, geom(pl), rows, t.ti, x, w, (float *)f);
    } else {
        TAD_LAUNCH("k_strided_forward_direct", k_strided_forward_direct, dim3((nf + 255) / 256), dim3(256), 0, s, geom(pl), x, w, (float *)f, nf);
    }
    return hipGetLastError() == hipSuccess ? TAD_OK : TAD_EDEVICE;
}

static StridedDx dx_plan(const tad_plan &pl) {
    StridedDx D;
    D.feas = pl.fast.feas;
    D.lvl[0] = pl.fast.flat[0];
    D.lvl[1] = pl.fast.flat[1];
    const GatherPlan &gp = pl.ap[0].dev;
    for (int c = 0; c < 3; ++c) { D.fY[c] = (int32_t)gp.offY[kSlotF][c]; D.wY[c] = (int32_t)gp.offY[1][c]; }
    for (int m = 0; m < 2; ++m) { D.fZ[m] = (int32_t)gp.offZ[kSlotF][m]; D.wZ[m] = (int32_t)gp.offZ[1][m]; }
    return D;
}

template <int TAPS>
static void launch_bwd_direct(const tad_plan &pl, const void *const *args, const void *f, const void *df,
                              void *const *dx, void *ws, int blocks_dx, int blocks_dw, hipStream_t s) {
    TAD_LAUNCH("k_strided_backward_direct", (k_strided_backward_direct<TAPS>), dim3(blocks_dx + blocks_dw), dim3(256), 0, s,
               geom(pl), dx_plan(pl), (const float *)args[0], (const float *)args[1], (const float *)f, (const float *)df,
               (float *)dx[0], (float *)ws, (int)pl.arg_count[0], (int)pl.f_count, blocks_dw);
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
    const int nf = (int)pl.f_count;
    const int taps = (int)(pl.fast.U * pl.fast.V);
    int blocks_dw = 0;
    const StridedGrad t = strided_grad(pl.fast.N, pl.fast.I, pl.fast.J, pl.fast.U, pl.fast.V, pl.fast.stride, pl.fast.P, pl.fast.Q);
    if (t.ti) {
        if (!dx[0] && !dx[1]) return TAD_OK;
        blocks_dw = t.blocks * (int)pl.fast.N;
        const dim3 grid((unsigned)t.blocks, (unsigned)pl.fast.N), block(256);
        const size_t lds = (size_t)(t.t_floats + t.x_floats) * 4;
        const StridedRows rows = row_walk(t.width, t.n_i, t.hu, t.hv);
        float *const part = dx[1] ? (float *)ws : nullptr;
#define TAD_STRIDED_BACKWARD(E)                                                                                                              \
    TAD_LAUNCH("k_strided_backward", (k_strided_backward<E>), grid, block, lds, s, geom(pl), rows, t.ti, t.t_floats, (const float *)args[0], \
               (const float *)args[1], (const float *)f, (const float *)df, (float *)dx[0], part)
        if (t.each == 1) TAD_STRIDED_BACKWARD(1);
        else if (t.each == 2) TAD_STRIDED_BACKWARD(2);
        else if (t.each == 4) TAD_STRIDED_BACKWARD(4);
        else TAD_STRIDED_BACKWARD(8);
#undef TAD_STRIDED_BACKWARD
    } else {
        const int blocks_dx = dx[0] ? (int)((pl.arg_count[0] + 255) / 256) : 0;
        blocks_dw = dx[1] ? (nf + kStridedDwElems - 1) / kStridedDwElems : 0;
        if (blocks_dx + blocks_dw == 0) return TAD_OK;
        TAD_TAPS_SWITCH(taps, (launch_bwd_direct<T_>(pl, args, f, df, dx, ws, blocks_dx, blocks_dw, s)));
    }
    if (hipGetLastError() != hipSuccess) return TAD_EDEVICE;
    if (dx[1]) {
        TAD_LAUNCH("k_strided_finish", k_strided_finish, dim3(taps), dim3(256), 0, s, (const float *)ws, blocks_dw,
                   taps, (float *)dx[1]);
        if (hipGetLastError() != hipSuccess) return TAD_EDEVICE;
    }
    return TAD_OK;
}

}  // namespace tad
