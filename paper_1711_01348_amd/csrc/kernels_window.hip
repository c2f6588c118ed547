// Sums over a window that moves with one function index (window.hpp): convolutions and correlations of a signal.
//
// Bound by launches: 262144 results and a window of 33 are 1 MB per tensor and 8.7 10^6 products for each of f, dx and dw.  The
// plan-driven kernels walk the plan for every element of dx and read df from memory for every term, and share an element of dw
// among whole workgroups (f 6.7 us, both gradients 25.2 us of calls in a row).  Here a workgroup holds 256 R results' inputs in LDS, widened to
// 64 bits once; a thread owns R results 256 apart, so that its reads are free of conflicts and an element of w, the same for all of them, is
// read once per R products.  dx is the same sum over df with the window turned round.  dw: a thread takes four neighbouring window
// elements and a part of the workgroup's results, four of them at a time: 11 reads for 16 products.  The workgroups' sums of dw are added
// by a second launch in a fixed order.  262144 x 33: f 3.6 us, gradients 9.1, three launches; a pass of both through Python 12.2 us.  The workgroups at the
// ends of the signal decide what a call takes if they test every term (gradients of 169877 x 63 36 us instead of 14), and where the signal is short they are
// all there is: groups of 16 terms are taken or left as a whole where they can be (dw alone of 1100 x 256 21 -> 10 us, the plan-driven kernels 7;
// 20000 x 256 16 -> 8.1).  Many parts of dw are added in two steps: one thread per window element would add up to 256 in a row (4000000 x 1,
// both gradients 31.7 -> 25.7 us, dw alone 28 -> 21); with the second launch's sums shared by a workgroup 22.8 and 17.6 (the plan-driven kernels 117
// and 12).
// Products of 32-bit operands are exact and sums are in 64 bits, so only the result is rounded.
#include <hip/hip_runtime.h>

#include "gather_loop.h"
#include "launch.h"
#include "profile.h"
#include "window.hpp"

namespace tad {

struct WindowArgs {
    const void *x, *w, *df;
    void *f, *dx;
    double *part;          // [n_w][workgroups] sums of dw, or null
    int N, K, q, first, last, n_x;
};

constexpr int kWindowPad = 3;   // in front of and behind the elements a thread's window elements reach beyond K

// Elements from .. from + count of p on their way to LDS, 0 outside lo .. hi (not empty): all loads of a kernel go out before the first
// of their results is stored.
template <typename T, int R>
struct WindowSlice {
    static constexpr int M = R + (int)kWindowSum / 256 + 1;   // count <= 256 M
    T v[M];
    __device__ __forceinline__ void load(const T *__restrict__ p, int from, int lo, int hi) {
#pragma unroll
        for (int m = 0; m < M; ++m) v[m] = p[min(max(from + (int)threadIdx.x + 256 * m, lo), hi)];
    }
    __device__ __forceinline__ void store(int from, int count, int lo, int hi, double *to) const {
#pragma unroll
        for (int m = 0; m < M; ++m) {
            const int j = (int)threadIdx.x + 256 * m, at = from + j;
            if (j < count) to[j] = at >= lo && at <= hi ? (double)v[m] : 0.0;
        }
    }
};

// out[n] for the workgroup's n: the sum over k of in[n + dir k] w[k], in[lo .. hi] being what terms read; 0 outside first .. last.
// s[0] is in[n0] (dir = 1) or in[n0 - (K - 1)].
template <typename T, int R>
__device__ __forceinline__ void window_sums(const double *s, const double *w, int K, int dir, int n0, int lo, int hi, int first, int last, int n_out,
                                            T *__restrict__ out) {
    const int tid = threadIdx.x;
    constexpr int U = R == 1 ? 8 : 4;   // terms whose reads go out together
    double acc[R];
#pragma unroll
    for (int r = 0; r < R; ++r) acc[r] = 0.0;
    const int reach = dir * (K - 1);
    const double *at = s + tid + (dir > 0 ? 0 : K - 1);
    if (n0 + min(reach, 0) >= lo && n0 + 256 * R - 1 + max(reach, 0) <= hi) {   // the same for the whole workgroup
#pragma unroll U
        for (int k = 0; k < K; ++k, at += dir) {
            const double wk = w[k];
#pragma unroll
            for (int r = 0; r < R; ++r) acc[r] += at[256 * r] * wk;
        }
    } else {   // a term that is not part of the sum is left out, not multiplied by zero: w may hold an infinity
#pragma unroll U
        for (int k = 0; k < K; ++k, at += dir) {
            const double wk = w[k];
#pragma unroll
            for (int r = 0; r < R; ++r) {
                const int m = n0 + tid + 256 * r + dir * k;
                const double next = acc[r] + at[256 * r] * wk;
                acc[r] = m >= lo && m <= hi ? next : acc[r];
            }
        }
    }
#pragma unroll
    for (int r = 0; r < R; ++r) {
        const int n = n0 + tid + 256 * r;
        if (n < n_out) out[n] = n >= first && n <= last ? (T)acc[r] : T(0);
    }
}

template <typename T, int R>
__global__ __launch_bounds__(256) void k_window_forward(const WindowArgs A) {
    __shared__ double s[256 * R + kWindowSum], w[kWindowSum];
    const int n0 = blockIdx.x * 256 * R;
    const int x0 = n0 - (A.q > 0 ? 0 : A.K - 1);
    WindowSlice<T, 0> wv;
    WindowSlice<T, R> xv;
    wv.load(static_cast<const T *>(A.w), 0, 0, A.K - 1);
    xv.load(static_cast<const T *>(A.x), x0, A.first, A.last);
    wv.store(0, A.K, 0, A.K - 1, w);
    xv.store(x0, 256 * R + A.K - 1, A.first, A.last, s);
    __syncthreads();
    window_sums<T, R>(s, w, A.K, A.q, n0, A.first, A.last, 0, A.N - 1, A.N, static_cast<T *>(A.f));
}

// dx of the workgroup's elements of x and its part of dw, the sum over its results i
// DX = false: dw alone, without the elements of df that only dx reads
template <typename T, int R, bool DX>
__global__ __launch_bounds__(256) void k_window_backward(const WindowArgs A) {
    constexpr int C = 256 * R;
    constexpr int X = C + (int)kWindowSum + 2 * kWindowPad;
    constexpr int HALO = DX ? (int)kWindowSum : 0;
    __shared__ double d[C + HALO], x[X > 1024 ? X : 1024], w[DX ? kWindowSum : 1];
    const int n0 = blockIdx.x * C, K = A.K, q = A.q, tid = threadIdx.x;
    const int ahead = DX && q > 0 ? K - 1 : 0;               // elements of d in front of n0
    const bool part = A.part && n0 < A.N;                    // the same for the whole workgroup
    const int x0 = n0 - (q > 0 ? 0 : K - 1);                 // element of x at x[kWindowPad]
    WindowSlice<T, 0> wv;
    WindowSlice<T, DX ? R : R - 2> dv;
    WindowSlice<T, R> xv;
    if constexpr (DX) wv.load(static_cast<const T *>(A.w), 0, 0, K - 1);
    dv.load(static_cast<const T *>(A.df), n0 - ahead, 0, A.N - 1);
    xv.load(static_cast<const T *>(A.x), x0 - kWindowPad, A.first, A.last);
    if constexpr (DX) wv.store(0, K, 0, K - 1, w);
    dv.store(n0 - ahead, DX ? C + K - 1 : C, 0, A.N - 1, d);
    xv.store(x0 - kWindowPad, C + K - 1 + 2 * kWindowPad, A.first, A.last, x);
    __syncthreads();
    if constexpr (DX) window_sums<T, R>(d, w, K, -q, n0, 0, A.N - 1, A.first, A.last, A.n_x, static_cast<T *>(A.dx));
    if (!part) return;
    const int groups = (K + 3) / 4, parts = 256 / groups;
    const int g = tid % groups, mine = tid / groups;
    double acc[4] = {0.0, 0.0, 0.0, 0.0};                    // of window element 4 g + a (q > 0) or 4 g + 3 - a
    if (mine < parts) {
        const int each = (C / 4 + parts - 1) / parts * 4, begin = mine * each, end = min(C, begin + each);
        const double *dp = d + ahead, *xp = x + kWindowPad + (q > 0 ? 4 * g : K - 4 - 4 * g);
        if (n0 + C <= A.N && x0 >= A.first && x0 + C + K - 2 <= A.last) {   // the same for the whole workgroup
            for (int i = begin; i < end; i += 4) {
                double dv[4], xv[7];
#pragma unroll
                for (int u = 0; u < 4; ++u) dv[u] = dp[i + u];
#pragma unroll
                for (int u = 0; u < 7; ++u) xv[u] = xp[i + u];
#pragma unroll
                for (int u = 0; u < 4; ++u)
#pragma unroll
                    for (int a = 0; a < 4; ++a) acc[a] += dv[u] * xv[u + a];
            }
        } else {
            for (int i = begin; i < end; i += 4) {
                const int m0 = n0 + i + (q > 0 ? 4 * g : -4 * g - 3);   // element of x at xv[0]
                if (m0 + 6 < A.first || m0 > A.last || n0 + i >= A.N) continue;   // none of the 16 terms exists
                double dv[4], xv[7];
                bool in_d[4], in_x[7];
#pragma unroll
                for (int u = 0; u < 4; ++u) { dv[u] = dp[i + u]; in_d[u] = n0 + i + u < A.N; }
#pragma unroll
                for (int u = 0; u < 7; ++u) { xv[u] = xp[i + u]; in_x[u] = m0 + u >= A.first && m0 + u <= A.last; }
                if (__all(m0 >= A.first && m0 + 6 <= A.last && n0 + i + 3 < A.N)) {
#pragma unroll
                    for (int u = 0; u < 4; ++u)
#pragma unroll
                        for (int a = 0; a < 4; ++a) acc[a] += dv[u] * xv[u + a];
                    continue;
                }
#pragma unroll
                for (int u = 0; u < 4; ++u)
#pragma unroll
                    for (int a = 0; a < 4; ++a) {
                        const double next = acc[a] + dv[u] * xv[u + a];
                        acc[a] = in_d[u] && in_x[u + a] ? next : acc[a];
                    }
            }
        }
    }
    __syncthreads();
    double *const red = x;                                   // [parts][4 groups], no more than 1024
#pragma unroll
    for (int a = 0; a < 4; ++a)
        if (mine < parts) red[mine * 4 * groups + (q > 0 ? 4 * g + a : 4 * g + 3 - a)] = acc[a];
    __syncthreads();
    const int cols = 4 * groups;
    const double *sums = red;
    int rows = parts;
    if (parts > 64) {                                        // in two steps; the same for the whole workgroup
        const int chunks = 256 / cols, each = (parts + chunks - 1) / chunks, c = tid % cols, chunk = tid / cols;
        if (chunk < chunks) {
            double s = 0.0;
            const int to = min(parts, (chunk + 1) * each);
#pragma unroll 4
            for (int p = chunk * each; p < to; ++p) s += red[p * cols + c];
            d[tid] = s;                                      // (nobody reads d any more)
        }
        __syncthreads();
        sums = d;
        rows = chunks;
    }
    if (tid < K) {
        double s = 0.0;
#pragma unroll 8
        for (int p = 0; p < rows; ++p) s += sums[p * cols + tid];
        A.part[(size_t)tid * ((A.N + C - 1) / C) + blockIdx.x] = s;
    }
}

// a wavefront per element of dw, or a workgroup where there are many sums to add; those behind the window are zero
template <typename T, int WAVES>
__global__ __launch_bounds__(256) void k_window_finish(const double *__restrict__ part, int blocks, int K, int n_w, T *__restrict__ dw) {
    __shared__ double sums[4];
    const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
    const int k = WAVES > 1 ? blockIdx.x : blockIdx.x * 4 + wave;
    if (k >= n_w) return;   // the whole wavefront leaves together, the whole workgroup where it works on one element
    double mine = 0.0;
    if (k < K) {
        const double *at = part + (size_t)k * blocks;
        constexpr int U = 4, STEP = 64 * WAVES;
        for (int b = WAVES > 1 ? threadIdx.x : lane; b < blocks; b += STEP * U) {
            double v[U];
#pragma unroll
            for (int u = 0; u < U; ++u) v[u] = b + STEP * u < blocks ? at[b + STEP * u] : 0.0;
#pragma unroll
            for (int u = 0; u < U; ++u) mine += v[u];
        }
    }
    double total;
    if constexpr (WAVES > 1) total = block_sum_256(mine, sums);
    else total = wave_sum_all(mine);
    if (lane == 0 && (WAVES == 1 || wave == 0)) dw[k] = (T)total;
}

static int launched() { return hipGetLastError() == hipSuccess ? TAD_OK : TAD_EDEVICE; }

static WindowArgs window_args(const WindowPlan &p, const void *const *args) {
    WindowArgs A{};
    A.x = args[p.x]; A.w = args[p.w];
    A.N = p.N; A.K = p.K; A.q = p.q; A.first = p.first; A.last = p.last; A.n_x = p.n_x;
    return A;
}

template <typename T, int R>
static int forward_t(const WindowPlan &p, const void *const *args, void *f, hipStream_t s) {
    WindowArgs A = window_args(p, args);
    A.f = f;
    TAD_LAUNCH("k_window_forward", (k_window_forward<T, R>), dim3((p.N + 256 * R - 1) / (256 * R)), dim3(256), 0, s, A);
    return launched();
}

template <typename T, int R>
static int backward_t(const WindowPlan &p, const void *const *args, const void *df, void *const *dx, void *ws, hipStream_t s) {
    WindowArgs A = window_args(p, args);
    A.df = df;
    A.dx = dx[p.x];
    A.part = dx[p.w] ? static_cast<double *>(ws) : nullptr;
    const int C = 256 * R, blocks = (p.N + C - 1) / C, of_x = A.dx ? (p.n_x + C - 1) / C : 0;
    if (!A.dx && !A.part) return TAD_OK;
    const dim3 grid(blocks > of_x ? blocks : of_x), block(256);
    if (A.dx) TAD_LAUNCH("k_window_backward", (k_window_backward<T, R, true>), grid, block, 0, s, A);
    else TAD_LAUNCH("k_window_backward", (k_window_backward<T, R, false>), grid, block, 0, s, A);
    if (launched()) return TAD_EDEVICE;
    if (!A.part) return TAD_OK;
    // Both gradients, sums added by a wavefront / a workgroup: 262144 x 33 (1024 sums) 10.2 / 9.1 us, 300000 x 1 (1172) 8.5 / 7.8, 4000000 x 1 (3907)
    // 25.7 / 22.8; up to 256 are one round of loads for either (and a workgroup for each of many elements behind the window would only write zeros)
    if (blocks > 256 && p.n_w <= 1024)
        TAD_LAUNCH("k_window_finish", (k_window_finish<T, 4>), dim3(p.n_w), dim3(256), 0, s, (const double *)A.part, blocks, p.K, p.n_w, static_cast<T *>(dx[p.w]));
    else
        TAD_LAUNCH("k_window_finish", (k_window_finish<T, 1>), dim3((p.n_w + 3) / 4), dim3(256), 0, s, (const double *)A.part, blocks, p.K, p.n_w, static_cast<T *>(dx[p.w]));
    return launched();
}

int window_forward(const tad_plan &pl, const void *const *args, void *f, hipStream_t s) {
    const WindowPlan &p = pl.window;
    if (pl.dtype == TAD_F64) return p.rows == 1 ? forward_t<double, 1>(p, args, f, s) : forward_t<double, 4>(p, args, f, s);
    return p.rows == 1 ? forward_t<float, 1>(p, args, f, s) : forward_t<float, 4>(p, args, f, s);
}

int window_backward(const tad_plan &pl, const void *const *args, const void *df, void *const *dx, void *ws, hipStream_t s) {
    const WindowPlan &p = pl.window;
    if (pl.dtype == TAD_F64) return p.rows == 1 ? backward_t<double, 1>(p, args, df, dx, ws, s) : backward_t<double, 4>(p, args, df, dx, ws, s);
    return p.rows == 1 ? backward_t<float, 1>(p, args, df, dx, ws, s) : backward_t<float, 4>(p, args, df, dx, ws, s);
}

}  // namespace tad
