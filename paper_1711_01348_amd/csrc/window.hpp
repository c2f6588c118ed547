// Sums over a window that moves with a single function index,
//
//     f_i = sum_k x_{i + q k} w_k,   q = 1 or -1,   0 <= i < N, 0 <= k < K,   over the k with  first <= i + q k <= last
//
// (correlations and causal or truncated convolutions).  Both gradients are sums of the same kind:
// dx_m = sum_k df_{m - q k} w_k for first <= m <= last, else 0, and dw_k = sum_i df_i x_{i + q k}.
#pragma once
#include <cstddef>
#include <cstdint>

struct tad_plan;

namespace tad {

struct WindowPlan {
    bool on = false;
    int x = 0, w = 0;              // operands
    int N = 0, K = 0, q = 1;
    int first = 0, last = -1;      // elements of x that terms read
    int n_x = 0, n_w = 0;          // elements of the tensors
    int rows = 1;                  // 256 `rows` results per workgroup
    size_t ws_bytes = 0;           // partial sums of dw
};

// Longest window and most results these kernels take: a window is held in LDS with the results' inputs, the partial sums of dw
// are one per window element and workgroup.
constexpr int64_t kWindowSum = 256, kWindowResults = (int64_t)1 << 24;

// Is the expression such a sum (plan.window)?
void match_window(tad_plan &plan);

}  // namespace tad
