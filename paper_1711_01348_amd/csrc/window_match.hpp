// Recognition of sums over a moving window (window.hpp).  Host only; included by families.cpp.
#pragma once
#include <algorithm>

#include "plan.hpp"
#include "window.hpp"

namespace tad {

void match_window(tad_plan &pl) {
    WindowPlan p;
    const tad_expr &e = pl.expr;
    if (e.body != TAD_BODY_MUL || pl.fwd_family != TAD_FAMILY_GENERIC || pl.has_alias || e.n_f != 1 || e.n_sum != 1 || e.sum_lo[0] != 0) return;
    for (const ArgPlan &ap : pl.ap)
        if (ap.derived && ap.family != TAD_FAMILY_GENERIC) return;
    auto row_is = [](const tad_arg &a, int64_t i, int64_t k) { return a.rank == 1 && a.index[0][0] == i && a.index[0][1] == k; };
    p.w = row_is(pl.args[1], 0, 1) ? 1 : 0;
    p.x = 1 - p.w;
    if (!row_is(pl.args[p.w], 0, 1)) return;
    p.q = row_is(pl.args[p.x], 1, 1) ? 1 : -1;
    if (!row_is(pl.args[p.x], 1, p.q)) return;
    // conditions may keep every term away from the end of the window, and w may then end before it: the terms are those of a window as long as w
    const int64_t N = e.f_shape[0], K = std::min(e.sum_hi[0] + 1, pl.arg_count[p.w]);
    if (N < 1 || K < 1 || N > kWindowResults || K > kWindowSum || pl.arg_count[p.x] > 2 * kWindowResults || pl.arg_count[p.w] > kWindowResults) return;
    int64_t first = p.q > 0 ? 0 : 1 - K, last = p.q > 0 ? N + K - 2 : N - 1;
    for (int c = 0; c < e.n_constraints; ++c) {   // s (i + q k) + c0 >= 0 with s = 1 or -1: a limit of the element of x
        const int64_t s = e.constraint[c][0], c0 = e.constraint[c][2];
        if ((s != 1 && s != -1) || e.constraint[c][1] != s * p.q || c0 > kWindowResults * 4 || c0 < -kWindowResults * 4) return;
        if (s > 0) first = std::max(first, -c0);
        else last = std::min(last, c0);
    }
    if (first < 0 || last >= pl.arg_count[p.x] || first > last) return;
    p.N = (int)N; p.K = (int)K;
    p.first = (int)first; p.last = (int)last;
    p.n_x = (int)pl.arg_count[p.x]; p.n_w = (int)pl.arg_count[p.w];
    // 256 results per workgroup as long as that is no more than a dozen workgroups per compute unit: their sums of dw are added by the second
    // launch.  Gradients with 256 / 1024: 131072 x 33 11.1 / 16.6 us, 262144 x 128 18.7 / 40.8, x 16 11.2 / 11.3, 522153 x 40 18.7 / 22.2, 670816 x 40
    // 23.2 / 26.2; 817544 x 3 20.3 / 13.1, 1048576 x 8 19.7 / 12.8, x 33 25.2 / 21.6.
    p.rows = N > (K < 24 ? 400000 : 750000) ? 4 : 1;
    p.ws_bytes = align256((size_t)K * (size_t)((N + 256 * p.rows - 1) / (256 * p.rows)) * sizeof(double));
    p.on = true;
    pl.window = p;
    pl.ws_full = std::max(pl.ws_full, p.ws_bytes);
}

}  // namespace tad
