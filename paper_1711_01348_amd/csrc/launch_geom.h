// Launch geometry and workspace layout shared by the host planner and the kernels: tile sizes of the specialised
// families, sizes of their per-tile partial sums, and how the plan-driven fallback kernels share long sums.
#pragma once
#include <cstddef>
#include <cstdint>

namespace tad {

constexpr int FWD_TI = 4;       // rows per forward block (1024 columns): 40.6 us at 8192^2 against 43 / 46 us with 8 / 2 rows
constexpr int BWD_TI = 256;     // rows per backward block
constexpr int BWD_TJ = 512;     // columns per backward block
constexpr int kWorkedMaxK = 8;  // longest summed index the direct (VALU) kernels are instantiated for

inline size_t align256(size_t v) { return (v + 255) & ~(size_t)255; }

// row partials [n_jt][K+2][I], column partials [n_it][K+1][J]
inline size_t worked_workspace_bytes(int64_t I, int64_t J, int64_t K) {
    size_t n_jt = (size_t)((J + BWD_TJ - 1) / BWD_TJ), n_it = (size_t)((I + BWD_TI - 1) / BWD_TI);
    return align256(n_jt * I * (K + 2) * 4) + align256(n_it * (K + 1) * J * 4);
}

// The worked expression with 64-bit sums (kernels_worked_wide.hip).
constexpr int kWideMaxK = 16, kWideMaxRows = 128;
// columns of a lane: as many as their sums and factors fit in registers
constexpr int wide_lane_columns(int K) { return K <= 7 ? 4 : 2; }
struct WideGeom {
    int tile_rows;       // rows of a tile, a multiple of 16
    int n_jt, n_it;      // tiles along the columns and the rows
    size_t col_offset, ws_bytes;   // row sums [n_jt][K + 2][I], then column sums [n_it][K][J]
};
inline WideGeom worked_wide_geom(int64_t I, int64_t J, int64_t K) {
    WideGeom g;
    const int64_t tj = 64 * wide_lane_columns((int)K);
    g.n_jt = (int)((J + tj - 1) / tj);
    // about two workgroups per compute unit; fewer rows per tile mean more column sums in memory
    int64_t rows = (I * g.n_jt + 511) / 512;
    rows = (rows + 15) / 16 * 16;
    g.tile_rows = (int)(rows > kWideMaxRows ? kWideMaxRows : rows);
    g.n_it = (int)((I + g.tile_rows - 1) / g.tile_rows);
    g.col_offset = align256((size_t)g.n_jt * (size_t)I * (size_t)(K + 2) * 8);
    g.ws_bytes = g.col_offset + align256((size_t)g.n_it * (size_t)K * (size_t)J * 8);
    return g;
}

// long summed index (MFMA family): pieces that each of the two contractions of the gradients has room for; one may take what the other does not need
constexpr int kMfmaSplit = 8, kMfmaMostPieces = 64;
inline size_t mfma_workspace_bytes(int64_t I, int64_t J, int64_t K) {
    return align256((size_t)I * 16) + align256((size_t)J * 4) + align256((size_t)kMfmaSplit * (I + J) * K * 4) +
           align256((size_t)kMfmaSplit * (2 * I + J) * 4);
}

// Terms that go through one chain of matrix instructions where the pieces may be longer (see kernels_mfma.hip)
constexpr int mfma_chain(int terms) { return 32 * ((terms + 255) / 256 < 8 ? (terms + 255) / 256 : 8); }
// The pieces that the sums over j and over i are cut into: every piece of a tile of rows is a workgroup of its own, and its partial results are
// written and read again.
struct MfmaPieces {
    int n_j, n_i;              // pieces of the sum over j (results for rows i), of the sum over i (rows j; 0: not wanted)
    int chunk_j, chunk_i;      // terms of a piece, a multiple of 32
    bool totals;               // chains of matrix instructions end within a piece
    double time;               // us, by the model
};

// Fallback (generic and program) kernels.  The cooperative form (one block per gradient element) pays off when
// an element sums many terms: measured on the worked expression at 8192 x 8192 x 5, the gradients with 8192 and
// 40960 terms per element take 0.8 ms this way against 11 ms with one thread per element.
inline bool use_cooperative_gather(long long n_elements, double terms_total) {
    return n_elements <= (1ll << 22) && terms_total / (double)(n_elements > 0 ? n_elements : 1) >= 1024.0;
}
// One block per element leaves most of the chip idle when the gradient has few elements (a filter, a bias, a
// scalar): the terms of an element are then shared by `splits` blocks, whose fp64 partial sums go to the
// workspace and are added in ascending order by a finishing kernel.  About 1024 blocks in all, at least 2048
// terms per block, at most 256 blocks per element.
inline int cooperative_splits(long long n_elements, double terms_total) {
    if (n_elements <= 0 || n_elements >= 1024 || !use_cooperative_gather(n_elements, terms_total)) return 1;
    const long long want = (1024 + n_elements - 1) / n_elements;
    const long long most = (long long)(terms_total / (double)n_elements / 2048.0);
    long long sp = want < most ? want : most;
    if (sp > 256) sp = 256;
    return sp < 1 ? 1 : (int)sp;
}
// partial sums [n_elements][splits] (fp64), then one flag per element (0: a mask zeroes it)
inline size_t split_workspace_bytes(long long n_elements, int splits) {
    return splits > 1 ? align256((size_t)n_elements * (size_t)splits * 8) + align256((size_t)n_elements * 4) : 0;
}

constexpr int kStridedDwElems = 1024;  // function elements per dw block of the strided family, direct form (multiple of 256)

// Strided family, forward: a workgroup takes ti rows i of f and stages the slice of x they read in LDS (0: the slice does not
// fit, direct kernel).
struct StridedTiling {
    int ti;
    int x_slice;    // floats of LDS for the slice of x
};
constexpr int kStridedLdsFloats = 10240;   // 40 KiB per block: four blocks per compute unit
constexpr int kStridedMaxPerThread = 4;    // function elements per thread
inline StridedTiling strided_tiling(int64_t N, int64_t I, int64_t J, int64_t U, int64_t s, int64_t Q) {
    StridedTiling t{0, 0};
    // rows s*i0 .. s*(i0+ti-1)+U-1 of x, whole rows; prefer at least 1024 blocks
    for (int ti = 8; ti >= 1; --ti) {
        const int64_t slice = (s * (ti - 1) + U) * Q;
        if (ti * J > 256 * kStridedMaxPerThread || slice > kStridedLdsFloats) continue;
        if (t.ti == 0) { t.ti = ti; t.x_slice = (int)slice; }
        if (N * ((I + ti - 1) / ti) >= 1024) { t.ti = ti; t.x_slice = (int)slice; break; }
    }
    return t;
}
// sums of dw of as many workgroups as the direct or the tiled forward kernel has
inline int64_t strided_parts(int64_t N, int64_t I, int64_t J, int64_t U, int64_t s, int64_t Q) {
    const StridedTiling t = strided_tiling(N, I, J, U, s, Q);
    const int64_t direct = (N * I * J + kStridedDwElems - 1) / kStridedDwElems, tiled = t.ti ? N * ((I + t.ti - 1) / t.ti) : 0;
    return direct > tiled ? direct : tiled;
}
inline size_t strided_workspace_bytes(int64_t N, int64_t I, int64_t J, int64_t U, int64_t V, int64_t s, int64_t Q) {
    return align256((size_t)strided_parts(N, I, J, U, s, Q) * (size_t)(U * V) * 4);
}
// dx by pairs (i, j): a workgroup takes ti steps of the stride along p, `each` pairs per thread (each = 0: by columns).
struct StridedPairs {
    int ti, each, blocks;          // blocks: workgroups per n
    int width, hu, hv;             // pairs in a row and the columns of t in front of them; see StridedRows
    int t_floats;                  // LDS
};
inline StridedPairs strided_pairs(int64_t N, int64_t U, int64_t V, int64_t s, int64_t P, int64_t Q) {
    const int64_t hu = (U - 1) / s, hv = (V - 1) / s, width = (Q + s - 1) / s + hv, n_i = (P + s - 1) / s;
    StridedPairs best{0, 0, 0, 0, 0, 0, 0};
    // What a pair stores is s apart from its neighbour's.  Columns / pairs, dx alone, taps and stride: 64 x 64 x 64 3 x 3, 4 8.1 / 11.7 us, 7 x 7, 4
    // 9.6 / 20, 7 x 7, 5 12 / 26; small tensors: 128 x 28 x 28 3 x 3, 3 3.9 / 4.9, 5 x 5, 3 (two taps at most in a direction) 4.3 / 6.5, 7 x 7, 2 7.9 / 7.8,
    // 64 x 56 x 56 5 x 5, 2 7.4 / 6.0; large ones 32 x 128 x 128 3 x 3, 2 8.2 / 6.4, 7 x 7, 2 24 / 11, 3 x 3, 3 10.8 / 8.5.
    const bool near = hu <= 1 && hv <= 1;
    if (s > 3 || (s > 1 && N * P * Q < ((int64_t)1 << (near ? 20 : 19)))) return best;
    // many pairs per thread share the waits; but at least two workgroups per compute unit
    const int order[] = {8, 1, 2, 4};
    for (int each : order) {
        int64_t ti = 256 * each / width;
        if (ti > n_i) ti = n_i;
        const int64_t t = (hv + hu * width + 256 * each + 3) & ~(int64_t)3;
        // rows of t in front of a workgroup's own are read again by every workgroup: 8 x 256 x 200, 49 x 1 pairs 25 us, columns 13; 16 x 200 x 200, 16 x 3
        // (hu = 15, ti = 5) 11 / 18
        if (ti < 1 || t > kStridedLdsFloats || hu > 4 * ti) continue;
        const int64_t blocks = (n_i + ti - 1) / ti;
        if (best.ti == 0 || best.each == 8 || N * blocks >= 512)
            best = {(int)ti, each, (int)blocks, (int)width, (int)hu, (int)hv, (int)t};
    }
    return best;
}
// dw: rows i of f per workgroup (ti = 0: elements in memory order).  As many as its threads take in as few passes as leave no more workgroups than
// compute units work on at once: a workgroup adds up all its taps over its wavefronts, whatever it has summed before.  Few taps: half as many, the
// workgroups of dx run beside them.  dw alone, old rows (at least 1024 workgroups, threads idle) / these: 128 x 28 x 28 7 x 7 13.0 / 10.9 us, 3 x 3 7.7 / 6.9;
// both gradients 32 x 112 x 112 3 x 3 9.9 / 8.6, 32 x 128 x 128 3 x 3, 2 10.9 / 9.9 (7 x 7 with 512 workgroups 24, with 1024 19).  Columns of dx have no LDS of
// their own: half of it leaves them eight workgroups per compute unit (32 x 112 x 112 3 x 3, 4 18 us with 20 KB, 22 with 40).
inline StridedTiling strided_dw_tiling(int64_t N, int64_t I, int64_t J, int64_t U, int64_t V, int64_t s, int64_t P, int64_t Q) {
    const int64_t parts = strided_parts(N, I, J, U, s, Q), most = U * V <= 9 ? 512 : 1024;
    const int64_t room = strided_pairs(N, U, V, s, P, Q).each ? kStridedLdsFloats : kStridedLdsFloats / 2;
    StridedTiling t{0, 0};
    for (int64_t passes = 1; passes <= kStridedMaxPerThread; ++passes) {
        int64_t ti = 256 * passes / J;
        if (ti > I) ti = I;
        while (ti > 1 && (s * (ti - 1) + U) * Q > room) --ti;
        if (ti < 1) continue;
        const int64_t slice = (s * (ti - 1) + U) * Q, blocks = N * ((I + ti - 1) / ti);
        if (slice > room || blocks > parts) continue;   // (the workspace holds `parts` sums)
        t.ti = (int)ti;
        t.x_slice = (int)slice;
        if (blocks <= most) break;
    }
    return t.ti ? t : strided_tiling(N, I, J, U, s, Q);
}

// antidiagonal pattern, backward: aligned tiles of df; a tile yields AD_TILE_ROWS + AD_TILE_COLS antidiagonal sums
constexpr int AD_TILE_ROWS = 256, AD_TILE_COLS = 256, AD_TILE_SUMS = AD_TILE_ROWS + AD_TILE_COLS;
inline size_t antidiag_workspace_bytes(int64_t I, int64_t J) {
    return align256((size_t)((I + AD_TILE_ROWS - 1) / AD_TILE_ROWS) * (size_t)((J + AD_TILE_COLS - 1) / AD_TILE_COLS) *
                    AD_TILE_SUMS * 4);
}

// The same with 64-bit sums and rows of any length (kernels_patterns_wide.hip): rows of a chunk, about 4096 wavefronts in all;
// partial sums [chunk][J + rows].
inline int antidiag_wide_rows(int64_t I, int64_t J) {
    const int64_t rows = (I * J / 64 / 4096 + 31) / 32 * 32;
    return (int)(rows < 32 ? 32 : rows > 512 ? 512 : rows);
}
inline size_t antidiag_wide_workspace_bytes(int64_t I, int64_t J) {
    const int64_t rows = antidiag_wide_rows(I, J);
    return align256((size_t)((I + rows - 1) / rows) * (size_t)(J + rows) * 8);
}

}  // namespace tad
