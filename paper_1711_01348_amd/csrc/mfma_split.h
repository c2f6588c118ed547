// The contractions of the worked expression with a long summed index on the bf16 matrix cores (kernels_mfma_split.hip).
#pragma once
#include <cstddef>
#include <cstdint>

#include "launch_geom.h"

namespace tad {

// Workspace behind that of the family: a flag, then the parts of a and b, six bytes an element, rows in whole tiles.
inline size_t long_workspace_bytes(int64_t I, int64_t J, int64_t K) {
    const size_t rows = (size_t)((I + 127) / 128 + (J + 127) / 128) * 128;
    return 256 + align256(rows * (size_t)K * 6);
}
// Longer sums of products would want their total apart from the sum that is being added up.
constexpr int kLongMaxK = 512;
// A chain of matrix instructions rounds its sum at every sixteen terms: the sum of 8192 terms of one sign was off by 2.2e-7 in two pieces of one chain each (the
// 32-bit instructions in eight pieces: 1.6e-7).  Totals in the kernel end the chains after 256 terms: 6e-8, and they cost 0.5 % for K <= 128, but 6 % above,
// where the tile takes the registers (4096 x 4096 x 256 128.6 us instead of 120).  There they are left out where the sums are cut short anyway: 1.2e-7 in four
// pieces; fewer are enough for short sums.
inline int64_t long_least_pieces(int64_t C) { return C <= 64 ? 1 : C <= 256 ? 2 : C <= 768 ? 3 : 4; }
// Gradients on the bf16 matrix cores / on the 32-bit ones, both of them with all four gradients, I x J x K: 1024 x 1024 x 32 18.9 / 21.1 us, x 64 21.0 / 23.7,
// x 128 26.3 / 25.9, x 256 35 / 31; 1400 x 1400 x 128 32.6 / 41.8, x 256 42.5 / 47.6; 4096 x 512 x 128 40.8 / 45.2, x 256 50 / 49; 4096 x 256 x 64 39 / 41, x 256 47 / 46;
// 2048 x 2048 x 256 54 / 58, x 512 83 / 95; 4096 x 4096 x 32 76 / 161, x 256 140 / 172.  Below the line there are too few workgroups of 128 rows.
inline bool long_pays(int64_t I, int64_t J, int64_t K) { return K <= kLongMaxK && I * J >= (K <= 64 ? 1 << 20 : 1900000); }
// ... and the forward pass: 4096 x 4096 x 64 32.2 / 33.5, x 128 43.8 / 51.1, x 256 63.8 / 82.1; 3000 x 3000 x 256 50 / 53; 4096 x 2048 x 64 21.6 / 20.5, x 128 28.1 / 29.7;
// 2045 x 3836 x 224 (480 tiles) 39.9 / 44.9; 2048 x 2048 x 256 (256 tiles) 31.9 / 27.7.
inline bool long_forward_pays(int64_t I, int64_t J, int64_t K) { return K >= 128 && ((I + 127) / 128) * ((J + 127) / 128) >= 480; }

#if defined(__HIPCC__)
struct LongProducts {
    const float *a, *b, *c, *d;
    float *rowv, *nb;
    void *parts;
    int *redo;             // set where a result is not finite: the 32-bit kernels are to do the work
    int I, J, K, c_ld;
};
int long_forward(const LongProducts &L, float *f, hipStream_t s);
// P_out, rowp (n_j pieces of chunk_j terms of the sum over j), T_out, colp (n_i pieces of the sum over i; 0: not wanted): as k_mfma_backward writes them;
// totals: see long_least_pieces
int long_backward(const LongProducts &L, const float *f, const float *df, float *P_out, float *rowp, int n_j, int chunk_j, float *T_out, float *colp, int n_i,
                  int chunk_i, bool totals, hipStream_t s);
#endif

}  // namespace tad
