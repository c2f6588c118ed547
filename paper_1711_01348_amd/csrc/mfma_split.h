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
// 32-bit instructions in eight pieces: 1.6e-7).  Totals in the kernel end the chains after 256 terms: 4e-8 to 6e-8, and they cost 0.5 % for K <= 128, but 6 % above,
// where the tile takes the registers (4096 x 4096 x 256 128.6 us instead of 120).  There they are left out where the sums are cut short anyway: 1.2e-7 in four
// pieces; fewer are enough for short sums.
inline int64_t long_least_pieces(int64_t C) { return C <= 64 ? 1 : C <= 256 ? 2 : C <= 768 ? 3 : 4; }
// Gradients on the bf16 matrix cores / on the 32-bit ones, both of them with all four gradients, I x J x K: 1024 x 1024 x 32 19.0 / 21.8 us, x 64 20.9 / 22.8,
// 4096 x 256 x 64 38.0 / 41.3, 16384 x 64 x 64 221 / 234; 1380 x 1380 x 96 28.8 / 40.3, x 256 39.8 / 45.7, x 512 52 / 65; 4096 x 512 x 128 39.5 / 45.6, x 256 48.0 / 50.3;
// 2048 x 2048 x 256 48.5 / 58, 4096 x 4096 x 256 120 / 176.  Below 1 900 000 results there are too few workgroups of 128 rows (1024 x 1024 x 128 26.3 / 25.9, x 256 35 / 31).
// Where one side is much longer than the other, its results leave few pieces to the other's and the short tiles stay empty: 256 x 16384 x 512 114 / 126, 180 x 11000 x 224 51 / 57,
// but 128 x 16384 x 256 60 / 58, x 512 109 / 93, 256 x 32000 x 256 137 / 125; 128 x 16384 x 192 54.8 / 55.3, 64 x 32768 x 192 111 / 77; 192 x 32000 x 128 89.6 / 92.5,
// 128 x 65536 x 128 169 / 142, 64 x 32768 x 96 80 / 71; not for narrow tiles, 64 x 65536 x 64 103 / 125.
inline bool long_pays(int64_t I, int64_t J, int64_t K) {
    if (K <= 64) return I * J >= 1 << 20;
    const int64_t shorter = I < J ? I : J, longer = I < J ? J : I;
    return K <= kLongMaxK && I * J >= 1900000 && longer <= shorter * (K <= 128 ? 160 : K <= 192 ? 128 : 64);
}
// ... and the forward pass: 4096 x 4096 x 64 32.2 / 33.5, x 128 43.8 / 51.1, x 256 63.8 / 82.1; 3000 x 3000 x 256 50 / 53; 4096 x 2048 x 64 21.6 / 20.5, x 128 28.1 / 29.7;
// 2045 x 3836 x 224 (480 tiles) 39.9 / 44.9; 2048 x 2048 x 256 (256 tiles) 31.9 / 27.7.  The parts of a and b are made for I J / (I + J) uses of each: 16384 x 512 x 128 31.7 / 32.2,
// 256 x 32000 x 128 34.0 / 32.3, 128 x 65536 x 128 38.0 / 36.8; 160 x 32000 x 256 44.6 / 47.5, 128 x 65536 x 256 69 / 58.
inline bool long_forward_pays(int64_t I, int64_t J, int64_t K) {
    return K >= 128 && K <= kLongMaxK && I * J >= 1900000 && ((I + 127) / 128) * ((J + 127) / 128) >= 480 && I * J >= (K < 256 ? 480 : 150) * (I + J);
}

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
