// Products of 32-bit matrices on the bf16 matrix cores (kernels_split.hip): geometry and the range of operands they take.
#pragma once
#include <cstddef>
#include <cstdint>

#include "launch_geom.h"

namespace tad {

struct SplitGeom {
    int gm, gn, q_blocks;               // tiles of 128 rows of either operand, fragments of 16 terms
    size_t a_offset, b_offset, bytes;   // workspace: exponents, parts of A, parts of B
};
inline SplitGeom split_geom(int64_t M, int64_t N, int64_t K) {
    SplitGeom g;
    g.gm = (int)((M + 127) / 128);
    g.gn = (int)((N + 127) / 128);
    g.q_blocks = (int)((K + 15) / 16);
    g.a_offset = 256 + align256((size_t)(g.gm + g.gn) * 4 * (size_t)((g.q_blocks + 15) / 16) * 4);
    g.b_offset = g.a_offset + (size_t)g.gm * 4 * g.q_blocks * 3072;
    g.bytes = g.b_offset + (size_t)g.gn * 4 * g.q_blocks * 3072;
    return g;
}
// Two tiles for every compute unit (a round of tiles takes as long however few they are) and a sum long enough for two short
// launches.  Splitting moves ten bytes per element of the operands, the product saves a fourth of its time: that pays where
// M N / (M + N), the length of the sums' other side, is large enough.  These and the 32-bit kernel, M x N x K with 4096 x 4096 x 4096 870 / 1042 us, 4096 x 4096 x 1024 229 / 286, and of the
// smallest taken 2048 x 4096 x 1024 128 / 146, 2944 x 2944 x 2048 369 / 414, 1024 x 8192 x 1024
// 137 / 149 (M N / (M + N) = 910); not taken 512 x 16384 x 1024 146 / 145 (496), x 4096 579 / 560, 256 x 32768 x 2048 366 / 288 (254),
// 128 x 65536 x 2048 506 / 298.
inline bool split_pays(int64_t M, int64_t N, int64_t K) {
    const SplitGeom g = split_geom(M, N, K);
    return (int64_t)g.gm * g.gn >= 512 && K >= 1024 && M * N >= 768 * (M + N);
}

#if defined(__HIPCC__)
constexpr float kSplitScale = 16777216.f;   // the operands are split this many times as large
// Fragments of 16 terms whose products are added up before they are scaled back and added to the total: an even number.
constexpr int kSplitChain = 8;
// range: largest exponents (biased by 127) of the operands.  Every number is finite, and stays so times 2^24, and 128 products
// of them (each below 2^71) do not overflow before they are scaled back.
__device__ __forceinline__ bool split_in_range(const int *range) {
    return range[0] <= 227 && range[1] <= 227 && range[0] + range[1] <= 2 * 127 + 69;
}
#endif

}  // namespace tad
