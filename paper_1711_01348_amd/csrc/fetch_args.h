// What a kernel reads of its arguments, asked for in one go.
//
// The arguments lie in memory, and a wavefront that comes to a field whose line the scalar cache does not hold waits some 850 cycles for it.
// Plans and lists are read field by field, behind tests of other fields, so that a launch of a few microseconds spends most of them on one such
// wait after the other.  A word of every line, all of them held at one point of the kernel, brings the lines in together.
#pragma once
#include <hip/hip_runtime.h>

#include <cstddef>

#include "plan_dev.h"

namespace tad {

// Up to 16 lines of 64 bytes from byte `from` of an argument on.
template <int BYTES> __device__ __forceinline__ void fetch_lines(const void *argument, int from = 0) {
    static_assert(BYTES >= 4 && BYTES <= 16 * 64, "16 words are held below");
    const int *const at = reinterpret_cast<const int *>(static_cast<const char *>(argument) + from);
    int w[16];
#pragma unroll
    for (int i = 0; i < 16; ++i) w[i] = at[16 * i < BYTES / 4 ? 16 * i : BYTES / 4 - 1];
    asm volatile("" :: "s"(w[0]), "s"(w[1]), "s"(w[2]), "s"(w[3]), "s"(w[4]), "s"(w[5]), "s"(w[6]), "s"(w[7]), "s"(w[8]), "s"(w[9]), "s"(w[10]),
                 "s"(w[11]), "s"(w[12]), "s"(w[13]), "s"(w[14]), "s"(w[15]));
}

// The fields of a gather plan that every element reads, and the first of its rows; `slot`: the tensor whose offsets are.  (Sums over antidiagonals
// of 712 elements, softplus 512 x 384 x 200: 5.6 -> 4.5 us.)
__device__ __forceinline__ void fetch_gather(const GatherPlan &P, int slot) {
    asm volatile("" :: "s"(P.rank), "s"(P.shape[3]), "s"(P.U[1][3]), "s"(P.diag[0]), "s"(P.C[0][0]), "s"(P.C[3][3]), "s"(P.feas[0].scale),
                 "s"(P.feas[1].k0), "s"(P.feas[3].k0), "s"((int)P.lo_begin[0]), "s"(P.rows[0].scale), "s"(P.rows[1].k0), "s"(P.rows[3].k0),
                 "s"(P.offY[slot][0]), "s"(P.offZ[slot][0]), "s"(P.offZ[slot][3]), "s"(P.live));
}

}  // namespace tad
