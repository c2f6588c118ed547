// Element-wise access to the operands of an expression without summation indices.
#pragma once
#include <hip/hip_runtime.h>

#include "launch.h"
#include "plan_dev.h"

namespace tad {

// Offsets of the operands at element `lin` of an expression without summation indices.
__device__ __forceinline__ void element_offsets(const ForwardPlan &P, int n_ops, int lin, int64_t *base) {
    // unrolled to the largest rank and cut short by tests of the uniform rank, so that every field of the plan comes from a
    // fixed place in the kernel arguments
    int32_t ext[kMaxExt];
    int t = lin;
#pragma unroll
    for (int d = kMaxExt - 1; d >= 1; --d) {
        ext[d] = 0;
        if (d < P.n_f) {
            const int s = P.f_shape[d], q = t / s;
            ext[d] = t - q * s;
            t = q;
        }
    }
    ext[0] = t;
#pragma unroll
    for (int p = 0; p < kMaxArgs; ++p) {
        if (p >= n_ops) continue;
        int64_t o = P.base0[p];
#pragma unroll
        for (int d = 0; d < kMaxExt; ++d)
            if (d < P.n_f) o += P.off[p][d] * (int64_t)ext[d];
        base[p] = o;
    }
}

// Values of the operands of `mask` at element `lin`, widened; the others are 0.
template <typename T, typename TV>
__device__ __forceinline__ void element_values(const ForwardPlan &P, int n_ops, uint32_t mask, const ArgPtrs &A, int lin, TV *v) {
    int64_t base[kMaxArgs];
    element_offsets(P, n_ops, lin, base);
#pragma unroll
    for (int p = 0; p < kMaxArgs; ++p) v[p] = p < n_ops && ((mask >> p) & 1u) ? (TV)static_cast<const T *>(A.p[p])[base[p]] : TV(0);
}

}  // namespace tad
