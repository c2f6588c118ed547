// Zeros of a matrix of which only the diagonal holds anything, and sums that a launch makes beside them.
#pragma once
#include <hip/hip_runtime.h>

#include <cstdint>

namespace tad {

constexpr int kZeroBytes = 4096;   // of a workgroup of 256 threads: 41 us for 256 MiB against 45 / 47 us with 8 / 16 KiB and more with tiles

// Workgroup `piece` of a launch: zeros for kZeroBytes of dc (n elements), but not for the first I elements of its diagonal (`step` elements apart), which
// somebody else writes.  The stores bypass the caches: they are faster through them where a program writes the same tensor again and again (8192 x 8192
// 33 us instead of 40), but with other tensors in between the caches are written back under the launches that follow (a pass of the worked expression
// at 8192 x 8192 x 5 203 us instead of 176, 7663 x 60 x 6 65 instead of 57).
template <typename T>
__device__ __forceinline__ void zeros_off_diagonal(T *dc, unsigned n, unsigned step, unsigned I, unsigned piece) {
    constexpr unsigned V = 16 / sizeof(T), PIECE = 256 * V;
    typedef T vec __attribute__((ext_vector_type(V)));
    const unsigned from = piece * PIECE, at = from + threadIdx.x * V;
    const unsigned row = __builtin_amdgcn_readfirstlane((from + step - 1) / step);   // the first one from here on
    const unsigned first = row < I ? row * step : 0xffffffffu;
    if (at >= n) return;
    // at most one of them in a piece that has whole, aligned stores: the others, and rows that are shorter, look at every element
    const bool plain = (reinterpret_cast<uintptr_t>(dc) & 15) == 0 && step >= PIECE && from + PIECE <= n;   // the same for the workgroup
    if (plain) {
        if (first < at || first >= at + V) {
            vec zero;
#pragma unroll
            for (unsigned v = 0; v < V; ++v) zero[v] = T(0);
            __builtin_nontemporal_store(zero, reinterpret_cast<vec *>(dc + at));
        } else {
#pragma unroll
            for (unsigned v = 0; v < V; ++v)
                if (at + v != first) dc[at + v] = T(0);
        }
        return;
    }
#pragma unroll
    for (unsigned v = 0; v < V; ++v)
        if (at + v < n && !((at + v) % step == 0 && (at + v) / step < I)) dc[at + v] = T(0);
}

// acc of wavefront 0 = (0 + 1) + (2 + 3) of the four wavefronts' acc, lane by lane.
template <int N, int M>
__device__ __forceinline__ void add_wavefronts(double (&acc)[N], double (&red)[2][M][64], int wave, int lane) {
    static_assert(N <= M, "no room");
    if (wave & 1)
#pragma unroll
        for (int n = 0; n < N; ++n) red[wave >> 1][n][lane] = acc[n];
    __syncthreads();
    if (!(wave & 1))
#pragma unroll
        for (int n = 0; n < N; ++n) acc[n] += red[wave >> 1][n][lane];
    __syncthreads();
    if (wave == 2)
#pragma unroll
        for (int n = 0; n < N; ++n) red[0][n][lane] = acc[n];
    __syncthreads();
    if (wave == 0)
#pragma unroll
        for (int n = 0; n < N; ++n) acc[n] += red[0][n][lane];
}

}  // namespace tad
