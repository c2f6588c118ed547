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
// One diagonal element at most lies in a piece where rows are as long as one, and none behind the last: no division there.  Shorter rows: each thread looks for
// the first one from its elements on.  (An element at a time with a division each, c of 60000 x 1000 beside 1000 x 64 results: 75 us; so 40.)
template <typename T>
__device__ __forceinline__ void zeros_off_diagonal(T *dc, unsigned n, unsigned step, unsigned I, unsigned piece) {
    constexpr unsigned V = 16 / sizeof(T), PIECE = 256 * V, NONE = 0xffffffffu;
    typedef T vec __attribute__((ext_vector_type(V)));
    const unsigned from = piece * PIECE, row = __builtin_amdgcn_readfirstlane((from + step - 1) / step);
    const unsigned first = row < I ? row * step : NONE;   // the first diagonal element from here on
    const bool several = step < PIECE && first != NONE, aligned = (reinterpret_cast<uintptr_t>(dc) & 15) == 0;   // the same for the workgroup
    const unsigned at = from + threadIdx.x * V;
    vec zero;
#pragma unroll
    for (unsigned v = 0; v < V; ++v) zero[v] = T(0);
    if (aligned && !several && from + PIECE <= n) {       // nearly all pieces: a short way through
        if (first < at || first >= at + V) {
            __builtin_nontemporal_store(zero, reinterpret_cast<vec *>(dc + at));
        } else {
#pragma unroll
            for (unsigned v = 0; v < V; ++v)
                if (at + v != first) dc[at + v] = T(0);
        }
        return;
    }
    auto on_diagonal = [&](unsigned e) { return several ? e % step == 0 && e / step < I : e == first; };
    if (!aligned) {
#pragma unroll
        for (unsigned v = 0; v < V; ++v) {
            const unsigned e = from + 256 * v + threadIdx.x;
            if (e < n && !on_diagonal(e)) dc[e] = T(0);
        }
        return;
    }
    if (at >= n) return;
    unsigned own = first;
    if (several) {
        const unsigned r = (at + step - 1) / step;
        own = r < I ? r * step : NONE;
    }
    if (at + V <= n && (own < at || own >= at + V)) {
        __builtin_nontemporal_store(zero, reinterpret_cast<vec *>(dc + at));
        return;
    }
#pragma unroll
    for (unsigned v = 0; v < V; ++v)
        if (at + v < n && !on_diagonal(at + v)) dc[at + v] = T(0);
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
