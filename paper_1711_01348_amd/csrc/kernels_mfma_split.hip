// Worked expression with a long summed index (kernels_mfma.hip: its contractions a . b, P = G b, T = (c G)^T a) on the bf16 matrix cores, to
// 32-bit precision.
//
// A 32-bit number is the sum of three bf16 numbers x1 + x2 + x3 (8 + 8 + 8 bits, each the nearest to what the ones before leave).  Six of the
// nine products of the parts are taken, each exact in 32 bits: what is left out is at most 2^-24 of |x y| (x2 y3 and x3 y2, 2^-25 each), of either sign
// and 2^-27.5 on average; sums of one term are as exact as the 32-bit instructions' (da 4.4e-8).  x1 y1 is added up by itself and the five smaller products
// by themselves, so that the roundings of those do not count; where pieces of a sum are long its chain ends after 256 terms (see mfma_split.h).
// v_mfma_f32_32x32x16_bf16 does sixteen times the work of v_mfma_f32_32x32x2f32 per cycle: six of them take 3 / 8 of its time.
//
// Operands that are tensors (a, b) are split once, by the launch that also forms the norms (k_long_prep), and written fragment by fragment in the
// order in which a wavefront feeds them to the matrix cores ([16 terms][32 rows][part][lane][8 terms], zeros beyond the edges): they go
// from there to LDS without passing through registers.  G = df f exists nowhere: it is formed, split and written to LDS by the
// threads that load df and f, one stage ahead.
//
// 4096 x 4096 x 256: forward pass 82 us on the 32-bit matrix instructions, 64 here; all four gradients 192 (six launches), 176 (the 32-bit kernels in three),
// 120 here; errors against 64 bits, 32-bit instructions in eight pieces and here, f 3.2e-8, 3.1e-8, da 3.0e-7, 1.4e-7, dc 9.3e-8, 7.6e-8, dd 1.5e-7, 1.4e-7.  What bounds them: the clock under load (1.8 GHz, as in
// kernels_split.hip) and, in the gradients, G, whose 134 MB are read twice and whose parts are formed on the vector ALU while both wavefronts of a
// SIMD wait for them.  Tried: fragments read from LDS half a stage ahead (132 -> 146 us), wavefronts of a SIMD that form G in turn (125 -> 137).
//
// Parts and their products have to stay normal numbers, as in kernels_split.hip: what is split is 2^24 times as large, so that the third part of the
// smallest 32-bit number is one, and the results are scaled back.  (Unscaled, G of 2^-115 gave da that was off by 2e-6, of 2^-118 by 2e-5, and db,
// whose G carries c, by more.)  A part that is no finite number turns every result it takes part in into one that is not finite, so the results tell
// whether all of it stayed below the upper end: if they do not (some sum of products beyond 2^80), a flag is set and the kernels of kernels_mfma.hip,
// launched behind these, do the work again.
#include <hip/hip_runtime.h>

#include "launch.h"
#include "launch_geom.h"
#include "mfma_split.h"
#include "profile.h"
#include "split.h"

namespace tad {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float float4l __attribute__((ext_vector_type(4)));
typedef float float16l __attribute__((ext_vector_type(16)));
typedef unsigned piece __attribute__((ext_vector_type(4)));   // 16 bytes, a lane's share of a part of a fragment
typedef const __attribute__((address_space(1))) void *global_ptr;
typedef __attribute__((address_space(3))) void *lds_ptr;

constexpr int kFragment = 3 * 64;       // pieces of a fragment of 32 rows and 16 terms
constexpr float kLog2eL = 1.4426950408889634f;
constexpr float kLongBack = 1.f / (kSplitScale * kSplitScale);   // of a sum of products

__device__ __forceinline__ int long_acc_row(int r, int lane) { return 8 * (r >> 2) + 4 * (lane >> 5) + (r & 3); }

// the parts of v[] times kSplitScale
__device__ __forceinline__ void split_three(const float (&v)[8], piece (&out)[3]) {
    bf16x8 p1, p2, p3;
#pragma unroll
    for (int e = 0; e < 8; ++e) {
        const float sv = v[e] * kSplitScale;
        p1[e] = (__bf16)sv;
        const float r = sv - (float)p1[e];
        p2[e] = (__bf16)r;
        p3[e] = (__bf16)(r - (float)p2[e]);
    }
    out[0] = __builtin_bit_cast(piece, p1);
    out[1] = __builtin_bit_cast(piece, p2);
    out[2] = __builtin_bit_cast(piece, p3);
}

// Behind it, what every wavefront of the workgroup has sent for is in LDS, and what it has read of LDS in registers.
__device__ __forceinline__ void landed() {
    __builtin_amdgcn_sched_barrier(0);
    asm volatile("" ::: "memory");
    __builtin_amdgcn_s_waitcnt(0x0070);   // vmcnt(0), lgkmcnt(0)
    __builtin_amdgcn_s_barrier();
    asm volatile("" ::: "memory");
    __builtin_amdgcn_sched_barrier(0);
}

// Six products of fragments av and bv: the largest one to `big`, the others, smallest first, to `small`.
__device__ __forceinline__ void six_products(const piece (&av)[3], const piece (&bv)[3], float16l &big, float16l &small) {
    auto mul = [&](int i, int j, float16l s) {
        return __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, av[i]), __builtin_bit_cast(bf16x8, bv[j]), s, 0, 0, 0);
    };
    small = mul(2, 0, small);
    big = mul(0, 0, big);
    small = mul(0, 2, small);
    small = mul(1, 1, small);
    small = mul(1, 0, small);
    small = mul(0, 1, small);
}

// ---------------------------------------------------------------------------------------------
// Parts and norms.  A workgroup takes 32 rows of a, or of b.  TURNED = false (forward pass): the rows of the fragments are those of the
// tensor, the terms are k; also rowv[i] = {|a_i|^2, -log2e c_ii, -log2e D_i, c_ii} with D_i = sum_k d_{i+k}^3, and nb[j] = |b_j|^2.
// TURNED = true (gradients): the rows of the fragments are k, the terms the rows of the tensor; rowv without D.
// ---------------------------------------------------------------------------------------------
struct LongPrep {
    const float *a, *b, *c, *d;
    float *rowv, *nb;
    piece *pa, *pb;
    int *redo;
    int I, J, K, c_ld;
    int blocks_a;          // workgroups of a
    int rows_a, rows_b;    // TURNED = false: fragments of 32 rows
};
template <bool TURNED>
__global__ __launch_bounds__(256) void k_long_prep(const LongPrep P) {
    __shared__ double red[2][8][33];
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, K = P.K;
    if (blockIdx.x == 0 && tid == 0) *P.redo = 0;
    const bool second = (int)blockIdx.x >= P.blocks_a;
    const int block = second ? (int)blockIdx.x - P.blocks_a : (int)blockIdx.x, r0 = block * 32, rows = second ? P.J : P.I;
    const float *src = second ? P.b : P.a;
    piece *out = second ? P.pb : P.pa;
    // the norms: eight threads to a row
    const int row = tid & 31, part = tid >> 5;
    const bool inside = r0 + row < rows;
    const float *own = src + (size_t)(inside ? r0 + row : 0) * K;
    double norm = 0.0, D = 0.0;
#pragma unroll 4
    for (int k = 4 * part; k < K; k += 32) {
        const float4l v = *reinterpret_cast<const float4l *>(own + k);
#pragma unroll
        for (int e = 0; e < 4; ++e) norm += (double)v[e] * (double)v[e];
    }
    if (!TURNED && !second) {   // the same for the whole workgroup
        __shared__ double cubes[32 + kLongMaxK];
        for (int n = tid; n < min(32, rows - r0) + K - 1; n += 256) {
            const double dv = P.d[r0 + n];
            cubes[n] = dv * dv * dv;
        }
        __syncthreads();
#pragma unroll 4
        for (int k = part; k < K; k += 8) D += cubes[row + k];   // (rows that do not exist: not used)
    }
    red[0][part][row] = norm;
    red[1][part][row] = D;
    if constexpr (!TURNED) {
        const int of = second ? P.rows_b : P.rows_a, r = lane & 31;
        for (int qb = wave; qb < K / 16; qb += 4) {
            float v[8];
            const float *at = src + (size_t)(r0 + r < rows ? r0 + r : 0) * K + qb * 16 + 8 * (lane >> 5);
#pragma unroll
            for (int h = 0; h < 2; ++h) {
                const float4l x = reinterpret_cast<const float4l *>(at)[h];
#pragma unroll
                for (int e = 0; e < 4; ++e) v[4 * h + e] = r0 + r < rows ? x[e] : 0.f;
            }
            piece p[3];
            split_three(v, p);
            piece *to = out + ((size_t)qb * of + block) * kFragment + lane;
#pragma unroll
            for (int s = 0; s < 3; ++s) to[64 * s] = p[s];
        }
    } else {
        // fragments in groups of eight along k: [group][16 terms][32 k]
        const int terms = 2 * ((rows + 31) / 32);
        for (int n = wave; n < K / 16; n += 4) {   // two times K / 32 fragments
            const int kb = n >> 1, h = n & 1, group = kb >> 3, wide = min(8, K / 32 - 8 * group), i0 = r0 + 16 * h + 8 * (lane >> 5);
            float v[8];
#pragma unroll
            for (int e = 0; e < 8; ++e) {
                const float x = src[(size_t)min(i0 + e, rows - 1) * K + kb * 32 + (lane & 31)];
                v[e] = i0 + e < rows ? x : 0.f;
            }
            piece p[3];
            split_three(v, p);
            piece *to = out + ((size_t)group * 8 * terms + (size_t)(2 * block + h) * wide + (kb & 7)) * kFragment + lane;
#pragma unroll
            for (int s = 0; s < 3; ++s) to[64 * s] = p[s];
        }
    }
    __syncthreads();
    if (tid >= 32 || r0 + tid >= rows) return;
    norm = D = 0.0;
#pragma unroll
    for (int p = 0; p < 8; ++p) {
        norm += red[0][p][tid];
        D += red[1][p][tid];
    }
    const int i = r0 + tid;
    if (second) {
        P.nb[i] = (float)norm;
        return;
    }
    const float cv = P.c[(size_t)i * P.c_ld + i];
    const float4l v = {(float)norm, -kLog2eL * cv, (float)(-(double)kLog2eL * D), cv};
    *reinterpret_cast<float4l *>(P.rowv + (size_t)i * 4) = v;
}

// ---------------------------------------------------------------------------------------------
// Forward pass: workgroup tile 128 x 128, four wavefronts of 64 x 64, 16 terms per stage in two sets of LDS.
// ---------------------------------------------------------------------------------------------
__global__ __launch_bounds__(256, 3) void k_long_forward(const piece *__restrict__ pa, const piece *__restrict__ pb, const float *__restrict__ rowv,
                                                         const float *__restrict__ nb, float *__restrict__ f, int *__restrict__ redo, int I, int J,
                                                         int q_blocks, int gi, int gj) {
    constexpr int PA = 4 * kFragment, STAGE = 2 * PA, LO = 68;
    __shared__ piece smem[2 * STAGE];
    static_assert(4 * 32 * LO * sizeof(float) <= sizeof(smem), "the results' stage does not fit");
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6), wm = wave >> 1, wn = wave & 1;
    // the dies take workgroups in turn: each gets a contiguous range of tiles, in groups of four tile rows
    const int total = gi * gj;
    int id = blockIdx.x;
    if (id < total / 8 * 8) id = (id % 8) * (total / 8) + id / 8;
    const int g0 = id / (4 * gj) * 4, rows = min(4, gi - g0), in = id - g0 * gj, ti = g0 + in % rows, tj = in / rows;
    const piece *at = pa + (size_t)ti * PA + wave * 64 + lane, *bt = pb + (size_t)tj * PA + wave * 64 + lane;
    const unsigned next_a = (unsigned)gi * PA, next_b = (unsigned)gj * PA;
    auto load = [&](int set) {
#pragma unroll
        for (int p = 0; p < 6; ++p)
            __builtin_amdgcn_global_load_lds((global_ptr)(p < 3 ? at + 256 * p : bt + 256 * (p - 3)), (lds_ptr)(smem + set * STAGE + wave * 64 + 256 * p), 16, 0, 0);
        at += next_a;
        bt += next_b;
    };
    float16l big[2][2], small[2][2];
#pragma unroll
    for (int x = 0; x < 2; ++x)
#pragma unroll
        for (int y = 0; y < 2; ++y)
#pragma unroll
            for (int r = 0; r < 16; ++r) big[x][y][r] = small[x][y][r] = 0.f;
    load(0);
    const int fa = wm * 2 * kFragment + lane, fb = PA + wn * 2 * kFragment + lane;
    for (int t = 0; t < q_blocks; ++t) {
        const int set = t & 1;
        landed();   // stage t is in LDS, stage t - 1 is not read any more
        if (t + 1 < q_blocks) load(set ^ 1);   // the same for the whole workgroup
        const piece *S = smem + set * STAGE;
        piece av[2][3], bv[2][3];
#pragma unroll
        for (int s = 0; s < 3; ++s)
#pragma unroll
            for (int x = 0; x < 2; ++x) {
                av[x][s] = S[fa + x * kFragment + s * 64];
                bv[x][s] = S[fb + x * kFragment + s * 64];
            }
#pragma unroll
        for (int x = 0; x < 2; ++x)
#pragma unroll
            for (int y = 0; y < 2; ++y) six_products(av[x], bv[y], big[x][y], small[x][y]);
    }
    __syncthreads();
    // f = exp2(c' (|a|^2 + |b|^2 + 2 a.b) + D'): each wavefront stages 32 x 64 results in its own quarter of LDS and stores whole rows of its tile
    float *const stage = reinterpret_cast<float *>(smem) + wave * (32 * LO);
    const int i0 = ti * 128 + wm * 64, j0 = tj * 128 + wn * 64;
    bool finite = true;
    const int c = (lane & 15) * 4, j = j0 + c;
    const float4l nbj = *reinterpret_cast<const float4l *>(nb + min(j, J - 4));
#pragma unroll
    for (int x = 0; x < 2; ++x) {
#pragma unroll
        for (int y = 0; y < 2; ++y)
#pragma unroll
            for (int r = 0; r < 16; ++r) stage[long_acc_row(r, lane) * LO + 32 * y + (lane & 31)] = big[x][y][r] + small[x][y][r];
#pragma unroll 2
        for (int n = 0; n < 8; ++n) {
            const int rl = n * 4 + (lane >> 4), i = i0 + 32 * x + rl;
            const float4l rv = reinterpret_cast<const float4l *>(rowv)[min(i, I - 1)], ab = *reinterpret_cast<const float4l *>(stage + rl * LO + c);
            float4l v;
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                finite = finite && __builtin_isfinite(ab[e]);
                v[e] = __builtin_amdgcn_exp2f(fmaf(rv[1], rv[0] + nbj[e] + 2.f * kLongBack * ab[e], rv[2]));
            }
            if (i < I && j < J) *reinterpret_cast<float4l *>(f + (size_t)i * J + j) = v;   // (J % 4 == 0: the four columns exist together)
        }
    }
    if (!finite) atomicOr(redo, 1);
}

// ---------------------------------------------------------------------------------------------
// The contractions of the gradients.  Workgroup tile 128 x 32 GROUP (rows x k), eight wavefronts, 32 terms per stage, the sum in pieces
// whose partial results and plain sums are those of k_mfma_backward:
//   TRANS = false:  rows i, terms j:  out = sum_j G_ij b_jk,       sums[2 s] = sum_j G_ij, sums[2 s + 1] = sum_j G_ij |b_j|^2
//   TRANS = true:   rows j, terms i:  out = sum_i c_ii G_ij a_ik,  sums[s] = sum_i c_ii G_ij
// ---------------------------------------------------------------------------------------------
struct LongSide {
    const piece *parts;
    float *out, *sums;
    int chunk, chain;          // terms of a piece, of a chain of instructions
};
struct LongBackward {
    const float *f, *df, *rowv, *nb;
    LongSide side[2];
    int *redo;
    int I, J, K;
    int first, n_j, n_i;       // workgroups of the first sum, pieces of either
};
template <bool TRANS, int RX, int RY, int WN, bool TOTALS>
__device__ __forceinline__ void long_contraction(const LongBackward &L, piece *const smem, const int tile, const int split) {
    constexpr int GROUP = RY * WN;                             // fragments of 32 columns
    static_assert(RX * (8 / WN) == 4, "128 rows");
    constexpr int A = 4 * 2 * kFragment, B = GROUP * 2 * kFragment, STAGE = A + B;
    const float *const __restrict__ f = L.f, *const __restrict__ df = L.df, *const __restrict__ rowv = L.rowv, *const __restrict__ nb = L.nb;
    const piece *const __restrict__ parts = L.side[TRANS].parts;
    float *const __restrict__ out = L.side[TRANS].out, *const __restrict__ sums = L.side[TRANS].sums;
    const int I = L.I, J = L.J, K = L.K, chunk = L.side[TRANS].chunk;
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6), wm = wave / WN, wn = wave % WN;
    const int M = TRANS ? J : I, C = TRANS ? I : J, m0 = tile * 128, z = blockIdx.y;
    const int begin = split * chunk, end = min(C, begin + chunk), wide = min(GROUP, K / 32 - GROUP * z);
    // G: a thread owns one row and eight neighbouring terms of a stage.  TRANS = false: lanes 16 rows x 4 octets (64 bytes of a row from each of
    // two loads); TRANS = true: 64 neighbouring rows j, an octet of i per wavefront.
    const int g_row = TRANS ? (wave & 1) * 64 + lane : wave * 16 + (lane & 15), oct = TRANS ? wave >> 1 : lane >> 4;
    const int m = min(m0 + g_row, M - 1);
    float gdf[8], gf[8], gc = 0.f;
    float4l gn[2];
    auto load_g = [&](int c0) {
        const int q = c0 + 8 * oct;
        if constexpr (TRANS) {
#pragma unroll
            for (int e = 0; e < 8; ++e) {
                const size_t at = (size_t)min(q + e, end - 1) * J + m;
                gdf[e] = df[at];
                gf[e] = f[at];
            }
            gc = rowv[4 * min(q + (lane & 7), end - 1) + 3];   // c_ii of the octet, one in each of eight lanes
        } else {
#pragma unroll
            for (int h = 0; h < 2; ++h) {
                const int j = min(q + 4 * h, end - 4);   // (J % 4 == 0: four terms exist together)
                const float4l x = *reinterpret_cast<const float4l *>(df + (size_t)m * J + j), y = *reinterpret_cast<const float4l *>(f + (size_t)m * J + j);
                gn[h] = *reinterpret_cast<const float4l *>(nb + j);
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    gdf[4 * h + e] = x[e];
                    gf[4 * h + e] = y[e];
                }
            }
        }
    };
    // 32-bit sums of a whole piece would be less exact than the products: those of a chain are added up in 64 bits (of every stage: 4096 x 4096 x 256 123.5 us
    // instead of 119.3, the additions wait for the matrix cores)
    float plain_chain = 0.f, weighted_chain = 0.f;
    double plain = 0.0, weighted = 0.0;
    const int g_to = ((g_row >> 5) * 2 + (oct >> 1)) * kFragment + (g_row & 31) + 32 * (oct & 1);
    auto stage_g = [&](int c0, int set) {   // forms G of the loaded stage
        const int q = c0 + 8 * oct;
        float g[8];
        const float c = q + (lane & 7) < end ? gc : 0.f;
#pragma unroll
        for (int e = 0; e < 8; ++e) {
            if constexpr (TRANS) {   // (beyond the end the last term again, times zero)
                g[e] = gdf[e] * gf[e] * __int_as_float(__builtin_amdgcn_readlane(__float_as_int(c), e));
            } else {
                g[e] = q + (e & 4) < end ? gdf[e] * gf[e] : 0.f;
            }
        }
        plain_chain += ((g[0] + g[1]) + (g[2] + g[3])) + ((g[4] + g[5]) + (g[6] + g[7]));
        if constexpr (!TRANS)
            weighted_chain += ((g[0] * gn[0][0] + g[1] * gn[0][1]) + (g[2] * gn[0][2] + g[3] * gn[0][3])) +
                              ((g[4] * gn[1][0] + g[5] * gn[1][1]) + (g[6] * gn[1][2] + g[7] * gn[1][3]));
        piece p[3];
        split_three(g, p);
#pragma unroll
        for (int s = 0; s < 3; ++s) smem[set * STAGE + g_to + 64 * s] = p[s];
    };
    // the other operand: two fragments of terms per stage, contiguous
    const int stage_pieces = 2 * wide * kFragment;
    const piece *const first = parts + (size_t)z * GROUP * (2 * ((C + 31) / 32)) * kFragment + tid;
    auto load_b = [&](int set, int c0) {
        const piece *const from = first + (size_t)(min(c0, end - 1) / 32) * stage_pieces;
#pragma unroll
        for (int p = 0; p < 2 * GROUP * kFragment; p += 512) {   // (wide * 6 wavefronts' loads: the rest of the last round is left out, uniform per wavefront)
            if (p + wave * 64 < stage_pieces)
                __builtin_amdgcn_global_load_lds((global_ptr)(from + p), (lds_ptr)(smem + set * STAGE + A + p + wave * 64), 16, 0, 0);
        }
        __builtin_amdgcn_sched_barrier(0);
        asm volatile("" ::: "memory");
    };
    // TOTALS: an eighth of the sum, at most 256 terms, is added up by itself and then to the total.  Tall tiles have no registers for three sums: their
    // smaller products start from zero for every fragment of terms and are added to the larger ones on the vector ALU.
    constexpr bool JOINED = TOTALS && RX > 1;
    const float16l zero = {};
    float16l big[RX][RY], small[RX][RY], total[RX][RY];
#pragma unroll
    for (int x = 0; x < RX; ++x)
#pragma unroll
        for (int y = 0; y < RY; ++y) big[x][y] = small[x][y] = total[x][y] = zero;
    const int have = min(RY, wide - wn * RY);   // column fragments of this wavefront that exist (may be negative)
    auto products = [&](int set, int qb) {      // (columns that do not exist are computed from the last one and not stored)
        const piece *S = smem + set * STAGE;
        piece av[RX][3], bv[RY][3];
#pragma unroll
        for (int s = 0; s < 3; ++s) {
#pragma unroll
            for (int x = 0; x < RX; ++x) av[x][s] = S[((wm * RX + x) * 2 + qb) * kFragment + 64 * s + lane];
#pragma unroll
            for (int y = 0; y < RY; ++y) bv[y][s] = S[A + (qb * wide + min(wn * RY + y, wide - 1)) * kFragment + 64 * s + lane];
        }
#pragma unroll
        for (int y = 0; y < RY; ++y)
#pragma unroll
            for (int x = 0; x < RX; ++x) {
                if constexpr (JOINED) {
                    float16l rest = zero;
                    six_products(av[x], bv[y], big[x][y], rest);
                    big[x][y] += rest;
                } else {
                    six_products(av[x], bv[y], big[x][y], small[x][y]);
                }
            }
    };
    auto end_of_chain = [&] {
        plain += (double)plain_chain;
        plain_chain = 0.f;
        if constexpr (!TRANS) {
            weighted += (double)weighted_chain;
            weighted_chain = 0.f;
        }
        if constexpr (TOTALS) {
#pragma unroll
            for (int x = 0; x < RX; ++x)
#pragma unroll
                for (int y = 0; y < RY; ++y) {
                    total[x][y] += big[x][y];
                    big[x][y] = zero;
                }
        }
    };
    const int chain = L.side[TRANS].chain;
    int left = chain;
    load_g(begin);
    int set = 1;
    // The first pass only brings the first stage to LDS.  Nothing here depends on whether there is a next stage (it is then the last one again, and
    // zeros for G): loads under a condition would be waited for where the paths meet.
#pragma unroll 1
    for (int c0 = begin - 32; c0 < end; c0 += 32, set ^= 1) {
        const bool work = have > 0 && c0 >= begin;   // the same for the wavefront
        load_b(set ^ 1, c0 + 32);
        if (work) products(set, 0);
        // G has to be here now, and the other operand's copies to LDS, half a stage old, are waited for with it: the barrier below then needs no
        // count of the loads of G that are issued in between and may still be on their way
        __builtin_amdgcn_sched_barrier(0);
        asm volatile("" ::: "memory");
        __builtin_amdgcn_s_waitcnt(0x0f70);   // vmcnt(0)
        asm volatile("" ::: "memory");
        __builtin_amdgcn_sched_barrier(0);
        stage_g(c0 + 32, set ^ 1);
        load_g(c0 + 64);
        if (work) products(set, 1);
        if (c0 >= begin && (left -= 32) == 0) {   // the same for the whole workgroup
            left = chain;
            end_of_chain();
        }
        // what this wavefront has written and read of LDS is done
        __builtin_amdgcn_sched_barrier(0);
        asm volatile("" ::: "memory");
        __builtin_amdgcn_s_waitcnt(0xc07f);   // lgkmcnt(0)
        __builtin_amdgcn_s_barrier();
        asm volatile("" ::: "memory");
    }
    landed();   // nothing is on its way to LDS any more
    // Each wavefront stages its results in LDS and stores whole rows.  (Code that runs once is fetched at some 200 cycles per 64 bytes:
    // as little of it as possible is unrolled.)
    constexpr int W = 32 * RY, LO = W + 4, ROWS = 256 / W;   // rows per store of the wavefront
    static_assert(8 * 32 * RX * LO * sizeof(float) <= 2 * STAGE * sizeof(piece), "the results' stage does not fit");
    float *const own = reinterpret_cast<float *>(smem) + wave * (32 * RX * LO);
#pragma unroll
    for (int x = 0; x < RX; ++x)
#pragma unroll
        for (int y = 0; y < RY; ++y)
#pragma unroll
            for (int r = 0; r < 16; ++r) own[(32 * x + long_acc_row(r, lane)) * LO + 32 * y + (lane & 31)] =
                    ((TOTALS ? total[x][y][r] : 0.f) + (JOINED ? big[x][y][r] : big[x][y][r] + small[x][y][r])) * kLongBack;
    bool finite = true;
    const int col = lane % (W / 4) * 4, k = (GROUP * z + wn * RY) * 32 + col;
    if (k < K) {   // (K % 32 == 0: the four columns exist together)
#pragma unroll 1
        for (int n = lane / (W / 4); n < 32 * RX; n += ROWS) {
            const int row = m0 + wm * RX * 32 + n;
            if (row >= M) break;
            const float4l v = *reinterpret_cast<const float4l *>(own + n * LO + col);
#pragma unroll
            for (int e = 0; e < 4; ++e) finite = finite && __builtin_isfinite(v[e]);
            *reinterpret_cast<float4l *>(out + ((size_t)split * M + row) * K + k) = v;
        }
    }
    __syncthreads();
    if (!finite) atomicOr(L.redo, 1);
    if (z != 0) return;
    // the four octets of a row
    double *const red = reinterpret_cast<double *>(smem);
    red[oct * 128 + g_row] = plain + (double)plain_chain;
    if constexpr (!TRANS) red[512 + oct * 128 + g_row] = weighted + (double)weighted_chain;
    __syncthreads();
    if (tid >= 128 || m0 + tid >= M) return;
    auto sum = [&](int at) { return (float)((red[at + tid] + red[at + 128 + tid]) + (red[at + 256 + tid] + red[at + 384 + tid])); };
    if constexpr (TRANS) sums[(size_t)split * J + m0 + tid] = sum(0);
    else {
        sums[((size_t)split * 2) * I + m0 + tid] = sum(0);
        sums[((size_t)split * 2 + 1) * I + m0 + tid] = sum(512);
    }
}

// Both contractions in one launch: tiles of rows i, then tiles of rows j.
template <int RX, int RY, int WN, bool TOTALS>
__global__ __launch_bounds__(512, 2) void k_long_backward(const LongBackward L) {
    __shared__ piece smem[2 * (4 + RY * WN) * 2 * kFragment];
    // the dies take workgroups in turn: each gets a contiguous range of them, of as few pieces of the tensors as can be
    const int total = gridDim.x, id = (int)blockIdx.x < total / 8 * 8 ? (int)blockIdx.x % 8 * (total / 8) + (int)blockIdx.x / 8 : (int)blockIdx.x, second = id - L.first;
    const int ti = L.first / L.n_j;
    if (id < L.first) long_contraction<false, RX, RY, WN, TOTALS>(L, smem, id % ti, id / ti);
    else long_contraction<true, RX, RY, WN, TOTALS>(L, smem, second % ((total - L.first) / L.n_i), second / ((total - L.first) / L.n_i));
}

int long_forward(const LongProducts &L, float *f, hipStream_t s) {
    const int gi = (L.I + 127) / 128, gj = (L.J + 127) / 128;
    LongPrep P{L.a, L.b, L.c, L.d, L.rowv, L.nb, static_cast<piece *>(L.parts), nullptr, L.redo, L.I, L.J, L.K, L.c_ld, 4 * gi, 4 * gi, 4 * gj};
    P.pb = P.pa + (size_t)P.rows_a * (L.K / 16) * kFragment;
    TAD_LAUNCH("k_long_prep", k_long_prep<false>, dim3(4 * (gi + gj)), dim3(256), 0, s, P);
    if (hipGetLastError() != hipSuccess) return TAD_EDEVICE;
    TAD_LAUNCH("k_long_forward", k_long_forward, dim3(gi * gj), dim3(256), 0, s, (const piece *)P.pa, (const piece *)P.pb, (const float *)L.rowv,
               (const float *)L.nb, f, L.redo, L.I, L.J, L.K / 16, gi, gj);
    return hipGetLastError() == hipSuccess ? TAD_OK : TAD_EDEVICE;
}

int long_backward(const LongProducts &L, const float *f, const float *df, float *P_out, float *rowp, int n_j, int chunk_j, float *T_out, float *colp, int n_i,
                  int chunk_i, bool totals, hipStream_t s) {
    LongPrep P{L.a, L.b, L.c, L.d, L.rowv, L.nb, static_cast<piece *>(L.parts), nullptr, L.redo, L.I, L.J, L.K, L.c_ld, (L.I + 31) / 32, 0, 0};
    P.pb = P.pa + (size_t)(2 * P.blocks_a) * (L.K / 32) * kFragment;
    TAD_LAUNCH("k_long_prep", k_long_prep<true>, dim3(P.blocks_a + (L.J + 31) / 32), dim3(256), 0, s, P);
    if (hipGetLastError() != hipSuccess) return TAD_EDEVICE;
    const int first = (L.I + 127) / 128 * n_j, blocks = first + (L.J + 127) / 128 * n_i;
    const LongBackward B{f, df, L.rowv, L.nb, {{P.pb, P_out, rowp, chunk_j, mfma_chain(L.J)}, {P.pa, T_out, colp, chunk_i, mfma_chain(L.I)}}, L.redo, L.I, L.J, L.K, first, n_j, n_i};
#define TAD_LONG(RX, RY, WN, TOTALS)                                                                                                             \
    TAD_LAUNCH("k_long_backward", (k_long_backward<RX, RY, WN, TOTALS>), dim3(blocks, (L.K / 32 + RY * WN - 1) / (RY * WN)), dim3(512), 0, s, B)
    // no more columns than there are
    if (L.K <= 64 && totals) TAD_LONG(1, 1, 2, true);
    else if (L.K <= 64) TAD_LONG(1, 1, 2, false);
    else if (L.K <= 128 && totals) TAD_LONG(1, 2, 2, true);
    else if (L.K <= 128) TAD_LONG(1, 2, 2, false);
    else if (totals) TAD_LONG(2, 2, 4, true);
    else TAD_LONG(2, 2, 4, false);
#undef TAD_LONG
    return hipGetLastError() == hipSuccess ? TAD_OK : TAD_EDEVICE;
}

}  // namespace tad
