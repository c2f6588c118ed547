// Large 32-bit matrix products on the bf16 matrix cores, to 32-bit precision.
//
// A 32-bit number is the sum of three bf16 numbers, x = x1 + x2 + x3 (8 + 8 + 8 bits of the significand, each the nearest to what
// the ones before leave), so x y is the sum of nine products of bf16 numbers, each exact in 32 bits; without x3 y3 it is off by at
// most 2^-32 x y.  v_mfma_f32_32x32x16_bf16 does sixteen times the work of v_mfma_f32_32x32x2f32 per cycle: eight of them take
// half its time.
// x1 y1 is added up by itself (for a single term that is exact), the seven smaller products by themselves, where a rounding counts 2^-7 of one of
// the sum, and after 128 terms both are added to the total on the vector ALU: the instruction does not round its sums to nearest, and long chains
// of it drift (all 4096 terms in one: 4.1e-7 for uniform operands, 1.2e-6 for nearly equal ones; the same additions after every 16 terms, with a
// vector instruction for every second matrix instruction, 4.1e-7 and 840 us).  Error against 64 bits, these and the 32-bit instructions, 4096 x 4096 x 4096:
// operands uniform in -1 .. 1 1.6e-7 / 1.15e-6, in 0 .. 1 1.1e-7 / 8.4e-7, nearly equal ones 1.1e-7 / 8.3e-7, normal times 2^(-20 .. 20) 1.7e-7 / 4.9e-7, one term per sum 2.5e-8 / 2.5e-8 (at most 0.5025 / 0.5 units in
// the last place).  (With six products into one total, uniform operands 1.0e-6 and one term 3.1e-8, 1.3 units.  Two fp16 parts, three products: 375 us, but
// one term is off by up to 8 units; three fp16 parts, six products: 650 us, and a range of 2^40 at most within a tensor.)
//
// Two passes.  k_split_planes (62 us for both operands there, 5.4 TB/s) writes the three parts of an operand fragment by fragment, in the order in which a wavefront
// feeds them to the matrix cores ([16 terms][32 rows][part][lane][8 terms]), with zeros beyond the edges: the product then copies
// contiguous memory to LDS, past the registers, reads LDS without conflicts, and has no edge cases but its stores.  k_split_product: workgroup
// tile 128 x 128, four wavefronts of 64 x 64 (three sums of it are 192 of the 256 registers two wavefronts per SIMD leave each), 24 KB of parts per 16
// terms in two sets; a stage is 32 matrix instructions per wavefront against 12 LDS reads and 6 loads of 16 bytes.
// 805 us, 171 TFLOP/s of 32-bit work, where the 32-bit instructions take 1030 us: 1.37 PFLOP/s of the bf16 cores, whose clock falls to 1.8 GHz under it
// (the same launch on zeros: 602 us at 2.4 GHz, 73 % of the peak).
//
// Parts and their products have to stay normal numbers: the operands are split 2^24 times as large, so that every part of the
// smallest 32-bit number is one and what is lost of a product lies below 2^-174.  That leaves infinities and operands whose
// products reach 2^71: the first pass also finds the largest exponent of either operand, and beyond the safe range the product
// leaves its work to the 32-bit kernel, which is launched behind it and returns at once otherwise.
#include <hip/hip_runtime.h>

#include "launch.h"
#include "profile.h"
#include "split.h"

namespace tad {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float float4s_ __attribute__((ext_vector_type(4)));
typedef float float16s __attribute__((ext_vector_type(16)));
typedef unsigned piece __attribute__((ext_vector_type(4)));   // 16 bytes
typedef const __attribute__((address_space(1))) void *split_global;
typedef __attribute__((address_space(3))) void *split_lds;

// One operand.  turned: element (row, q) at src[q * ld + row], else at src[row * ld + q]; R, Q and ld are multiples of four.
struct SplitOperand {
    const float *src;
    bf16x8 *out;
    int R, Q, ld, turned, row_blocks;
};
struct SplitPass {
    SplitOperand op[2];
    int q_blocks, q_groups;   // fragments along the terms, groups of 16 of them
    int first;                // workgroups of the first operand
    int *seen;                // per workgroup: largest exponent
};

// A wavefront writes four fragments of 32 rows and 16 terms, a workgroup sixteen along the terms: 1 KB of a row.
__global__ __launch_bounds__(256) void k_split_planes(const SplitPass P) {
    __shared__ int red[4];
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const bool second = (int)blockIdx.x >= P.first;
    const SplitOperand &o = P.op[second ? 1 : 0];
    const int id = (int)blockIdx.x - (second ? P.first : 0), rb = id / P.q_groups, group = id - rb * P.q_groups;
    const int row = rb * 32 + (lane & 31);
    int hi = 0;
    // the loads of all four fragments go out before the first of them is used: they share lines of memory
    float v[4][8];
    const int first = group * 16 + wave * 4;
    if (!o.turned) {   // the same for the workgroup
#pragma unroll
        for (int k = 0; k < 4; ++k)
#pragma unroll
            for (int h = 0; h < 2; ++h) {
                const int q = (first + k) * 16 + 8 * (lane >> 5) + 4 * h;
                const bool there = row < o.R && q < o.Q;
                const float4s_ x = *reinterpret_cast<const float4s_ *>(o.src + (there ? (size_t)row * o.ld + q : 0));
#pragma unroll
                for (int e = 0; e < 4; ++e) v[k][4 * h + e] = there ? x[e] : 0.f;
            }
    } else {
#pragma unroll
        for (int k = 0; k < 4; ++k)
#pragma unroll
            for (int e = 0; e < 8; ++e) {
                const int q = (first + k) * 16 + 8 * (lane >> 5) + e;
                const bool there = row < o.R && q < o.Q;
                const float x = o.src[there ? (size_t)q * o.ld + row : 0];
                v[k][e] = there ? x : 0.f;
            }
    }
#pragma unroll
    for (int k = 0; k < 4; ++k) {
        const int qb = first + k;
        if (qb >= P.q_blocks) break;   // the same for the wavefront
        bf16x8 p1, p2, p3;
#pragma unroll
        for (int e = 0; e < 8; ++e) {
            hi = max(hi, (int)((__float_as_uint(v[k][e]) & 0x7fffffffu) >> 23));   // (zero: exponent 0)
            const float sv = v[k][e] * kSplitScale;
            p1[e] = (__bf16)sv;
            const float r1 = sv - (float)p1[e];
            p2[e] = (__bf16)r1;
            p3[e] = (__bf16)(r1 - (float)p2[e]);
        }
        bf16x8 *to = o.out + ((size_t)qb * o.row_blocks + rb) * 192 + lane;
        to[0] = p1;
        to[64] = p2;
        to[128] = p3;
    }
#pragma unroll
    for (int m = 32; m >= 1; m >>= 1) hi = max(hi, __shfl_xor(hi, m, 64));
    if (lane == 0) red[wave] = hi;
    __syncthreads();
    if (threadIdx.x == 0) P.seen[blockIdx.x] = max(max(red[0], red[1]), max(red[2], red[3]));
}

// range[0], range[1]: largest exponent of the first operand, of the second one
__global__ __launch_bounds__(1024) void k_split_range(const int *__restrict__ seen, int first, int total, int *range) {
    __shared__ int red[2][16];
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    int v[2] = {0, 0};
    for (int i = threadIdx.x; i < total; i += 1024) {
        const int hi = seen[i];
        if (i < first) v[0] = max(v[0], hi);
        else v[1] = max(v[1], hi);
    }
#pragma unroll
    for (int q = 0; q < 2; ++q) {
#pragma unroll
        for (int m = 32; m >= 1; m >>= 1) v[q] = max(v[q], __shfl_xor(v[q], m, 64));
        if (lane == 0) red[q][wave] = v[q];
    }
    __syncthreads();
    if (threadIdx.x < 2) {
        int x = red[threadIdx.x][0];
        for (int w = 1; w < 16; ++w) x = max(x, red[threadIdx.x][w]);
        range[threadIdx.x] = x;
    }
}

__device__ __forceinline__ void split_tile(int gm, int gn, int &tm, int &tn) {
    // the dies take workgroups in turn: each gets a contiguous range of tiles, in groups of four tile rows
    const int total = gm * gn;
    int lid = blockIdx.x;
    if (total % 8 == 0) lid = (lid % 8) * (total / 8) + lid / 8;
    const int group = 4 * gn, g0 = (lid / group) * 4, rows = min(4, gm - g0), in = lid - (lid / group) * group;
    tm = g0 + in % rows;
    tn = in / rows;
}

__global__ __launch_bounds__(256, 2) void k_split_product(const piece *__restrict__ a, const piece *__restrict__ b, float *__restrict__ c, int M,
                                                          int N, int q_blocks, int gm, int gn, const int *__restrict__ range) {
    if (!split_in_range(range)) return;   // the same for the whole launch
    constexpr int PA = 4 * 192, PB = 4 * 192, STAGE = PA + PB;   // 16-byte pieces of a stage
    __shared__ piece smem[2 * STAGE];
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6), wm = wave >> 1, wn = wave & 1;
    int tm, tn;
    split_tile(gm, gn, tm, tn);
    // the pieces of a stage are contiguous in either operand and go to LDS as they are
    const piece *pa = a + (size_t)tm * PA + wave * 64 + lane, *pb = b + (size_t)tn * PB + wave * 64 + lane;
    const unsigned next_a = (unsigned)gm * PA, next_b = (unsigned)gn * PB;
    auto load = [&](int set) {
#pragma unroll
        for (int p = 0; p < 6; ++p)
            __builtin_amdgcn_global_load_lds((split_global)(p < 3 ? pa + 256 * p : pb + 256 * (p - 3)), (split_lds)(smem + set * STAGE + wave * 64 + 256 * p), 16, 0, 0);
        pa += next_a;
        pb += next_b;
    };
    const float16s zero = {};
    float16s acc[2][2], large[2][2], small[2][2];
#pragma unroll
    for (int x = 0; x < 2; ++x)
#pragma unroll
        for (int y = 0; y < 2; ++y) acc[x][y] = large[x][y] = small[x][y] = zero;
    const int fa = wm * 2 * 192 + lane, fb = PA + wn * 2 * 192 + lane;
    constexpr float back = 1.f / (kSplitScale * kSplitScale);
    auto step = [&](int t, int set) {
        // stage t is in LDS, and nobody reads stage t - 1 any more
        __builtin_amdgcn_sched_barrier(0);
        asm volatile("" ::: "memory");
        __builtin_amdgcn_s_waitcnt(0x0070);   // vmcnt(0), lgkmcnt(0)
        __builtin_amdgcn_s_barrier();
        asm volatile("" ::: "memory");
        if (t + 1 < q_blocks) load(set ^ 1);   // the same for the whole workgroup
        const bf16x8 *S = reinterpret_cast<const bf16x8 *>(smem) + set * STAGE;
        bf16x8 av[2][3], bv[2][3];
#pragma unroll
        for (int y = 0; y < 2; ++y)
#pragma unroll
            for (int s = 0; s < 3; ++s) bv[y][s] = S[fb + y * 192 + s * 64];
#pragma unroll
        for (int s = 0; s < 3; ++s) av[0][s] = S[fa + s * 64];
#pragma unroll
        for (int x = 0; x < 2; ++x) {
            if (x == 0) {
#pragma unroll
                for (int s = 0; s < 3; ++s) av[1][s] = S[fa + 192 + s * 64];
            }
            __builtin_amdgcn_sched_barrier(0);
            // two results in turn: an instruction does not wait for the one before it
            auto mul = [&](int i, int j, float16s(&sum)[2]) {
#pragma unroll
                for (int y = 0; y < 2; ++y) sum[y] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(av[x][i], bv[y][j], sum[y], 0, 0, 0);
            };
            mul(2, 1, small[x]);   // the smallest products first
            mul(0, 0, large[x]);
            mul(1, 2, small[x]);
            mul(2, 0, small[x]);
            mul(0, 2, small[x]);
            mul(1, 1, small[x]);
            mul(1, 0, small[x]);
            mul(0, 1, small[x]);
            __builtin_amdgcn_sched_barrier(0);
        }
    };
    auto flush = [&] {
#pragma unroll
        for (int x = 0; x < 2; ++x)
#pragma unroll
            for (int y = 0; y < 2; ++y) {
                acc[x][y] += large[x][y] * back;
                acc[x][y] += small[x][y] * back;
                large[x][y] = small[x][y] = zero;
            }
    };
    load(0);
    int t = 0;
    for (; t + kSplitChain <= q_blocks; t += kSplitChain) {
#pragma unroll 1
        for (int u = 0; u < kSplitChain; u += 2) {
            step(t + u, 0);
            step(t + u + 1, 1);
        }
        flush();
    }
    for (; t < q_blocks; ++t) step(t, t & 1);
    flush();
    const int m0 = tm * 128 + wm * 64 + 4 * (lane >> 5), n0 = tn * 128 + wn * 64 + (lane & 31);
#pragma unroll
    for (int x = 0; x < 2; ++x)
#pragma unroll
        for (int y = 0; y < 2; ++y)
#pragma unroll
            for (int r = 0; r < 16; ++r) {
                const int m = m0 + x * 32 + 8 * (r >> 2) + (r & 3), n = n0 + y * 32;
                if (m < M && n < N) c[(size_t)m * N + n] = acc[x][y][r];
            }
}

int split_product(const GemmDesc &g, const float *a, const float *b, float *c, void *ws, const int **range_out, hipStream_t s) {
    const SplitGeom q = split_geom(g.M, g.N, g.Kc);
    char *w = static_cast<char *>(ws);
    int *const range = reinterpret_cast<int *>(w);
    bf16x8 *const pa = reinterpret_cast<bf16x8 *>(w + q.a_offset), *const pb = reinterpret_cast<bf16x8 *>(w + q.b_offset);
    SplitPass P;
    P.q_blocks = q.q_blocks;
    P.q_groups = (q.q_blocks + 15) / 16;
    P.op[0] = SplitOperand{a, pa, g.M, g.Kc, g.lda, g.at, q.gm * 4};
    P.op[1] = SplitOperand{b, pb, g.N, g.Kc, g.ldb, !g.bt, q.gn * 4};
    P.first = P.op[0].row_blocks * P.q_groups;
    const int total = P.first + P.op[1].row_blocks * P.q_groups;
    P.seen = reinterpret_cast<int *>(w + 256);
    TAD_LAUNCH("k_split_planes", k_split_planes, dim3(total), dim3(256), 0, s, P);
    if (hipGetLastError() != hipSuccess) return TAD_EDEVICE;
    TAD_LAUNCH("k_split_range", k_split_range, dim3(1), dim3(1024), 0, s, (const int *)P.seen, P.first, total, range);
    if (hipGetLastError() != hipSuccess) return TAD_EDEVICE;
    TAD_LAUNCH("k_split_product", k_split_product, dim3(q.gm * q.gn), dim3(256), 0, s, reinterpret_cast<const piece *>(pa),
               reinterpret_cast<const piece *>(pb), c, g.M, g.N, q.q_blocks, q.gm, q.gn, (const int *)range);
    *range_out = range;
    return hipGetLastError() == hipSuccess ? TAD_OK : TAD_EDEVICE;
}

}  // namespace tad
