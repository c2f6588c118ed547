// Worked expression with a long summed index (K a multiple of 32, fp32): the contraction over k is a
// genuine dense matrix product, so it runs on the matrix cores (v_mfma_f32_32x32x2f32).
//
//   forward   s_ij = |a_i|^2 + |b_j|^2 + 2 a_i . b_j        (expanded square; a . b^T on MFMA)
//             f_ij = exp(-(c_ii s_ij + D_i)),  D_i = sum_k d_{i+k}^3
//   backward  G_ij = df_ij f_ij
//             P = G b        (I x K, contraction over the collapsed kernel coordinate j, split in chunks)
//             T = (c G)^T a  (J x K, contraction over the collapsed kernel coordinate i, split in chunks)
//             r_i = sum_j G_ij, Q_i = sum_j G_ij |b_j|^2, t_j = sum_i c_ii G_ij   (accumulated while G is staged)
//             da_ik = -2 c_ii (a_ik r_i + P_ik)      db_jk = -2 (T_jk + b_jk t_j)
//             dc_ii = -(|a_i|^2 r_i + 2 sum_k a_ik P_ik + Q_i)      dd_m = -3 d_m^2 sum_{i in window(m)} r_i
// All partial results are combined in a fixed order (no atomics).
//
// MFMA operand layout used below (wave64): A operand lane l = A[m = l % 32][k = l / 32],
// B operand lane l = B[k = l / 32][n = l % 32], result register r of lane l = D[8 (r / 4) + 4 (l / 32) + r % 4][l % 32].
#include <hip/hip_runtime.h>

#include <algorithm>

#include "launch.h"
#include "plan_dev.h"
#include "profile.h"
#include "launch_geom.h"
#include "mfma_split.h"

namespace tad {

typedef float float4v __attribute__((ext_vector_type(4)));
typedef float float16v __attribute__((ext_vector_type(16)));

constexpr float kLog2eM = 1.4426950408889634f;

template <int CTRL, int ROW_MASK>
__device__ __forceinline__ float dpp_add_m(float v) {
    int t = __builtin_amdgcn_update_dpp(0, __float_as_int(v), CTRL, ROW_MASK, 0xf, ROW_MASK == 0xf);
    return v + __int_as_float(t);
}
__device__ __forceinline__ float wave_sum63m(float v) {   // total valid in lane 63
    v = dpp_add_m<0x111, 0xf>(v);
    v = dpp_add_m<0x112, 0xf>(v);
    v = dpp_add_m<0x114, 0xf>(v);
    v = dpp_add_m<0x118, 0xf>(v);
    v = dpp_add_m<0x142, 0xa>(v);
    v = dpp_add_m<0x143, 0xc>(v);
    return v;
}

__device__ __forceinline__ int acc_row(int r, int lane) { return 8 * (r >> 2) + 4 * (lane >> 5) + (r & 3); }

// ---------------------------------------------------------------------------------------------
// per-row and per-column quantities: rowv[i] = {|a_i|^2, -log2e c_ii, -log2e D_i, c_ii}, nb[j] = |b_j|^2
// one wave per row
// ---------------------------------------------------------------------------------------------
__global__ __launch_bounds__(256) void k_mfma_prep(const float *__restrict__ a, const float *__restrict__ b,
                                                   const float *__restrict__ c, const float *__restrict__ d,
                                                   float *__restrict__ rowv, float *__restrict__ nb, int I, int J,
                                                   int K, int c_ld) {
    const int lane = threadIdx.x & 63;
    const int row = blockIdx.x * 4 + (threadIdx.x >> 6);
    if (row < I) {
        float na = 0.f, D = 0.f;
        for (int k = lane; k < K; k += 64) {
            const float av = a[(size_t)row * K + k], dv = d[row + k];
            na = fmaf(av, av, na);
            D = fmaf(dv * dv, dv, D);
        }
        na = wave_sum63m(na);
        D = wave_sum63m(D);
        if (lane == 63) {
            const float cv = c[(size_t)row * c_ld + row];
            rowv[row * 4 + 0] = na;
            rowv[row * 4 + 1] = -kLog2eM * cv;
            rowv[row * 4 + 2] = -kLog2eM * D;
            rowv[row * 4 + 3] = cv;
        }
    } else if (row - I < J) {
        const int j = row - I;
        float s = 0.f;
        for (int k = lane; k < K; k += 64) {
            const float bv = b[(size_t)j * K + k];
            s = fmaf(bv, bv, s);
        }
        s = wave_sum63m(s);
        if (lane == 63) nb[j] = s;
    }
}

// ---------------------------------------------------------------------------------------------
// forward: block tile 64 NX x 64 NX, 2 x 2 waves of 32 NX x 32 NX, k tile 32, global -> register -> LDS staging.  NX = 1: four wavefronts
// per SIMD, which wait for their barriers, loads and stores in turn, and tiles that fill the chip sooner; NX = 2: two, half the LDS reads per
// matrix instruction.  Forward passes with 128 x 128 / 64 x 64: 1024 x 1024 x 256 26 / 11 us, 3000 x 300 x 224 24 / 11, 3000 x 3000 x 256 66 / 50 (a second round
// of 64 tiles), 130 x 32636 x 288 54.0 / 52.0 (half empty), 4096 x 4096 x 64 34.1 / 31.5, x 128 50.4 / 47.8, x 256 81.0 / 83.6, x 512 146 / 153,
// 4096 x 2048 x 512 78.1 / 81.3, 8192 x 4096 x 256 155 / 162: the large tiles from K = 256 on, where they and their last round are nearly full.
// ---------------------------------------------------------------------------------------------
constexpr int MF_KT = 32;
constexpr int MF_LD = 33;   // odd row stride: conflict-free ds_read_b32 of [row][k] tiles

static bool large_forward_tiles(int64_t I, int64_t J, int64_t K) {
    const int64_t tiles = ((I + 127) / 128) * ((J + 127) / 128), last = (tiles - 1) % 512 + 1;   // 512 at once
    return K >= 256 && last >= 480 && 16 * I * J >= 15 * tiles * 128 * 128;
}

template <int NX>
__device__ __forceinline__ void mfma_forward_tile(const float *__restrict__ a, const float *__restrict__ b, const float *__restrict__ rowv,
                                                  const float *__restrict__ nb, float *__restrict__ f, int I, int J, int K) {
    constexpr int T = 64 * NX, W = 32 * NX, P = 2 * NX;
    constexpr int LO = W + 2;                     // row stride of the output stage
    constexpr int TILES = 2 * T * MF_LD, STAGE = 4 * 32 * LO;
    __shared__ float smem[TILES > STAGE ? TILES : STAGE];   // A tile then B tile; reused as the output stage in the epilogue
    __shared__ float rv[T][4];
    float (*As)[MF_LD] = reinterpret_cast<float (*)[MF_LD]>(smem);
    float (*Bs)[MF_LD] = reinterpret_cast<float (*)[MF_LD]>(smem + T * MF_LD);
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int wm = wave >> 1, wn = wave & 1;
    const int i0 = blockIdx.y * T, j0 = blockIdx.x * T;
    if (tid < T) {
        const int i = i0 + tid;
#pragma unroll
        for (int q = 0; q < 4; ++q) rv[tid][q] = i < I ? rowv[i * 4 + q] : 0.f;
    }
    float16v acc[NX][NX];
#pragma unroll
    for (int x = 0; x < NX; ++x)
#pragma unroll
        for (int y = 0; y < NX; ++y)
#pragma unroll
            for (int r = 0; r < 16; ++r) acc[x][y][r] = 0.f;
    float4v ra[P], rb[P];
    auto gload = [&](int k0) {
#pragma unroll
        for (int p = 0; p < P; ++p) {
            const int idx = tid + 256 * p, row = idx >> 3, kq = idx & 7;
            // (rows beyond the edge repeat the last one: their results are not stored)
            ra[p] = *reinterpret_cast<const float4v *>(a + (size_t)min(i0 + row, I - 1) * K + k0 + 4 * kq);
            rb[p] = *reinterpret_cast<const float4v *>(b + (size_t)min(j0 + row, J - 1) * K + k0 + 4 * kq);
        }
    };
    gload(0);
    const int mrow = lane & 31, kof = lane >> 5;
    for (int k0 = 0; k0 < K; k0 += MF_KT) {
#pragma unroll
        for (int p = 0; p < P; ++p) {
            const int idx = tid + 256 * p, row = idx >> 3, kq = idx & 7;
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                As[row][4 * kq + q] = ra[p][q];
                Bs[row][4 * kq + q] = rb[p][q];
            }
        }
        __syncthreads();
        if (k0 + MF_KT < K) gload(k0 + MF_KT);
        // the operands of step ks + 1 are read from LDS before the MFMAs of step ks are issued
        const float *ap = &As[wm * W + mrow][kof], *bp = &Bs[wn * W + mrow][kof];
        float fa[NX], fb[NX];
#pragma unroll
        for (int x = 0; x < NX; ++x) { fa[x] = ap[32 * x * MF_LD]; fb[x] = bp[32 * x * MF_LD]; }
#pragma unroll
        for (int ks = 0; ks < MF_KT / 2; ++ks) {
            float na[NX] = {}, nf[NX] = {};
            if (ks + 1 < MF_KT / 2) {
#pragma unroll
                for (int x = 0; x < NX; ++x) { na[x] = ap[32 * x * MF_LD + 2 * ks + 2]; nf[x] = bp[32 * x * MF_LD + 2 * ks + 2]; }
            }
            __builtin_amdgcn_sched_barrier(0);
#pragma unroll
            for (int x = 0; x < NX; ++x)
#pragma unroll
                for (int y = 0; y < NX; ++y) acc[x][y] = __builtin_amdgcn_mfma_f32_32x32x2f32(fa[x], fb[y], acc[x][y], 0, 0, 0);
            __builtin_amdgcn_sched_barrier(0);
#pragma unroll
            for (int x = 0; x < NX; ++x) { fa[x] = na[x]; fb[x] = nf[x]; }
        }
        __syncthreads();
    }
    // epilogue: f = exp2(c' (|a|^2 + |b|^2 + 2 a.b) + D').  Each wave stages 32 x W results at a time in its own
    // quarter of the tile memory and writes them as 16-byte stores, whole rows of the wave's tile.
    // (the last barrier of the loop guarantees that nobody still reads the tiles)
    constexpr int ROWS = 256 / W;                 // rows per store of the wavefront
    float *stage = smem + wave * (32 * LO);
#pragma unroll
    for (int x = 0; x < NX; ++x) {
#pragma unroll
        for (int y = 0; y < NX; ++y) {
            const int j = j0 + wn * W + 32 * y + mrow;
            const float nbj = j < J ? nb[j] : 0.f;
#pragma unroll
            for (int r = 0; r < 16; ++r) {
                const int mloc = acc_row(r, lane), m = wm * W + 32 * x + mloc;
                const float s = rv[m][0] + nbj + 2.f * acc[x][y][r];
                stage[mloc * LO + 32 * y + mrow] = __builtin_amdgcn_exp2f(fmaf(rv[m][1], s, rv[m][2]));
            }
        }
        // the wave reads back only what it wrote itself: no barrier needed, LDS operations of a wave are ordered
#pragma unroll
        for (int it = 0; it < 32 / ROWS; ++it) {
            const int rl = it * ROWS + lane / (W / 4), c = lane % (W / 4) * 4;
            const int i = i0 + wm * W + 32 * x + rl, j = j0 + wn * W + c;
            if (i < I && j < J) {   // J % 4 == 0: the four columns exist together
                const float4v v = {stage[rl * LO + c], stage[rl * LO + c + 1], stage[rl * LO + c + 2], stage[rl * LO + c + 3]};
                *reinterpret_cast<float4v *>(f + (size_t)i * J + j) = v;
            }
        }
    }
}

__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(4, 4))) void k_mfma_forward(const float *__restrict__ a, const float *__restrict__ b,
                                                      const float *__restrict__ rowv, const float *__restrict__ nb,
                                                      float *__restrict__ f, int I, int J, int K, const int *__restrict__ redo) {
    if (redo && !*redo) return;   // done on the bf16 matrix cores
    mfma_forward_tile<1>(a, b, rowv, nb, f, I, J, K);
}
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(2, 2))) void k_mfma_forward_large(const float *__restrict__ a, const float *__restrict__ b,
                                                      const float *__restrict__ rowv, const float *__restrict__ nb,
                                                      float *__restrict__ f, int I, int J, int K, const int *__restrict__ redo) {
    if (redo && !*redo) return;
    mfma_forward_tile<2>(a, b, rowv, nb, f, I, J, K);
}

// ---------------------------------------------------------------------------------------------
// backward contractions.  Block tile 64 (M) x 256 (N = k), 2 x 4 waves of 32 x 64, contraction tile 32 (four waves of 64 x 64 are two per
// SIMD instead of four: 93.0 us instead of 89.8 for 4096 x 4096 x 256, not transposed; the other one the same).
//   TRANS_A = false:  M = i, contraction over j in [cs, ce):  A[m][kk] = df f            B[kk][n] = b[j][k]
//   TRANS_A = true:   M = j, contraction over i in [cs, ce):  A[m][kk] = c_ii df f (read transposed), B[kk][n] = a[i][k]
// out[(split * Mtot + m) * K + n]
// ---------------------------------------------------------------------------------------------
// While G is staged, the same thread keeps meeting the same rows (TRANS_A = false) or the same columns
// (TRANS_A = true), so the plain sums over the collapsed index are accumulated on the side, those of a chain in 32 bits, all of
// them in 64 (in 32 bits they drift with the length of the pieces: dc of 8192 x 8192 x 256 1.6e-7, now 7.5e-8; eight pieces in 32 bits 1.1e-7):
//   TRANS_A = false:  sums[(split * 2 + 0) * I + i] = sum_j G_ij,  sums[(split * 2 + 1) * I + i] = sum_j G_ij |b_j|^2
//   TRANS_A = true:   sums[split * J + j] = sum_i c_ii G_ij
struct MfmaTiles {
    float a[64 * MF_LD], b[32][256];
    double red[8][64], side[4][512];
};
// The matrix instructions add two terms at a time, and every addition rounds the chain's sum: an eighth of the sum, at most 256 terms, is added up by itself
// and then to the total (TOTALS; not needed where the pieces are no longer than that).  Error of da against 64 bits with one chain to a piece of up to the
// whole sum / with totals / with eight pieces of one chain, 4096 x 4096 x 640: 4.2e-7 / 2.2e-7 / 3.0e-7; a sum of 8192 terms of one sign 6.0e-7 / 6.4e-8 / 1.6e-7.
// All four gradients 471 / 479 / 536 us (4096 x 4096 x 640), 256 x 1024 x 64 16.7 / 17.5 / 33.5.
template <bool TRANS_A, bool TOTALS>
__device__ __forceinline__ void mfma_contraction(MfmaTiles &S, int tile, int split, const float *__restrict__ f, const float *__restrict__ df,
                                                 const float *__restrict__ bmat, const float *__restrict__ rowv, const float *__restrict__ nb,
                                                 float *__restrict__ out, float *__restrict__ sums, int I, int J, int K, int chunk) {
    float (*const As)[TRANS_A ? 64 : MF_LD] = reinterpret_cast<float (*)[TRANS_A ? 64 : MF_LD]>(S.a);
    float (*const Bs)[256] = S.b;
    double (*const tred)[64] = S.red;
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6), wm = wave & 1, wn = wave >> 1;
    const int Mtot = TRANS_A ? J : I, Ctot = TRANS_A ? I : J;
    const int m0 = tile * 64, n0 = blockIdx.y * 256;
    const int cs = split * chunk, ce = min(Ctot, cs + chunk);
    const int chain = TOTALS ? mfma_chain(Ctot) : chunk;
    const float16v zero16 = {};
    float16v acc[2] = {zero16, zero16}, total[2] = {zero16, zero16};
    float4v ga, gb[4];
    // what the loads of G bring in; the products and the sums on the side are formed one tile later, when the
    // tile is staged, so that nothing waits for these loads before the matrix instructions of the current tile
    float4v rdf, rf, rnv;
    float rc;
    const float4v zero4 = {0.f, 0.f, 0.f, 0.f};
    float sr = 0.f, sq = 0.f;   // TRANS_A = false: row sums of the thread's row, of one chain
    float4v st = zero4;         // TRANS_A = true: column sums of the thread's four columns
#pragma unroll
    for (int e = 0; e < 4; ++e) S.side[e][tid] = 0.0;   // ... and of those before, in LDS: the registers are taken
    // the four elements of G of the thread: i = m0 + g_row, j = c0 + 4 g_quad, or (TRANS_A) i = c0 + g_row, j = m0 + 4 g_quad
    const int g_row = TRANS_A ? tid >> 4 : tid >> 3, g_quad = TRANS_A ? tid & 15 : tid & 7;
    auto gload = [&](int c0) {
        rdf = zero4; rf = zero4; rnv = zero4; rc = 0.f;
        const int i = (TRANS_A ? c0 : m0) + g_row, j = (TRANS_A ? m0 : c0) + 4 * g_quad;
        if (i < (TRANS_A ? ce : I) && j < (TRANS_A ? J : ce)) {
            const size_t off = (size_t)i * J + j;
            rdf = *reinterpret_cast<const float4v *>(df + off);
            rf = *reinterpret_cast<const float4v *>(f + off);
            if (TRANS_A) rc = rowv[i * 4 + 3];
            else rnv = *reinterpret_cast<const float4v *>(nb + j);
        }
#pragma unroll
        for (int p = 0; p < 4; ++p) {
            const int cc = c0 + wave + 8 * p, n = n0 + 4 * lane;
            gb[p] = (cc < ce && n < K) ? *reinterpret_cast<const float4v *>(bmat + (size_t)cc * K + n) : zero4;
        }
    };
    auto gprep = [&]() {   // G of the loaded tile and its plain sums (zeros where nothing was loaded)
        if (!TRANS_A) {
            ga = rdf * rf;
            sr += (ga[0] + ga[1]) + (ga[2] + ga[3]);
            sq += (ga[0] * rnv[0] + ga[1] * rnv[1]) + (ga[2] * rnv[2] + ga[3] * rnv[3]);
        } else {
            ga = rdf * rf * rc;
            st += ga;
        }
    };
    gload(cs);
    const int mrow = lane & 31, kof = lane >> 5;
    auto stage = [&](int c0) {
        gprep();
        if (!TRANS_A) {
#pragma unroll
            for (int e = 0; e < 4; ++e) As[g_row][4 * g_quad + e] = ga[e];
        } else {
            *reinterpret_cast<float4v *>(&As[g_row][4 * g_quad]) = ga;
        }
#pragma unroll
        for (int p = 0; p < 4; ++p) *reinterpret_cast<float4v *>(&Bs[wave + 8 * p][4 * lane]) = gb[p];
        __syncthreads();
        if (c0 + MF_KT < ce) gload(c0 + MF_KT);
        auto afrag = [&](int kk) -> float { return TRANS_A ? As[kk + kof][32 * wm + mrow] : As[32 * wm + mrow][kk + kof]; };
        // the operands of step ks + 1 are read from LDS before the MFMAs of step ks are issued
        float a0 = afrag(0), b0 = Bs[kof][wn * 64 + mrow], b1 = Bs[kof][wn * 64 + 32 + mrow];
#pragma unroll
        for (int ks = 0; ks < MF_KT / 2; ++ks) {
            float na0 = 0.f, nb0 = 0.f, nb1 = 0.f;
            if (ks + 1 < MF_KT / 2) {
                na0 = afrag(2 * ks + 2);
                nb0 = Bs[2 * ks + 2 + kof][wn * 64 + mrow];
                nb1 = Bs[2 * ks + 2 + kof][wn * 64 + 32 + mrow];
            }
            __builtin_amdgcn_sched_barrier(0);
            acc[0] = __builtin_amdgcn_mfma_f32_32x32x2f32(a0, b0, acc[0], 0, 0, 0);
            acc[1] = __builtin_amdgcn_mfma_f32_32x32x2f32(a0, b1, acc[1], 0, 0, 0);
            __builtin_amdgcn_sched_barrier(0);
            a0 = na0; b0 = nb0; b1 = nb1;
        }
        __syncthreads();
    };
#pragma unroll 1
    for (int first = cs; first < ce; first += chain) {
        acc[0] = acc[1] = zero16;
        const int end = min(ce, first + chain);
#pragma unroll 1
        for (int c0 = first; c0 < end; c0 += MF_KT) stage(c0);
        if (TRANS_A) {
#pragma unroll
            for (int e = 0; e < 4; ++e) S.side[e][tid] += (double)st[e];
            st = zero4;
        } else {
            S.side[0][tid] += (double)sr;
            S.side[1][tid] += (double)sq;
            sr = sq = 0.f;
        }
        if constexpr (!TOTALS) break;
#pragma unroll
        for (int x = 0; x < 2; ++x) total[x] += acc[x];
    }
    int late = tid;   // places of the results from the thread's number again: kept through the loop they would not fit in registers
    asm volatile("" : "+v"(late));
#pragma unroll
    for (int tn = 0; tn < 2; ++tn) {
        const int n = n0 + wn * 64 + tn * 32 + (late & 31);
#pragma unroll
        for (int r = 0; r < 16; ++r) {
            const int m = m0 + wm * 32 + acc_row(r, late & 63);
            if (m < Mtot && n < K) out[((size_t)split * Mtot + m) * K + n] = (TOTALS ? total : acc)[tn][r];
        }
    }
    if (blockIdx.y != 0) return;
    double tr = S.side[0][tid], tq = S.side[1][tid], tt[4];   // (its own)
    if (!TRANS_A) {
        // eight consecutive lanes share a row: add them in a fixed order
#pragma unroll
        for (int m = 1; m <= 4; m <<= 1) {
            tr += __shfl_xor(tr, m, 64);
            tq += __shfl_xor(tq, m, 64);
        }
        const int i = m0 + g_row;
        if (g_quad == 0 && i < I) {
            sums[((size_t)split * 2 + 0) * I + i] = (float)tr;
            sums[((size_t)split * 2 + 1) * I + i] = (float)tq;
        }
    } else {
        // lanes q, q+16, q+32, q+48 of every wave hold the same four columns: add within the wave, then the waves
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            tt[e] = S.side[e][tid];
            tt[e] += __shfl_xor(tt[e], 16, 64);
            tt[e] += __shfl_xor(tt[e], 32, 64);
        }
        if (lane < 16)
#pragma unroll
            for (int e = 0; e < 4; ++e) tred[wave][lane * 4 + e] = tt[e];
        __syncthreads();
        if (tid < 64) {
            const int j = m0 + tid;
            if (j < J) sums[(size_t)split * J + j] = (float)(((tred[0][tid] + tred[1][tid]) + (tred[2][tid] + tred[3][tid])) + ((tred[4][tid] + tred[5][tid]) + (tred[6][tid] + tred[7][tid])));
        }
    }
}

// Both contractions in one launch, tiles of rows i, then tiles of rows j: small ones fill the chip together.
struct MfmaSide {
    const float *mat;
    float *out, *sums;
    int chunk;
};
template <bool TOTALS>
__global__ __launch_bounds__(512, 4) void k_mfma_backward(const float *__restrict__ f, const float *__restrict__ df, const float *__restrict__ rowv,
                                                          const float *__restrict__ nb, const MfmaSide P, const MfmaSide T, int I, int J, int K, int first,
                                                          int n_j, int n_i, const int *__restrict__ redo) {
    if (redo && !*redo) return;   // done on the bf16 matrix cores
    __shared__ __attribute__((aligned(16))) MfmaTiles S;
    const int id = blockIdx.x, second = id - first;   // (neighbours share a tile of rows)
    if (id < first) mfma_contraction<false, TOTALS>(S, id / n_j, id % n_j, f, df, P.mat, rowv, nb, P.out, P.sums, I, J, K, P.chunk);
    else mfma_contraction<true, TOTALS>(S, second / n_i, second % n_i, f, df, T.mat, rowv, nb, T.out, T.sums, I, J, K, T.chunk);
}

// ---------------------------------------------------------------------------------------------
// finishing, in one launch: rows i (da, dc_ii and the zeros of that row of dc), rows j (db), dd, rows of dc beyond I; one wavefront per output row, a
// lane owns four consecutive k.  Fixed summation order, pieces added in 64 bits (up to 64 of them: in 32 bits da of 64 x 2048 x 32, terms of one sign, was off by
// 1.1e-7, so by 2.5e-8; 4096 x 4096 x 256 120 -> 120.5 us).  The zeros (64 MB at 4096 x 4096) go out while the others wait for their partial sums.
// ---------------------------------------------------------------------------------------------
struct MfmaFinish {
    const float *a, *b, *d, *rowv, *P, *T, *rowp, *colp;
    float *da, *db, *dc, *dd;
    long long n_c;             // elements of c
    int I, J, K, c_ld, n_d;
    int n_j, n_i;              // pieces of the sums over j and over i
    int rows, cols, window;    // workgroups for rows i, for rows j, for dd; the rest: zeros beyond row I
};
// to[0 .. n) = 0, but to[at] = v; 16-byte stores whatever the alignment of the row
__device__ __forceinline__ void mfma_zeros(float *to, int n, int at, float v, int lane) {
    const int head = min(n, (int)((16 - (reinterpret_cast<uintptr_t>(to) & 15)) & 15) / 4), body = (n - head) / 4;
    if (lane < head) to[lane] = lane == at ? v : 0.f;
    for (int q = lane; q < body; q += 64) {
        const int first = head + 4 * q;
        float4v z;
#pragma unroll
        for (int e = 0; e < 4; ++e) z[e] = first + e == at ? v : 0.f;
        __builtin_nontemporal_store(z, reinterpret_cast<float4v *>(to + first));
    }
    const int rest = head + 4 * body + lane;
    if (rest < n) to[rest] = rest == at ? v : 0.f;
}
constexpr int kZeroPiece = 4096;   // floats of a wavefront
__global__ __launch_bounds__(256) void k_mfma_finish(const MfmaFinish F, const FlatFeas feas, const FlatLevel win, int iy, int iz) {
    const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6, I = F.I, J = F.J, K = F.K;
    int block = blockIdx.x;
    if (block < F.rows) {
        const int i = block * 4 + wv;
        if (i >= I) return;
        double r = 0.0, Q = 0.0;
#pragma unroll 4
        for (int s = 0; s < F.n_j; ++s) {
            r += (double)F.rowp[((size_t)s * 2 + 0) * I + i];
            Q += (double)F.rowp[((size_t)s * 2 + 1) * I + i];
        }
        const double ci = (double)F.rowv[i * 4 + 3], na = (double)F.rowv[i * 4 + 0];
        float cross = 0.f;
        if (F.da || F.dc)
            for (int k = lane * 4; k < K; k += 256) {
                double P[4] = {};
#pragma unroll 4
                for (int s = 0; s < F.n_j; ++s) {
                    const float4v v = *reinterpret_cast<const float4v *>(F.P + ((size_t)s * I + i) * K + k);
#pragma unroll
                    for (int e = 0; e < 4; ++e) P[e] += (double)v[e];
                }
                const float4v av = *reinterpret_cast<const float4v *>(F.a + (size_t)i * K + k);
                if (F.da) {
                    float4v o;
#pragma unroll
                    for (int e = 0; e < 4; ++e) o[e] = (float)(-2.0 * ci * ((double)av[e] * r + P[e]));
                    *reinterpret_cast<float4v *>(F.da + (size_t)i * K + k) = o;
                }
                cross += (av[0] * (float)P[0] + av[1] * (float)P[1]) + (av[2] * (float)P[2] + av[3] * (float)P[3]);
            }
        if (!F.dc) return;
        cross = wave_sum63m(cross);
        const float total = __int_as_float(__builtin_amdgcn_readlane(__float_as_int(cross), 63));
        mfma_zeros(F.dc + (size_t)i * F.c_ld, F.c_ld, i, (float)(-(na * r + 2.0 * (double)total + Q)), lane);
        return;
    }
    block -= F.rows;
    if (block < F.cols) {
        const int j = block * 4 + wv;
        if (j >= J) return;
        double t = 0.0;
#pragma unroll 4
        for (int s = 0; s < F.n_i; ++s) t += (double)F.colp[(size_t)s * J + j];
        for (int k = lane * 4; k < K; k += 256) {
            double T[4] = {};
#pragma unroll 4
            for (int s = 0; s < F.n_i; ++s) {
                const float4v v = *reinterpret_cast<const float4v *>(F.T + ((size_t)s * J + j) * K + k);
#pragma unroll
                for (int e = 0; e < 4; ++e) T[e] += (double)v[e];
            }
            const float4v bv = *reinterpret_cast<const float4v *>(F.b + (size_t)j * K + k);
            float4v o;
#pragma unroll
            for (int e = 0; e < 4; ++e) o[e] = (float)(-2.0 * (T[e] + (double)bv[e] * t));
            *reinterpret_cast<float4v *>(F.db + (size_t)j * K + k) = o;
        }
        return;
    }
    block -= F.cols;
    if (block < F.window) {
        // dd_m = -3 d_m^2 sum_{i in window(m)} r_i; window and masks from the plan of d
        const int m = block * 4 + wv;
        if (m >= F.n_d) return;
        const int32_t y[3] = {m, 0, 0};
        float s = 0.f;
        const bool ok = flat_feasible(feas, y);
        if (ok) {
            int32_t lo, hi;
            flat_bounds(win, y, lo, hi);
            for (int32_t w = lo + lane; w <= hi; w += 64) {
                double r = 0.0;
#pragma unroll 4
                for (int p = 0; p < F.n_j; ++p) r += (double)F.rowp[(size_t)p * 2 * I + iy * y[0] + iz * w];
                s += (float)r;
            }
        }
        s = wave_sum63m(s);
        if (lane == 63) {
            const float dm = F.d[m];
            F.dd[m] = ok ? -3.f * dm * dm * s : 0.f;
        }
        return;
    }
    const long long from = (long long)I * F.c_ld + ((long long)(block - F.window) * 4 + wv) * kZeroPiece;
    if (from < F.n_c) mfma_zeros(F.dc + from, (int)min((long long)kZeroPiece, F.n_c - from), -1, 0.f, lane);
}

// ---------------------------------------------------------------------------------------------
// host side
// ---------------------------------------------------------------------------------------------
struct MfmaWs {
    float *rowv, *nb, *partial, *sums;
};
static MfmaWs carve_mfma(void *ws, int64_t I, int64_t J, int64_t K) {
    MfmaWs w;
    char *p = static_cast<char *>(ws);
    auto take = [&](size_t bytes) { float *r = reinterpret_cast<float *>(p); p += align256(bytes); return r; };
    w.rowv = take((size_t)I * 16);
    w.nb = take((size_t)J * 4);
    w.partial = take((size_t)kMfmaSplit * (I + J) * K * 4);
    w.sums = take((size_t)kMfmaSplit * (2 * I + J) * 4);
    return w;
}

static int prep(const tad_plan &pl, const void *const *args, const MfmaWs &w, hipStream_t s) {
    const int I = (int)pl.fast.I, J = (int)pl.fast.J, K = (int)pl.fast.K;
    TAD_LAUNCH("k_mfma_prep", k_mfma_prep, dim3((I + J + 3) / 4), dim3(256), 0, s, (const float *)args[0],
               (const float *)args[1], (const float *)args[2], (const float *)args[3], w.rowv, w.nb, I, J, K,
               (int)pl.fast.c_ld);
    return hipGetLastError() == hipSuccess ? TAD_OK : TAD_EDEVICE;
}

// ---------------------------------------------------------------------------------------------
// The same forward pass in the direct form  s_ij = sum_k (a_ik + b_jk)^2  on the vector ALUs (one add and one fused
// multiply-add per (i, j, k): 2 I J K lane operations): block tile 64 x 64, a
// thread owns 4 x 4 results, k tile 32 through LDS.  Kept to measure the expanded form against (TAD_PLAN_DIRECT_FORM).
// ---------------------------------------------------------------------------------------------
__global__ __launch_bounds__(256) void k_worked_forward_direct(const float *__restrict__ a, const float *__restrict__ b,
                                                               const float *__restrict__ rowv, float *__restrict__ f,
                                                               int I, int J, int K) {
    __shared__ __attribute__((aligned(16))) float As[32][68];   // [k][row]
    __shared__ __attribute__((aligned(16))) float Bs[32][68];   // [k][row]: a thread reads four consecutive rows as one 16-byte load
    const int tid = threadIdx.x, tx = tid & 15, ty = tid >> 4;
    const int i0 = blockIdx.y * 64, j0 = blockIdx.x * 64;
    float acc[4][4];
#pragma unroll
    for (int x = 0; x < 4; ++x)
#pragma unroll
        for (int y = 0; y < 4; ++y) acc[x][y] = 0.f;
    const float4v zero4 = {0.f, 0.f, 0.f, 0.f};
    for (int k0 = 0; k0 < K; k0 += 32) {
        // 64 rows x 32 k of a and of b: 512 16-byte loads each, two per thread (K % 32 == 0)
#pragma unroll
        for (int p = 0; p < 2; ++p) {
            const int idx = tid + 256 * p, row = idx >> 3, kq = idx & 7;
            const float4v va = (i0 + row < I) ? *reinterpret_cast<const float4v *>(a + (size_t)(i0 + row) * K + k0 + 4 * kq) : zero4;
            const float4v vb = (j0 + row < J) ? *reinterpret_cast<const float4v *>(b + (size_t)(j0 + row) * K + k0 + 4 * kq) : zero4;
#pragma unroll
            for (int q = 0; q < 4; ++q) { As[4 * kq + q][row] = va[q]; Bs[4 * kq + q][row] = vb[q]; }
        }
        __syncthreads();
#pragma unroll 8
        for (int k = 0; k < 32; ++k) {
            const float4v av = *reinterpret_cast<const float4v *>(&As[k][4 * ty]);
            const float4v bv = *reinterpret_cast<const float4v *>(&Bs[k][4 * tx]);
#pragma unroll
            for (int x = 0; x < 4; ++x)
#pragma unroll
                for (int y = 0; y < 4; ++y) {
                    const float t = av[x] + bv[y];
                    acc[x][y] = fmaf(t, t, acc[x][y]);
                }
        }
        __syncthreads();
    }
#pragma unroll
    for (int x = 0; x < 4; ++x) {
        const int i = i0 + 4 * ty + x, j = j0 + 4 * tx;
        if (i < I && j < J) {   // J % 4 == 0
            const float c = rowv[i * 4 + 1], D = rowv[i * 4 + 2];   // -log2e c_ii, -log2e D_i
            float4v o;
#pragma unroll
            for (int y = 0; y < 4; ++y) o[y] = __builtin_amdgcn_exp2f(fmaf(c, acc[x][y], D));
            *reinterpret_cast<float4v *>(f + (size_t)i * J + j) = o;
        }
    }
}

static LongProducts long_products(const tad_plan &pl, const void *const *args, const MfmaWs &w, void *ws) {
    int *const redo = reinterpret_cast<int *>(static_cast<char *>(ws) + align256(pl.ws_bytes));
    return {(const float *)args[0], (const float *)args[1], (const float *)args[2], (const float *)args[3], w.rowv, w.nb, redo + 64, redo,
            (int)pl.fast.I, (int)pl.fast.J, (int)pl.fast.K, (int)pl.fast.c_ld};
}

// full: the workspace holds the parts of a and b; the contractions run on the bf16 matrix cores where that pays, and the kernels here do again what was not finite
int mfma_forward(const tad_plan &pl, const void *const *args, void *f, void *ws, bool full, hipStream_t s) {
    const int I = (int)pl.fast.I, J = (int)pl.fast.J, K = (int)pl.fast.K;
    MfmaWs w = carve_mfma(ws, I, J, K);
    const bool direct = pl.flags & TAD_PLAN_DIRECT_FORM;
    const int *redo = nullptr;
    int rc;
    if (full && !direct && long_forward_pays(I, J, K)) {
        const LongProducts L = long_products(pl, args, w, ws);
        rc = long_forward(L, (float *)f, s);
        redo = L.redo;
    } else {
        rc = prep(pl, args, w, s);
    }
    if (rc) return rc;
    if (direct) {
        TAD_LAUNCH("k_worked_forward_direct", k_worked_forward_direct, dim3((J + 63) / 64, (I + 63) / 64), dim3(256), 0, s,
                   (const float *)args[0], (const float *)args[1], w.rowv, (float *)f, I, J, K);
        return hipGetLastError() == hipSuccess ? TAD_OK : TAD_EDEVICE;
    }
    // (c has at least I x I elements, fewer than 2^31 in all: the tiles along i fit the second axis of a grid)
    if (large_forward_tiles(I, J, K))
        TAD_LAUNCH("k_mfma_forward", k_mfma_forward_large, dim3((J + 127) / 128, (I + 127) / 128), dim3(256), 0, s,
                   (const float *)args[0], (const float *)args[1], w.rowv, w.nb, (float *)f, I, J, K, redo);
    else
        TAD_LAUNCH("k_mfma_forward", k_mfma_forward, dim3((J + 63) / 64, (I + 63) / 64), dim3(256), 0, s,
                   (const float *)args[0], (const float *)args[1], w.rowv, w.nb, (float *)f, I, J, K, redo);
    return hipGetLastError() == hipSuccess ? TAD_OK : TAD_EDEVICE;
}

int mfma_backward(const tad_plan &pl, const void *const *args, const void *f_, const void *df_, void *const *dx,
                  void *ws, bool full, hipStream_t s) {
    const int I = (int)pl.fast.I, J = (int)pl.fast.J, K = (int)pl.fast.K, c_ld = (int)pl.fast.c_ld;
    MfmaWs w = carve_mfma(ws, I, J, K);
    const float *a = (const float *)args[0], *b = (const float *)args[1], *d = (const float *)args[3];
    const float *f = (const float *)f_, *df = (const float *)df_;
    const int *redo = nullptr;
    const bool cols = dx[1] != nullptr, split = full && long_pays(I, J, K);
    const MfmaPieces &n = pl.mfma_pieces[split][cols];
    // partial results for rows i, then for rows j; sums of rows i, then of rows j
    const MfmaSide P{b, w.partial, w.sums, n.chunk_j}, T{a, w.partial + (size_t)n.n_j * I * K, w.sums + (size_t)n.n_j * 2 * I, n.chunk_i};
    int rc;
    if (split) {
        const LongProducts L = long_products(pl, args, w, ws);
        rc = long_backward(L, f, df, P.out, P.sums, n.n_j, n.chunk_j, T.out, T.sums, n.n_i, n.chunk_i, n.totals, s);
        redo = L.redo;
    } else {
        rc = prep(pl, args, w, s);
    }
    if (rc) return rc;
    // the row pass always runs: r_i feeds da, dc and dd; the column pass only for db
    const int tiles = (I + 63) / 64, columns = (K + 255) / 256, first = tiles * n.n_j, blocks_both = first + (cols ? (J + 63) / 64 * n.n_i : 0);
#define TAD_CONTRACTIONS(TOTALS)                                                                                                                          \
    TAD_LAUNCH("k_mfma_backward", k_mfma_backward<TOTALS>, dim3(blocks_both, columns), dim3(512), 0, s, f, df, (const float *)w.rowv, (const float *)w.nb, P, T, I, J, \
               K, first, n.n_j, n.n_i, redo)
    if (split || n.totals) TAD_CONTRACTIONS(true);   // (behind the bf16 kernels: pieces that are theirs)
    else TAD_CONTRACTIONS(false);
#undef TAD_CONTRACTIONS
    if (hipGetLastError() != hipSuccess) return TAD_EDEVICE;
    MfmaFinish F{a, b, d, w.rowv, P.out, T.out, P.sums, T.sums, (float *)dx[0], (float *)dx[1], (float *)dx[2], (float *)dx[3], (long long)pl.arg_count[2],
                 I, J, K, c_ld, (int)pl.arg_count[3], n.n_j, n.n_i, (I + 3) / 4, cols ? (J + 3) / 4 : 0, 0};
    if (dx[3]) F.window = (F.n_d + 3) / 4;
    const long long beyond = dx[2] ? F.n_c - (long long)I * c_ld : 0;
    if (!dx[0] && !dx[2]) F.rows = 0;
    const unsigned blocks = (unsigned)(F.rows + F.cols + F.window + (beyond + 4 * kZeroPiece - 1) / (4 * kZeroPiece));
    TAD_LAUNCH("k_mfma_finish", k_mfma_finish, dim3(blocks), dim3(256), 0, s, F, pl.fast.feas, pl.fast.flat[0], pl.fast.dd_iy, pl.fast.dd_iz);
    return hipGetLastError() == hipSuccess ? TAD_OK : TAD_EDEVICE;
}

}  // namespace tad
