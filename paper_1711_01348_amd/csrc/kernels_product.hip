// Dense products with 64-bit accumulation on the matrix cores (v_mfma_f64_16x16x4_f64): the sums of product.hpp and
// their gradients, in either precision and for any extents and strides.  The general kernels add the terms of such a
// sum in 64 bits, so these do: a 32-bit operand is widened when it is staged, its products are then exact, and the
// result is rounded once.
//
// C[r][c] = sum_q A(r, q) B(q, c).  A workgroup of eight wavefronts computes a tile of 16 NR x 64 results: a wavefront owns 16 columns
// of it and one half of every stage's values of q, and the two halves are added at the end.  What the tile's height is for: a 16 x 16 x 4
// instruction occupies its matrix core for 64 cycles (78.6 TFLOP/s), everything else is to fit under that, so the best that can be done is
// to give the 1024 matrix cores equal numbers of 16 x 16 blocks.  product_shape picks NR (1 .. 7, up to 5 with 64-bit operands) and the
// orientation for that: 1000 x 1203 is 247 tiles of 80 x 64, one for each compute unit and 93 % of an even share, where tiles of 32 x 32 are
// 2.4 rounds that cost three and fetch twice the operands through L2.
// The operands go through registers into LDS, widened to 64 bits on the way, [row][q] with 16 bytes behind each row (fragment reads of 16
// bytes without conflicts); there are two sets of tiles, so that a stage takes one barrier.
// Instructions that are issued beside a matrix instruction cost nothing, in a row of their own they hold it back: every read, store and
// load has its place between two matrix instructions, and the fragments are read one chunk ahead.  1000 x 1203 x 777 in 64 bits, forward:
// 32 x 32 tiles 72 us, these tiles 55, fragments read ahead 47, everything in its place 41 (46 TFLOP/s; 247 of 256 compute units;
// the matrix cores are busy for 61750 cycles, 63 % of that); both gradients 104 -> 90; 512 x 1024 x 768 in 32 bits 24 -> 20,
// gradients 43 -> 36; 2000 x 2000 x 2000 311 -> 287.
// Everything that depends on the tile's place is settled before the loop: a row beyond the edge repeats the last row (its
// results are not stored), so that the loads are unconditional, from a uniform base plus a constant 32-bit offset per thread,
// and only the last stages look at the end of the sum, where zeros are staged.
// Operands of 64 bits: the rounding of the sum is all there is, so it is kept as small as that of the general kernels, which
// share a sum among 64 lanes: a wavefront adds up 16 products at a time, those sums to a subtotal, and every so many stages the subtotal
// to a total, the last two chains of about the same length (60 x 50 x 777: 1.87e-16 of the norm, 40 x 40 x 1203 1.91e-16).
//
// MFMA operand layout: A operand lane l = A[l % 16][l / 16], B operand lane l = B[l / 16][l % 16], result register i of
// lane l = D[4 i + l / 16][l % 16].  Which q a lane group takes is free as long as both operands agree: each takes
// consecutive ones, for wide reads from LDS.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cmath>
#include <type_traits>
#include <utility>

#include "launch.h"
#include "product.hpp"
#include "product_outer.h"
#include "profile.h"

namespace tad {

typedef double double4p __attribute__((ext_vector_type(4)));

struct ProductTask {
    const void *a, *b;
    void *c;           // the result, or (pieces > 1) the partial sums [piece][r][c] in 64 bits
    int R, C, Q;
    int ar, aq, bq, bc;
    int gr, gc;        // tiles along r and c
    int pieces, chunk; // pieces of q, values of q per piece
    int wide;          // store 64-bit results
    int turned;        // store the result [c][r]
    int flush;         // stages of a subtotal (64-bit operands)
    int scaled;        // see ProductJob
    const double *by[2];
    void *to[2];
    int to_wide[2];
};
// One or two products (the derivatives of the two factors of a sum) in one launch: workgroup b works on the first one for
// b < first, else on the second one.
struct ProductArgs {
    ProductTask task[2];
    int first;
    int columns_first;      // workgroups from here on: column sums
    ProductColumns columns;
};
// Neighbouring workgroups go to different dies: each die gets a contiguous range of tiles, walked in groups of eight
// tile rows, so that workgroups that run together share operand tiles in their L2.
__device__ __forceinline__ void product_tile(int lid, int gr, int gc, int &tr, int &tc) {
    const int total = gr * gc;
    const int per = total >> 3;
    if (lid < (per << 3)) lid = (lid & 7) * per + (lid >> 3);
    const int group = 8 * gc;
    const int g0 = (lid / group) * 8;
    const int rows = min(8, gr - g0);
    const int in = lid - (lid / group) * group;
    tr = g0 + in % rows;
    tc = in / rows;
}

typedef double double2p __attribute__((ext_vector_type(2)));

// Sums of 16 columns: 32 threads to a column, whose loads go out eight at a time, added in a fixed order.
constexpr int kColumnSums = 16;
template <typename T>
__device__ __forceinline__ void column_sums(const ProductColumns &S, int block, double *red) {
    constexpr int PARTS = 512 / kColumnSums, U = 8;
    const int tid = threadIdx.x, col = tid % kColumnSums, part = tid / kColumnSums, c = block * kColumnSums + col;
    const T *at = static_cast<const T *>(S.g) + (size_t)min(part, S.R - 1) * S.C + min(c, S.C - 1);
    double sum = 0.0;
    for (int r = part; r < S.R; r += U * PARTS, at += (size_t)U * PARTS * S.C) {
        T v[U];
#pragma unroll
        for (int u = 0; u < U; ++u) v[u] = at[(size_t)(r + u * PARTS < S.R ? u * PARTS : 0) * S.C];
#pragma unroll
        for (int u = 0; u < U; ++u) sum += r + u * PARTS < S.R ? (double)v[u] : 0.0;
    }
    red[tid] = sum;
    __syncthreads();
    if (part != 0 || c >= S.C) return;
    sum = 0.0;
#pragma unroll
    for (int p = 0; p < PARTS; ++p) sum += red[p * kColumnSums + col];
    static_cast<T *>(S.out)[c] = (T)sum;
}

// What the program that is applied to a low tile's results reads besides the sums fits in registers and is sent for before the sum is begun: behind it, the
// addresses and the wait took 1.4 us of a launch (dense 31 x 142 x 80 7.4 -> 6.5 us, softplus 512 x 384 x 200 17.3 -> 16.4).
template <typename TO, int NR> struct OuterOperands {
    static constexpr int ER = 16 * NR, EC = kProductCols, RESULTS = ER * EC / 512, U = RESULTS < ProgWidth<TO>::U ? RESULTS : ProgWidth<TO>::U;
    static constexpr bool EARLY = RESULTS <= U;
    TO w[kMaxArgs][U], d[U];
    int at[U], place[U];   // element of the result (-1: none), place of the sum in LDS
    __device__ __forceinline__ void fetch(const ProductTask &P, const ProductOuter *O, int tid, int r0, int c0) {
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const int n = tid + 512 * u, ir = P.turned ? n % ER : n / EC, ic = P.turned ? n / ER : n % EC, r = r0 + ir, c = c0 + ic;
            const bool inside = r < P.R && c < P.C;
            place[u] = ir * (EC + 1) + ic;
            at[u] = !inside ? -1 : P.turned ? c * P.R + r : r * P.C + c;
#pragma unroll
            for (int q = 0; q < kMaxArgs; ++q)
                w[q][u] = O->args.p[q] ? static_cast<const TO *>(O->args.p[q])[inside ? O->off_r[q] * r + O->off_c[q] * c : 0] : TO(0);
            d[u] = O->df ? static_cast<const TO *>(O->df)[max(at[u], 0)] : TO(1);
        }
    }
};
template <int NR> struct OuterOperands<void, NR> {
    static constexpr bool EARLY = false;
};

// EXTRA: scaled results or column sums (their code in every kernel: 1000 x 1203 x 777 in 64 bits 130 -> 134 us with its gradients)
template <typename TA, typename TB, int NR, typename TO, bool EXTRA>
__device__ __forceinline__ void product_kernel(const ProductArgs &M, const ProductOuter *O) {
    constexpr bool BLOCKED = sizeof(TA) == 8 && sizeof(TB) == 8;   // sums of 16 products added to a subtotal
    constexpr int NT = 512, ER = 16 * NR, EC = kProductCols;
    constexpr int KT = kProductStage;               // values of q per stage
    constexpr int KL = KT / 8;                      // ... of one lane: half a stage among the four lane groups
    constexpr int CHUNKS = KL / 2;                  // ... read two at a time
    constexpr int LDK = KT + 2;                     // row length in LDS
    constexpr int PA = ER * KT / NT, PB = EC * KT / NT;   // elements of each operand a thread stages
    constexpr int AHEAD = NR <= 2 ? 2 : 1;          // stages in registers: one lasts about as long as a load with low tiles
    constexpr int LDS_SUM = EC + 1;
    constexpr int SIZE_A = ER * LDK, SIZE_B = EC * LDK, TILES = 2 * (SIZE_A + SIZE_B), SUMS = ER * LDS_SUM;
    static_assert(PA * NT == ER * KT && PB * NT == EC * KT && CHUNKS % 2 == 0, "whole stages");
    __shared__ __attribute__((aligned(16))) double lds[TILES > SUMS ? TILES : SUMS];
    double *const As = lds, *const Bs = lds + 2 * SIZE_A;
    if constexpr (EXTRA) {
        if ((int)blockIdx.x >= M.columns_first) {
            if (M.columns.wide) column_sums<double>(M.columns, (int)blockIdx.x - M.columns_first, lds);
            else column_sums<float>(M.columns, (int)blockIdx.x - M.columns_first, lds);
            return;
        }
    }
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const ProductTask &P = M.task[(int)blockIdx.x < M.first ? 0 : 1];   // the same for the whole workgroup
    const int id = (int)blockIdx.x - ((int)blockIdx.x < M.first ? 0 : M.first), tiles = P.gr * P.gc, piece = id / tiles;
    int tr, tc;
    product_tile(id - piece * tiles, P.gr, P.gc, tr, tc);
    const int r0 = tr * ER, c0 = tc * EC;
    const int q_begin = piece * P.chunk, q_end = min(P.Q, q_begin + P.chunk);
    // staging: neighbouring threads along q or along the rows, whichever is contiguous in memory
    const bool a_q = P.aq <= P.ar, b_q = P.bq <= P.bc;   // uniform
    // (groups of G rows, the largest power of two in ER: constant steps from one element of a thread to the next)
    constexpr int G = ER & -ER, PG = KT * G / NT;
    const int a_row = a_q ? tid / KT : tid % G, a_k = a_q ? tid % KT : tid / G;
    const int b_row = b_q ? tid / KT : tid % EC, b_k = b_q ? tid % KT : tid / EC;
    auto a_dr = [&](int p) { return a_q ? p * (NT / KT) : p / PG * G; };
    auto a_dk = [&](int p) { return a_q ? 0 : p % PG * (NT / G); };
    auto b_dr = [&](int p) { return b_q ? p * (NT / KT) : 0; };
    auto b_dk = [&](int p) { return b_q ? 0 : p * (NT / EC); };
    using Outer = OuterOperands<TO, NR>;
    Outer outer;
    if constexpr (Outer::EARLY) outer.fetch(P, O, tid, r0, c0);
    unsigned ao[PA], bo[PB];       // byte offsets within a stage
#pragma unroll
    for (int p = 0; p < PA; ++p)
        ao[p] = (unsigned)(min(a_row + a_dr(p), P.R - 1 - r0) * P.ar + (a_k + a_dk(p)) * P.aq) * (unsigned)sizeof(TA);
#pragma unroll
    for (int p = 0; p < PB; ++p)
        bo[p] = (unsigned)(min(b_row + b_dr(p), P.C - 1 - c0) * P.bc + (b_k + b_dk(p)) * P.bq) * (unsigned)sizeof(TB);
    const char *pa = reinterpret_cast<const char *>(static_cast<const TA *>(P.a) + (size_t)r0 * P.ar + (size_t)q_begin * P.aq);
    const char *pb = reinterpret_cast<const char *>(static_cast<const TB *>(P.b) + (size_t)c0 * P.bc + (size_t)q_begin * P.bq);
    struct Staged { TA a[PA]; TB b[PB]; } regs[AHEAD];
    auto load = [&](int q0, Staged &v) {
        if (q0 + KT <= q_end) {   // the same for the whole workgroup
#pragma unroll
            for (int p = 0; p < PA; ++p) v.a[p] = *reinterpret_cast<const TA *>(pa + ao[p]);
#pragma unroll
            for (int p = 0; p < PB; ++p) v.b[p] = *reinterpret_cast<const TB *>(pb + bo[p]);
        } else {                  // the last stage: beyond the end of the sum the last value is read and a zero staged
#pragma unroll
            for (int p = 0; p < PA; ++p) {
                const int over = max(q0 + a_k + a_dk(p) - (q_end - 1), 0);
                const TA t = *reinterpret_cast<const TA *>(pa + (ao[p] - (unsigned)(over * P.aq) * (unsigned)sizeof(TA)));
                v.a[p] = over ? TA(0) : t;
            }
#pragma unroll
            for (int p = 0; p < PB; ++p) {
                const int over = max(q0 + b_k + b_dk(p) - (q_end - 1), 0);
                const TB t = *reinterpret_cast<const TB *>(pb + (bo[p] - (unsigned)(over * P.bq) * (unsigned)sizeof(TB)));
                v.b[p] = over ? TB(0) : t;
            }
        }
        pa += (size_t)KT * P.aq * sizeof(TA);
        pb += (size_t)KT * P.bq * sizeof(TB);
    };
    const int as = a_row * LDK + a_k, bs = b_row * LDK + b_k;
    auto stage = [&](int set, const Staged &v) {
#pragma unroll
        for (int p = 0; p < PA; ++p) As[set * SIZE_A + as + a_dr(p) * LDK + a_dk(p)] = (double)v.a[p];
#pragma unroll
        for (int p = 0; p < PB; ++p) Bs[set * SIZE_B + bs + b_dr(p) * LDK + b_dk(p)] = (double)v.b[p];
    };
    const double4p zero = {0., 0., 0., 0.};
    double4p acc[NR], sub[BLOCKED ? NR : 1], total[BLOCKED ? NR : 1];
#pragma unroll
    for (int x = 0; x < NR; ++x) {
        acc[x] = zero;
        if constexpr (BLOCKED) sub[x] = total[x] = zero;
    }
    const int col = wave & 3, half = wave >> 2;
    const int fk = half * (KT / 2) + (lane >> 4) * KL;
    const int fa = (lane & 15) * LDK + fk, fb = (16 * col + (lane & 15)) * LDK + fk;
    double2p fragments[2][NR + 1];
    auto read = [&](int set, int c, double2p (&v)[NR + 1]) {
#pragma unroll
        for (int x = 0; x < NR; ++x) v[x] = *reinterpret_cast<const double2p *>(As + set * SIZE_A + fa + x * 16 * LDK + c * 2);
        v[NR] = *reinterpret_cast<const double2p *>(Bs + set * SIZE_B + fb + c * 2);
    };
    {
        Staged begin;   // the first loads all go out before the first of them is waited for
        load(q_begin, begin);
#pragma unroll
        for (int n = 1; n <= AHEAD; ++n)
            if (q_begin + n * KT < q_end) load(q_begin + n * KT, regs[n % AHEAD]);
        if constexpr (!std::is_same<TO, void>::value) fetch_program(O->prog);
        stage(0, begin);
    }
    __syncthreads();
    read(0, 0, fragments[0]);
    // One stage.  The fragments of a chunk are read among the matrix instructions of the chunk before it, also across the barrier, and so
    // is everything else that goes to memory: a wavefront that sends its loads and stores out in a row holds back its own matrix
    // instructions and, being in step with it, those of the other wavefront of its SIMD.  WHOLE: the stage that is to be loaded exists and
    // is a whole one, so that there is nothing to ask.  The scheduling barriers keep the compiler from moving the reads down to their use.
    auto step = [&](int q0, auto parity, auto whole) {
        constexpr int SET = decltype(parity)::value, MF = 2 * NR;   // matrix instructions of a chunk
        constexpr bool WHOLE = decltype(whole)::value;
        Staged &v = regs[(SET + 1) % AHEAD];
        int as_now = as, bs_now = bs;
        asm volatile("" : "+v"(as_now), "+v"(bs_now));   // an address is one addition at its use, and a register each if they are kept
#pragma unroll
        for (int c = 0; c < CHUNKS; ++c) {
            const bool last = c + 1 == CHUNKS;
            const double2p(&now)[NR + 1] = fragments[c & 1];
            double2p(&next)[NR + 1] = fragments[(c + 1) & 1];
            // elements of the stage that this chunk takes from registers to LDS and loads again
            const int e0 = last ? 0 : c * (PA + PB) / (CHUNKS - 1), e1 = last ? 0 : (c + 1) * (PA + PB) / (CHUNKS - 1);
            const int first = last ? MF / 2 : 0;   // matrix instructions before the barrier
            const int ops = NR + 1 + (WHOLE ? e1 - e0 : 0), slots = MF - first;
#pragma unroll
            for (int m = 0; m < MF; ++m) {
                const int x = m % NR, i = m / NR;
                if (last && m == first) __syncthreads();
                if (m >= first) {
#pragma unroll
                    for (int o = 0; o < ops; ++o) {
                        if (o < (m - first) * ops / slots || o >= (m - first + 1) * ops / slots) continue;
                        if (o <= NR) {   // (behind the last stage: whatever is there, it is not used)
                            const int set = last ? SET ^ 1 : SET, at = last ? 0 : (c + 1) * 2, row = (o + NR) % (NR + 1);   // the common fragment first
                            next[row] = *reinterpret_cast<const double2p *>(row < NR ? As + set * SIZE_A + fa + row * 16 * LDK + at : Bs + set * SIZE_B + fb + at);
                        } else {
                            const int e = e0 + o - NR - 1, p = e < PA ? e : e - PA;
                            unsigned from = e < PA ? ao[p] : bo[p];
                            asm volatile("" : "+v"(from));   // 32 bits beside a uniform base, not widened ahead of time
                            if (e < PA) {
                                As[(SET ^ 1) * SIZE_A + as_now + a_dr(p) * LDK + a_dk(p)] = (double)v.a[p];
                                v.a[p] = *reinterpret_cast<const TA *>(pa + from);
                            } else {
                                Bs[(SET ^ 1) * SIZE_B + bs_now + b_dr(p) * LDK + b_dk(p)] = (double)v.b[p];
                                v.b[p] = *reinterpret_cast<const TB *>(pb + from);
                            }
                        }
                    }
                    __builtin_amdgcn_sched_barrier(0);
                }
                acc[x] = __builtin_amdgcn_mfma_f64_16x16x4f64(now[x][i], now[NR][i], BLOCKED && i == 0 && c % 2 == 0 ? zero : acc[x], 0, 0, 0);
                __builtin_amdgcn_sched_barrier(0);
            }
            if constexpr (BLOCKED) {
                if (c % 2 == 1) {
#pragma unroll
                    for (int x = 0; x < NR; ++x) sub[x] += acc[x];
                }
            }
            if constexpr (!WHOLE) {
                if (c == CHUNKS / 2 - 1) {
                    if (q0 + KT < q_end) stage(SET ^ 1, v);   // the same for the whole workgroup
                    if (q0 + (1 + AHEAD) * KT < q_end) load(q0 + (1 + AHEAD) * KT, v);
                }
            }
        }
        if constexpr (WHOLE) {
            pa += (size_t)KT * P.aq * sizeof(TA);
            pb += (size_t)KT * P.bq * sizeof(TB);
        }
    };
    int left = P.flush;
    auto flush = [&] {
        if constexpr (BLOCKED) {
            if (--left) return;
            left = P.flush;
#pragma unroll
            for (int x = 0; x < NR; ++x) {
                total[x] += sub[x];
                sub[x] = zero;
            }
        }
    };
    // (two stages at a time, and no way out in between: that would cost a second set of registers for the sums)
    const std::integral_constant<int, 0> even{};
    const std::integral_constant<int, 1> odd{};
    int q0 = q_begin;
    for (; q0 + (3 + AHEAD) * KT <= q_end; q0 += 2 * KT) {
        step(q0, even, std::true_type());
        flush();
        step(q0 + KT, odd, std::true_type());
        flush();
    }
    for (; q0 + KT < q_end; q0 += 2 * KT) {
        step(q0, even, std::false_type());
        flush();
        step(q0 + KT, odd, std::false_type());
        flush();
    }
    if (q0 < q_end) step(q0, even, std::false_type());
    if constexpr (BLOCKED) {
#pragma unroll
        for (int x = 0; x < NR; ++x) acc[x] = total[x] + sub[x];
    }
    // the two halves of the sum (behind the last barrier of the loop the tiles are free)
    double *const sums = lds;
    const int own = (lane >> 4) * LDS_SUM + 16 * col + (lane & 15);
    if (half) {
#pragma unroll
        for (int x = 0; x < NR; ++x)
#pragma unroll
            for (int i = 0; i < 4; ++i) sums[own + (16 * x + 4 * i) * LDS_SUM] = acc[x][i];
    }
    __syncthreads();
    if (!half) {
#pragma unroll
        for (int x = 0; x < NR; ++x)
#pragma unroll
            for (int i = 0; i < 4; ++i) sums[own + (16 * x + 4 * i) * LDS_SUM] += acc[x][i];
    }
    __syncthreads();
    char *out = static_cast<char *>(P.c) + (size_t)piece * P.R * P.C * sizeof(double);   // (one piece: 0)
    constexpr int RESULTS = ER * EC / NT;
    if constexpr (std::is_same<TO, void>::value) {
        // neighbouring threads along the direction that is contiguous in the result
        if constexpr (EXTRA) {
#pragma unroll 1
            for (int t = 0; t < P.scaled; ++t) {   // the same for the whole workgroup
                const double *const by = P.by[t];
                double v[RESULTS];
                int at[RESULTS];
#pragma unroll
                for (int p = 0; p < RESULTS; ++p) {
                    const int n = tid + NT * p, ir = P.turned ? n % ER : n / EC, ic = P.turned ? n / ER : n % EC, r = r0 + ir, c = c0 + ic;
                    const int place = P.turned ? c * P.R + r : r * P.C + c;
                    at[p] = r < P.R && c < P.C ? place : -1;
                    v[p] = by[max(at[p], 0)];
                }
#pragma unroll
                for (int p = 0; p < RESULTS; ++p) {
                    const int n = tid + NT * p, ir = P.turned ? n % ER : n / EC, ic = P.turned ? n / ER : n % EC;
                    v[p] *= sums[ir * LDS_SUM + ic];
                    if (at[p] < 0) continue;
                    if (P.to_wide[t]) static_cast<double *>(P.to[t])[at[p]] = v[p];
                    else static_cast<float *>(P.to[t])[at[p]] = (float)v[p];
                }
            }
            if (P.scaled) return;
        }
#pragma unroll
        for (int p = 0; p < RESULTS; ++p) {
            const int n = tid + NT * p, ir = P.turned ? n % ER : n / EC, ic = P.turned ? n / ER : n % EC, r = r0 + ir, c = c0 + ic;
            const double v = sums[ir * LDS_SUM + ic];
            if (r >= P.R || c >= P.C) continue;
            const size_t at = P.turned ? (size_t)c * P.R + r : (size_t)r * P.C + c;
            if (P.wide) reinterpret_cast<double *>(out)[at] = v;
            else reinterpret_cast<float *>(out)[at] = (float)v;
        }
    } else if constexpr (Outer::EARLY) {
        TO s[Outer::U], o[Outer::U];
#pragma unroll
        for (int u = 0; u < Outer::U; ++u) s[u] = (TO)sums[outer.place[u]];
        prog_eval_block<TO, Outer::U, true>(O->prog, outer.w, s, o);
#pragma unroll
        for (int u = 0; u < Outer::U; ++u) {
            if (outer.at[u] < 0) continue;
            reinterpret_cast<TO *>(out)[outer.at[u]] = O->df ? outer.d[u] * o[u] : o[u];
            if (O->s_out) static_cast<TO *>(O->s_out)[outer.at[u]] = s[u];
        }
    } else {
        // U results per pass of the interpreter: an operation costs more to fetch than to carry out. df is read behind the program: before it, its registers
        // cost the tall tiles more than the wait (dense 2000 x 1000 x 64: 22.4 us instead of 21.2).
        constexpr int U = ProgWidth<TO>::U;
#pragma unroll 1
        for (int p0 = 0; p0 < RESULTS; p0 += U) {
            TO s[U], w[kMaxArgs][U], o[U];
            int at[U];
            bool inside[U];
#pragma unroll
            for (int u = 0; u < U; ++u) {
                const int n = min(tid + NT * (p0 + u), ER * EC - 1), ir = P.turned ? n % ER : n / EC, ic = P.turned ? n / ER : n % EC;
                const int r = r0 + ir, c = c0 + ic;
                s[u] = (TO)sums[ir * LDS_SUM + ic];
                inside[u] = p0 + u < RESULTS && r < P.R && c < P.C;
                at[u] = !inside[u] ? 0 : P.turned ? c * P.R + r : r * P.C + c;
#pragma unroll
                for (int q = 0; q < kMaxArgs; ++q)
                    w[q][u] = O->args.p[q] ? static_cast<const TO *>(O->args.p[q])[inside[u] ? O->off_r[q] * r + O->off_c[q] * c : 0] : TO(0);
            }
            prog_eval_block<TO, U, true>(O->prog, w, s, o);
#pragma unroll
            for (int u = 0; u < U; ++u) {
                if (!inside[u]) continue;
                reinterpret_cast<TO *>(out)[at[u]] = O->df ? static_cast<const TO *>(O->df)[at[u]] * o[u] : o[u];
                if (O->s_out) static_cast<TO *>(O->s_out)[at[u]] = s[u];
            }
        }
    }
}

template <typename TA, typename TB, int NR>
__global__ __launch_bounds__(512, 2) void k_product(const ProductArgs M) {
    product_kernel<TA, TB, NR, void, false>(M, nullptr);
}
// ... which are scaled, or with column sums beside them
template <typename TA, typename TB, int NR>
__global__ __launch_bounds__(512, 2) void k_product_extra(const ProductArgs M) {
    product_kernel<TA, TB, NR, void, true>(M, nullptr);
}
// sums of type TO that go through a program first
template <typename TA, typename TB, typename TO, int NR>
__global__ __launch_bounds__(512, 2) void k_product_outer(const ProductArgs M, const ProductOuter O) {
    product_kernel<TA, TB, NR, TO, false>(M, &O);
}

// c[i] = the pieces' partial sums of element i.  A workgroup takes 256 / GROUPS elements, GROUPS threads for each, whose loads go out
// four at a time: with a thread per element a long chain of loads took longer than the product (a gradient of 8 x 16 over 100001
// rows, 313 pieces: 82 -> 15 us with the product).  Up to four pieces are one batch of a single thread (2 pieces of 384 x 200, shortest
// of 28 launches: on eight threads 2.1 us, on one 1.4).
constexpr int kReduceGroups = 8, kReduceBatch = 4;
template <typename T, int GROUPS>
__global__ __launch_bounds__(256) void k_product_reduce(const double *__restrict__ part, T *__restrict__ c, long long n, int pieces) {
    constexpr int COLS = 256 / GROUPS, U = kReduceBatch;
    __shared__ double red[GROUPS][COLS + 1];
    const int col = threadIdx.x % COLS, group = threadIdx.x / COLS;
    const long long i = (long long)blockIdx.x * COLS + col;
    double s = 0.0;
    if (i < n) {
        const double *at = part + group * n + i;
        for (int p = group; p < pieces; p += U * GROUPS, at += U * GROUPS * n) {
            double v[U];
#pragma unroll
            for (int u = 0; u < U; ++u) v[u] = p + u * GROUPS < pieces ? at[u * GROUPS * n] : 0.0;
#pragma unroll
            for (int u = 0; u < U; ++u) s += v[u];
        }
    }
    if constexpr (GROUPS > 1) {
        red[group][col] = s;
        __syncthreads();
        if (group != 0) return;
#pragma unroll
        for (int g = 1; g < GROUPS; ++g) s += red[g][col];
    }
    if (i < n) c[i] = (T)s;
}
template <typename T>
static int reduce_pieces(const void *part, void *c, long long n, int pieces, hipStream_t s) {
    if (pieces <= kReduceBatch)
        TAD_LAUNCH("k_product_reduce", (k_product_reduce<T, 1>), dim3((unsigned)((n + 255) / 256)), dim3(256), 0, s, (const double *)part, (T *)c, n, pieces);
    else
        TAD_LAUNCH("k_product_reduce", (k_product_reduce<T, kReduceGroups>), dim3((unsigned)((n + 256 / kReduceGroups - 1) / (256 / kReduceGroups))),
                   dim3(256), 0, s, (const double *)part, (T *)c, n, pieces);
    return hipGetLastError() == hipSuccess ? TAD_OK : TAD_EDEVICE;
}

static ProductTask product_task(const ProductJob &j, int rows, bool share, void *ws) {
    const ProductDesc &d = *j.desc;
    const int edge = 16 * rows;
    ProductTask P;
    P.a = j.a; P.b = j.b;
    P.pieces = share ? d.pieces : 1;
    P.chunk = P.pieces > 1 ? d.chunk : d.Q;
    P.c = P.pieces > 1 ? ws : j.c;
    P.R = d.R; P.C = d.C; P.Q = d.Q;
    P.ar = (int)d.ar; P.aq = (int)d.aq; P.bq = (int)d.bq; P.bc = (int)d.bc;
    P.gr = (d.R + edge - 1) / edge; P.gc = (d.C + kProductCols - 1) / kProductCols;
    P.wide = j.c64 || P.pieces > 1;
    P.turned = j.turned;
    P.scaled = j.scaled;
    for (int t = 0; t < 2; ++t) {
        P.by[t] = j.by[t];
        P.to[t] = j.to[t];
        P.to_wide[t] = j.to64[t];
    }
    // 16 products in a row, then `flush` stages of a subtotal, then the total: the last two chains of about the same length
    const double blocks = P.chunk / 32.0, per_stage = kProductStage / 32.0;   // of a wavefront: half the sum
    P.flush = std::max(1, (int)(std::sqrt(blocks) / per_stage + 0.5));
    return P;
}

template <typename TA, typename TB, int NR>
static int launch_product(const ProductArgs &M, unsigned blocks, const ProductOuter *outer, bool c64, hipStream_t s) {
    const dim3 grid(blocks), block(512);
    if (!outer && (M.columns.out || M.task[0].scaled || M.task[1].scaled)) TAD_LAUNCH("k_product", (k_product_extra<TA, TB, NR>), grid, block, 0, s, M);
    else if (!outer) TAD_LAUNCH("k_product", (k_product<TA, TB, NR>), grid, block, 0, s, M);
    else if constexpr (sizeof(TA) == 8 && sizeof(TB) == 8) {
        if (c64) TAD_LAUNCH("k_product_outer", (k_product_outer<TA, TB, double, NR>), grid, block, 0, s, M, *outer);
        else TAD_LAUNCH("k_product_outer", (k_product_outer<TA, TB, float, NR>), grid, block, 0, s, M, *outer);
    } else {   // (a 32-bit operand is one of a 32-bit expression)
        TAD_LAUNCH("k_product_outer", (k_product_outer<TA, TB, float, NR>), grid, block, 0, s, M, *outer);
    }
    return hipGetLastError() == hipSuccess ? TAD_OK : TAD_EDEVICE;
}
template <typename TA, typename TB>
static int launch_rows(const ProductArgs &M, int rows, unsigned blocks, const ProductOuter *outer, bool c64, hipStream_t s) {
    switch (rows) {
    case 1: return launch_product<TA, TB, 1>(M, blocks, outer, c64, s);
    case 2: return launch_product<TA, TB, 2>(M, blocks, outer, c64, s);
    case 3: return launch_product<TA, TB, 3>(M, blocks, outer, c64, s);
    case 4: return launch_product<TA, TB, 4>(M, blocks, outer, c64, s);
    case 5: return launch_product<TA, TB, 5>(M, blocks, outer, c64, s);
    default:
        if constexpr (sizeof(TA) == 4 || sizeof(TB) == 4) {
            if (rows == 6) return launch_product<TA, TB, 6>(M, blocks, outer, c64, s);
            if (rows == 7) return launch_product<TA, TB, 7>(M, blocks, outer, c64, s);
        }
        return TAD_EUNSUPPORTED;
    }
}

// the product with its operands exchanged, stored back in place
static ProductJob exchanged(const ProductJob &j, ProductDesc &d) {
    d = product_turned(*j.desc);
    ProductJob t = j;
    t.desc = &d;
    std::swap(t.a, t.b);
    std::swap(t.a64, t.b64);
    t.turned = !j.turned;
    return t;
}

// count (1 or 2) products of the same operand types in one launch; share: their sums in pieces (one product only)
static int launch_jobs(const ProductJob *jobs, int count, int rows, bool share, const ProductOuter *outer, void *ws, hipStream_t s,
                       const ProductColumns *columns = nullptr) {
    ProductArgs M{};
    unsigned blocks = 0;
    for (int q = 0; q < count; ++q) {
        M.task[q] = product_task(jobs[q], rows, share, ws);
        blocks += (unsigned)(M.task[q].gr * M.task[q].gc * M.task[q].pieces);
        if (q == 0) M.first = (int)blocks;
    }
    M.columns_first = (int)blocks;
    if (columns) {
        M.columns = *columns;
        blocks += (unsigned)((columns->C + kColumnSums - 1) / kColumnSums);
    }
    const ProductJob &j = jobs[0];
    int rc;
    if (j.a64 && j.b64) rc = launch_rows<double, double>(M, rows, blocks, outer, j.c64, s);
    else if (j.a64) rc = launch_rows<double, float>(M, rows, blocks, outer, j.c64, s);
    else if (j.b64) rc = launch_rows<float, double>(M, rows, blocks, outer, j.c64, s);
    else rc = launch_rows<float, float>(M, rows, blocks, outer, j.c64, s);
    if (rc || !share || j.desc->pieces == 1) return rc;
    const long long n = (long long)j.desc->R * j.desc->C;
    return j.c64 ? reduce_pieces<double>(ws, j.c, n, j.desc->pieces, s) : reduce_pieces<float>(ws, j.c, n, j.desc->pieces, s);
}

int product_run(const ProductJob &j, void *ws, hipStream_t s, const ProductColumns *columns) {
    ProductDesc d;
    const ProductJob job = j.desc->flip ? exchanged(j, d) : j;
    return launch_jobs(&job, 1, j.desc->rows, true, nullptr, ws, s, columns);
}

bool product_scales(const ProductDesc &d, bool one_of_two) { return (one_of_two && d.pair_rows) || d.pieces == 1; }

bool product_outer_fits(const ProductDesc &d) { return d.pieces == 1; }

int product_run_outer(const ProductJob &j, const ProductOuter &o, hipStream_t s) {
    if (!j.desc->flip) return launch_jobs(&j, 1, j.desc->rows, false, &o, nullptr, s);
    ProductDesc d;
    const ProductJob job = exchanged(j, d);
    ProductOuter t = o;
    for (int q = 0; q < kMaxArgs; ++q) std::swap(t.off_r[q], t.off_c[q]);
    return launch_jobs(&job, 1, d.rows, false, &t, nullptr, s);
}

int product_run_two(const ProductJob &x, const ProductJob &y, void *ws, hipStream_t s, const ProductColumns *columns) {
    // one launch for both where that is faster: two products fill the chip better than one (product_pair)
    if (x.desc->pair_rows) {
        ProductDesc d[2];
        ProductJob jobs[2] = {x.desc->pair_flip ? exchanged(x, d[0]) : x, y.desc->pair_flip ? exchanged(y, d[1]) : y};
        if (x.desc->Q < y.desc->Q) std::swap(jobs[0], jobs[1]);   // the longer ones first
        return launch_jobs(jobs, 2, x.desc->pair_rows, false, nullptr, ws, s, columns);
    }
    const int rc = product_run(x, ws, s, columns);
    return rc ? rc : product_run(y, ws, s);
}

int product_forward(const tad_plan &pl, const ProductSet &set, const void *const *args, void *f, void *ws, hipStream_t s) {
    const ProductPlan &pp = pl.prod;
    const bool f64 = pl.dtype == TAD_F64;
    const ProductJob j = {&set.forward, args[pp.side[0].operand], f64, args[pp.side[1].operand], f64, f, f64};
    return product_run(j, static_cast<char *>(ws) + pp.ws_offset, s);
}

int product_backward(const tad_plan &pl, const ProductSet &set, const void *const *args, const void *df, void **dx, void *ws, hipStream_t s) {
    const ProductPlan &pp = pl.prod;
    const bool f64 = pl.dtype == TAD_F64;
    void *const part = static_cast<char *>(ws) + pp.ws_offset;   // used by the products in turn
    ProductJob jobs[2];
    int n = 0;
    for (int q = 0; q < 2; ++q) {
        const ProductSide &sd = pp.side[q];
        if (!sd.grad || !dx[sd.operand]) continue;
        const void *other = args[pp.side[1 - q].operand];
        jobs[n++] = {&set.grad[q], sd.k_major ? other : df, f64, sd.k_major ? df : other, f64, dx[sd.operand], f64};
        dx[sd.operand] = nullptr;
    }
    return n == 2 ? product_run_two(jobs[0], jobs[1], part, s) : n == 1 ? product_run(jobs[0], part, s) : TAD_OK;
}

}  // namespace tad
