// The worked expression of the paper (kernels_worked.hip) with 64-bit sums: for the forms the fused 32-bit kernels do not take
// (64-bit tensors, rows of f that start anywhere, K up to 16) and for tensors that do not fill the chip with the large tiles of
// those.  The plan-driven kernels, which evaluate the former otherwise, accumulate in 64 bits, so these do; sums are of the terms
// as they stand, not expanded,
//
//     t_ijk = a_ik + b_jk,  q_ij = sum_k t_ijk^2,  g_ij = df_ij f_ij:       f_ij = exp(-(c_ii q_ij + sum_k d_{i+k}^3))
//     da_ik = -2 c_ii sum_j g_ij t_ijk     db_jk = -2 sum_i c_ii g_ij t_ijk     dc_ii = -sum_j g_ij q_ij
//     dd_m  = -3 d_m^2 sum over the window of sum_j g_ij
//
// and one pass over df and f yields all of them: column sums stay in registers while a wavefront walks down its rows, the
// K + 2 row sums are added up across the wavefront for two rows at a time.  4 K + 5 operations in 64 bits per element are about
// as long as the two reads: 3001 x 2047 x 7, 32 bits.
// Columns are 64 apart within a lane, so that every load of a wavefront covers one contiguous piece of a row wherever it starts.
#include <hip/hip_runtime.h>

#include "gather_loop.h"
#include "launch.h"
#include "launch_geom.h"
#include "plan_dev.h"
#include "profile.h"
#include "zeros.h"

namespace tad {

template <typename T> struct WideExp;
template <> struct WideExp<float> { static __device__ __forceinline__ float of(double s) { return expf((float)s); } };
template <> struct WideExp<double> { static __device__ __forceinline__ double of(double s) { return exp(s); } };

// ---------------------------------------------------------------------------------------------
// forward: 512 columns x 8 rows per workgroup, two columns per thread
// ---------------------------------------------------------------------------------------------
constexpr int WIDE_FWD_ROWS = 8, WIDE_FWD_COLS = 512;

template <typename T, int K>
__global__ __launch_bounds__(256) void k_worked_wide_forward(const T *__restrict__ a, const T *__restrict__ b, const T *__restrict__ c,
                                                             const T *__restrict__ d, T *__restrict__ f, int I, int J, int c_ld) {
    constexpr int CW = WIDE_FWD_COLS / 256;
    __shared__ double rd[WIDE_FWD_ROWS][K + 2];
    const int tid = threadIdx.x, i0 = blockIdx.y * WIDE_FWD_ROWS, rows = min(WIDE_FWD_ROWS, I - i0);
    if (tid < rows) {
        const int i = i0 + tid;
        double D = 0.0;
#pragma unroll
        for (int k = 0; k < K; ++k) {
            rd[tid][k] = (double)a[(size_t)i * K + k];
            const double dv = (double)d[i + k];
            D = fma(dv * dv, dv, D);
        }
        rd[tid][K] = (double)c[(size_t)i * c_ld + i];
        rd[tid][K + 1] = D;
    }
    __syncthreads();
    const int j0 = blockIdx.x * WIDE_FWD_COLS + tid;
    double bj[CW][K];
#pragma unroll
    for (int v = 0; v < CW; ++v)
#pragma unroll
        for (int k = 0; k < K; ++k) bj[v][k] = (double)b[(size_t)min(j0 + v * 256, J - 1) * K + k];
    T *fp = f + (size_t)i0 * J + j0;
    for (int r = 0; r < rows; ++r, fp += J) {
        double q[CW] = {};
#pragma unroll
        for (int k = 0; k < K; ++k) {
            const double ai = rd[r][k];
#pragma unroll
            for (int v = 0; v < CW; ++v) {
                const double t = ai + bj[v][k];
                q[v] = fma(t, t, q[v]);
            }
        }
        const double ci = rd[r][K], D = rd[r][K + 1];
#pragma unroll
        for (int v = 0; v < CW; ++v)
            if (j0 + v * 256 < J) __builtin_nontemporal_store(WideExp<T>::of(-fma(ci, q[v], D)), fp + v * 256);
    }
}

// ---------------------------------------------------------------------------------------------
// backward
// ---------------------------------------------------------------------------------------------

// Sums of N values over the 64 lanes.  The first two steps halve the number of registers instead of the number of lanes that
// count: two values exchange halves (rows of 16 lanes) and are added as one register.  After the call v[p] holds, in the lanes
// 16 s .. 16 s + 15, the total of value 4 p + {0, 2, 1, 3}[s].
__device__ __forceinline__ double swap32_add(double x, double y) {
    const auto lo = __builtin_amdgcn_permlane32_swap((unsigned)__double2loint(x), (unsigned)__double2loint(y), false, false);
    const auto hi = __builtin_amdgcn_permlane32_swap((unsigned)__double2hiint(x), (unsigned)__double2hiint(y), false, false);
    return __hiloint2double((int)hi[0], (int)lo[0]) + __hiloint2double((int)hi[1], (int)lo[1]);
}
__device__ __forceinline__ double swap16_add(double x, double y) {
    const auto lo = __builtin_amdgcn_permlane16_swap((unsigned)__double2loint(x), (unsigned)__double2loint(y), false, false);
    const auto hi = __builtin_amdgcn_permlane16_swap((unsigned)__double2hiint(x), (unsigned)__double2hiint(y), false, false);
    return __hiloint2double((int)hi[0], (int)lo[0]) + __hiloint2double((int)hi[1], (int)lo[1]);
}
template <int CTRL> __device__ __forceinline__ double row_add(double v) {   // rotation within 16 lanes
    const int lo = __builtin_amdgcn_update_dpp(0, __double2loint(v), CTRL, 0xf, 0xf, true);
    const int hi = __builtin_amdgcn_update_dpp(0, __double2hiint(v), CTRL, 0xf, 0xf, true);
    return v + __hiloint2double(hi, lo);
}
template <int N> __device__ __forceinline__ void wave_totals(double (&v)[N]) {
    constexpr int H = (N + 1) / 2, Q = (H + 1) / 2;
    double h[2 * Q];
#pragma unroll
    for (int p = 0; p < H; ++p) h[p] = swap32_add(v[2 * p], 2 * p + 1 < N ? v[2 * p + 1] : 0.0);
    if (H < 2 * Q) h[2 * Q - 1] = 0.0;
#pragma unroll
    for (int p = 0; p < Q; ++p) v[p] = swap16_add(h[2 * p], h[2 * p + 1]);
#pragma unroll
    for (int p = 0; p < Q; ++p) v[p] = row_add<0x128>(v[p]);
#pragma unroll
    for (int p = 0; p < Q; ++p) v[p] = row_add<0x124>(v[p]);
#pragma unroll
    for (int p = 0; p < Q; ++p) v[p] = row_add<0x122>(v[p]);
#pragma unroll
    for (int p = 0; p < Q; ++p) v[p] = row_add<0x121>(v[p]);
}

// Block: four wavefronts on the same columns, each a quarter of the rows.  rowp[column tile][r, P_0 .., Q][i],
// colp[row tile][k][j]: sums of the tile.
template <typename T, int K>
__global__ __launch_bounds__(256, 2) void k_worked_wide_backward(const T *__restrict__ a, const T *__restrict__ b, const T *__restrict__ c,
                                                                 const T *__restrict__ f, const T *__restrict__ df,
                                                                 double *__restrict__ rowp, double *__restrict__ colp, int I, int J,
                                                                 int c_ld, int tile_rows) {
    constexpr int CW = wide_lane_columns(K), TJ = 64 * CW, RP = K + 2;
    __shared__ double rd[kWideMaxRows][K + 1];          // a_i0 .., c_ii
    __shared__ double rows_out[RP][kWideMaxRows];
    __shared__ double cred[4][TJ];
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int i0 = blockIdx.y * tile_rows, jb = blockIdx.x * TJ;
    const int rows = min(tile_rows, I - i0);
    for (int t = tid; t < rows; t += 256) {
        const int i = i0 + t;
#pragma unroll
        for (int k = 0; k < K; ++k) rd[t][k] = (double)a[(size_t)i * K + k];
        rd[t][K] = (double)c[(size_t)i * c_ld + i];
    }
    double bj[CW][K], tc[CW][K];
    int jo[CW];
    bool live[CW];
#pragma unroll
    for (int v = 0; v < CW; ++v) {
        live[v] = jb + v * 64 + lane < J;
        jo[v] = min(jb + v * 64 + lane, J - 1);
#pragma unroll
        for (int k = 0; k < K; ++k) {
            bj[v][k] = (double)b[(size_t)jo[v] * K + k];
            tc[v][k] = 0.0;
        }
    }
    __syncthreads();
    const int per = tile_rows >> 2, first = min(wave * per, rows), last = min(first + per, rows);
    const bool inside = jb + TJ <= J;   // the same for the whole block
    // NR rows from r on: values fv, dv
    auto work = [&](auto nr, int r, const T (&fv)[2][CW], const T (&dv)[2][CW]) {
        constexpr int NR = decltype(nr)::value;
        double part[NR * RP];
#pragma unroll
        for (int p = 0; p < NR * RP; ++p) part[p] = 0.0;
#pragma unroll
        for (int m = 0; m < NR; ++m) {
            double ai[K];
#pragma unroll
            for (int k = 0; k < K; ++k) ai[k] = rd[r + m][k];
            const double ci = rd[r + m][K];
#pragma unroll
            for (int v = 0; v < CW; ++v) {
                if (!inside && !live[v]) continue;   // columns beyond the edge: nothing is added, whatever is in there
                const double g = (double)dv[m][v] * (double)fv[m][v], gc = g * ci;
                double q = 0.0;
#pragma unroll
                for (int k = 0; k < K; ++k) {
                    const double t = ai[k] + bj[v][k];
                    q = fma(t, t, q);
                    part[m * RP + 1 + k] = fma(g, t, part[m * RP + 1 + k]);
                    tc[v][k] = fma(gc, t, tc[v][k]);
                }
                part[m * RP] += g;
                part[m * RP + K + 1] = fma(g, q, part[m * RP + K + 1]);
            }
        }
        wave_totals(part);
        if ((lane & 15) == 0) {
            const int s = lane >> 4, at = s == 1 ? 2 : s == 2 ? 1 : s;
#pragma unroll
            for (int p = 0; p < (NR * RP + 3) / 4; ++p) {
                const int value = 4 * p + at;
                if (value < NR * RP) rows_out[value % RP][r + value / RP] = part[p];
            }
        }
    };
    T fv[2][2][CW], dv[2][2][CW];   // the rows of the next step are loaded before those of the current one are used
    auto load = [&](int set, int r) {
#pragma unroll
        for (int m = 0; m < 2; ++m) {
            const size_t row = (size_t)(i0 + min(r + m, last - 1)) * J;
#pragma unroll
            for (int v = 0; v < CW; ++v) {
                fv[set][m][v] = __builtin_nontemporal_load(f + row + jo[v]);
                dv[set][m][v] = __builtin_nontemporal_load(df + row + jo[v]);
            }
        }
    };
    if (first < last) {
        load(0, first);
        for (int r = first; r < last; r += 4) {
            if (r + 2 < last) load(1, r + 2);
            if (r + 1 < last) work(std::integral_constant<int, 2>{}, r, fv[0], dv[0]);
            else work(std::integral_constant<int, 1>{}, r, fv[0], dv[0]);
            if (r + 2 >= last) break;
            if (r + 4 < last) load(0, r + 4);
            if (r + 3 < last) work(std::integral_constant<int, 2>{}, r + 2, fv[1], dv[1]);
            else work(std::integral_constant<int, 1>{}, r + 2, fv[1], dv[1]);
        }
    }
    // column sums of the four wavefronts, added in a fixed order
#pragma unroll
    for (int k = 0; k < K; ++k) {
        __syncthreads();
#pragma unroll
        for (int v = 0; v < CW; ++v) cred[wave][v * 64 + lane] = tc[v][k];
        __syncthreads();
        for (int col = tid; col < TJ; col += 256)
            if (jb + col < J)
                colp[((size_t)blockIdx.y * K + k) * J + jb + col] = (cred[0][col] + cred[1][col]) + (cred[2][col] + cred[3][col]);
    }
    for (int t = tid; t < rows; t += 256)
#pragma unroll
        for (int p = 0; p < RP; ++p) rowp[((size_t)blockIdx.x * RP + p) * I + i0 + t] = rows_out[p][t];
}

// Finishing pass, three block roles with 64 outputs per block; the four wavefronts split the tiles' sums and are added in a
// fixed order: rows (da, diagonal of dc), columns (db), dd (masks and window from the plan of d).
template <typename T, int K>
__global__ __launch_bounds__(256) void k_worked_wide_finish(const FlatFeas feas, const FlatLevel win, int iy, int iz, const T *__restrict__ c,
                                                            const T *__restrict__ d, const double *__restrict__ rowp, int n_jt,
                                                            const double *__restrict__ colp, int n_it, T *__restrict__ da,
                                                            T *__restrict__ db, T *__restrict__ dc, T *__restrict__ dd, int I, int J,
                                                            int c_ld, int n_d, int blocks_rows, int blocks_cols, int cols, int blocks_dd, int n_c) {
    constexpr int RP = K + 2;
    __shared__ double red[2][RP][64];
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    int blk = blockIdx.x;
    if (blk >= blocks_rows + blocks_cols + blocks_dd) {
        // dc is zero but for the first I elements of its diagonal, which the row blocks write
        zeros_off_diagonal(dc, (unsigned)n_c, (unsigned)c_ld + 1u, (unsigned)I, (unsigned)(blk - blocks_rows - blocks_cols - blocks_dd));
        return;
    }
    if (blk < blocks_rows) {
        const int i = blk * 64 + lane;
        double acc[RP] = {};
        const double ci = (double)c[(size_t)min(i, I - 1) * c_ld + min(i, I - 1)];
        if (i < I) {
            // the loads of U tiles go out together: one after the other, the chain of them is longer than the pass over df and f
            constexpr int U = K <= 4 ? 4 : 2;
            int jt = wave;
            for (; jt + 4 * (U - 1) < n_jt; jt += 4 * U) {
                double v[U][RP];
#pragma unroll
                for (int u = 0; u < U; ++u)
#pragma unroll
                    for (int p = 0; p < RP; ++p) v[u][p] = rowp[((size_t)(jt + 4 * u) * RP + p) * I + i];
#pragma unroll
                for (int u = 0; u < U; ++u)
#pragma unroll
                    for (int p = 0; p < RP; ++p) acc[p] += v[u][p];
            }
            for (; jt < n_jt; jt += 4)
#pragma unroll
                for (int p = 0; p < RP; ++p) acc[p] += rowp[((size_t)jt * RP + p) * I + i];
        }
        add_wavefronts(acc, red, wave, lane);
        if (wave != 0 || i >= I) return;
        if (da)
#pragma unroll
            for (int k = 0; k < K; ++k) da[(size_t)i * K + k] = (T)(-2.0 * ci * acc[1 + k]);
        if (dc) dc[(size_t)i * c_ld + i] = (T)-acc[K + 1];
        return;
    }
    blk -= blocks_rows;
    if (blk < blocks_cols) {
        // `cols` neighbouring columns, 256 / cols threads to each: a column is one sum per tile of rows, however few columns there are
        const int j = blk * cols + lane % cols, parts = 256 / cols;
        double acc[K] = {};
        if (j < J && db) {
            constexpr int U = K <= 4 ? 8 : 4;   // as above
            int it = (int)threadIdx.x / cols;
            for (; it + parts * (U - 1) < n_it; it += parts * U) {
                double v[U][K];
#pragma unroll
                for (int u = 0; u < U; ++u)
#pragma unroll
                    for (int k = 0; k < K; ++k) v[u][k] = colp[((size_t)(it + parts * u) * K + k) * J + j];
#pragma unroll
                for (int u = 0; u < U; ++u)
#pragma unroll
                    for (int k = 0; k < K; ++k) acc[k] += v[u][k];
            }
            for (; it < n_it; it += parts)
#pragma unroll
                for (int k = 0; k < K; ++k) acc[k] += colp[((size_t)it * K + k) * J + j];
        }
        for (int m = cols; m < 64; m <<= 1)   // the same for the whole workgroup
#pragma unroll
            for (int k = 0; k < K; ++k) acc[k] += __shfl_xor(acc[k], m, 64);
        add_wavefronts(acc, red, wave, lane);
        if (wave != 0 || lane >= cols || j >= J || !db) return;
#pragma unroll
        for (int k = 0; k < K; ++k) db[(size_t)j * K + k] = (T)(-2.0 * acc[k]);
        return;
    }
    blk -= blocks_cols;
    const int m = blk * 64 + lane;
    double s[1] = {0.0};
    bool nonzero = false;
    if (m < n_d && dd) {
        const int32_t y[3] = {m, 0, 0};   // the transformed index is the gradient index (checked on the host)
        if (flat_feasible(feas, y)) {
            nonzero = true;
            int32_t lo, hi;
            flat_bounds(win, y, lo, hi);
            // the loads of a window go out together
            constexpr int U = K < 8 ? K : 8;
            for (int jt = wave; jt < n_jt; jt += 4)
                for (int32_t w0 = lo; w0 <= hi; w0 += U) {
                    double v[U];
#pragma unroll
                    for (int u = 0; u < U; ++u) v[u] = rowp[(size_t)jt * RP * I + iy * y[0] + iz * min(w0 + u, hi)];
#pragma unroll
                    for (int u = 0; u < U; ++u) s[0] += w0 + u <= hi ? v[u] : 0.0;
                }
        }
    }
    add_wavefronts(s, red, wave, lane);
    if (wave != 0 || m >= n_d || !dd) return;
    T out = T(0);
    if (nonzero) {
        const double dm = (double)d[m];
        out = (T)(-3.0 * dm * dm * s[0]);
    }
    dd[m] = out;
}

template <typename T, int K>
static int fwd_k(const tad_plan &pl, const void *const *args, void *f, hipStream_t s) {
    const int I = (int)pl.fast.I, J = (int)pl.fast.J;
    const dim3 grid((J + WIDE_FWD_COLS - 1) / WIDE_FWD_COLS, (I + WIDE_FWD_ROWS - 1) / WIDE_FWD_ROWS);
    TAD_LAUNCH("k_worked_wide_forward", (k_worked_wide_forward<T, K>), grid, dim3(256), 0, s, (const T *)args[0], (const T *)args[1],
               (const T *)args[2], (const T *)args[3], (T *)f, I, J, (int)pl.fast.c_ld);
    return hipGetLastError() == hipSuccess ? TAD_OK : TAD_EDEVICE;
}

template <typename T, int K>
static int bwd_k(const tad_plan &pl, const void *const *args, const void *f, const void *df, void *const *dx, void *ws, hipStream_t s) {
    const int I = (int)pl.fast.I, J = (int)pl.fast.J, c_ld = (int)pl.fast.c_ld, n_d = (int)pl.arg_count[3];
    const WideGeom g = worked_wide_geom(I, J, K);
    double *const rowp = static_cast<double *>(ws);
    double *const colp = reinterpret_cast<double *>(static_cast<char *>(ws) + g.col_offset);
    T *const dc = (T *)dx[2];
    TAD_LAUNCH("k_worked_wide_backward", (k_worked_wide_backward<T, K>), dim3(g.n_jt, g.n_it), dim3(256), 0, s, (const T *)args[0],
               (const T *)args[1], (const T *)args[2], (const T *)f, (const T *)df, rowp, colp, I, J, c_ld, g.tile_rows);
    if (hipGetLastError() != hipSuccess) return TAD_EDEVICE;
    // Columns of a workgroup that finishes them: as few as leave a thread about a dozen sums, whose loads go out four or eight at a time.  Gradients
    // with 64 columns always / by this rule, I x J x K: 7663 x 60 x 6 (479 tiles of rows) 54 / 45 us, without dc 33 / 14; 5000 x 120 x 3 32 / 22.5, 333 x 6000 x 8 31 / 22,
    // 4000 x 500 x 7 35 / 28, 2000 x 2000 x 4 20.0 / 17.7; 64 bits 1024 x 40 x 16 22.4 / 17.9.
    const int cols = g.n_it <= 48 ? 64 : g.n_it <= 192 ? 16 : 4;
    const int br = (I + 63) / 64, bc = dx[1] ? (J + cols - 1) / cols : 0, bd = (n_d + 63) / 64;
    // the zeros of dc in the same launch (behind the read pass: a write burst right before it slows the reads down)
    const int n_c = (int)pl.arg_count[2], bz = dc ? (int)(((long long)n_c * (int)sizeof(T) + kZeroBytes - 1) / kZeroBytes) : 0;
    TAD_LAUNCH("k_worked_wide_finish", (k_worked_wide_finish<T, K>), dim3(br + bc + bd + bz), dim3(256), 0, s, pl.fast.feas, pl.fast.flat[0],
               pl.fast.dd_iy, pl.fast.dd_iz, (const T *)args[2], (const T *)args[3], (const double *)rowp, g.n_jt, (const double *)colp,
               g.n_it, (T *)dx[0], (T *)dx[1], dc, (T *)dx[3], I, J, c_ld, n_d, br, bc, cols, bd, n_c);
    return hipGetLastError() == hipSuccess ? TAD_OK : TAD_EDEVICE;
}

#define TAD_K(fn, k, ...) case k: return pl.dtype == TAD_F64 ? fn<double, k>(__VA_ARGS__) : fn<float, k>(__VA_ARGS__);
#define TAD_K_SWITCH(fn, ...)                                                                                                  \
    switch (pl.fast.K) {                                                                                                       \
        TAD_K(fn, 1, __VA_ARGS__) TAD_K(fn, 2, __VA_ARGS__) TAD_K(fn, 3, __VA_ARGS__) TAD_K(fn, 4, __VA_ARGS__)                  \
        TAD_K(fn, 5, __VA_ARGS__) TAD_K(fn, 6, __VA_ARGS__) TAD_K(fn, 7, __VA_ARGS__) TAD_K(fn, 8, __VA_ARGS__)                  \
        TAD_K(fn, 9, __VA_ARGS__) TAD_K(fn, 10, __VA_ARGS__) TAD_K(fn, 11, __VA_ARGS__) TAD_K(fn, 12, __VA_ARGS__)               \
        TAD_K(fn, 13, __VA_ARGS__) TAD_K(fn, 14, __VA_ARGS__) TAD_K(fn, 15, __VA_ARGS__) TAD_K(fn, 16, __VA_ARGS__)              \
    default: return TAD_EUNSUPPORTED;                                                                                          \
    }

int worked_wide_forward(const tad_plan &pl, const void *const *args, void *f, hipStream_t s) {
    TAD_K_SWITCH(fwd_k, pl, args, f, s)
}

int worked_wide_backward(const tad_plan &pl, const void *const *args, const void *f, const void *df, void *const *dx, void *ws,
                         hipStream_t s) {
    TAD_K_SWITCH(bwd_k, pl, args, f, df, dx, ws, s)
}

}  // namespace tad
