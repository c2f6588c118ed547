// Sums of products that separate over the function indices,
//
//     s_mn = sum_k A(m, k) B(k, n),
//
// where m stands for the leading function indices, n for the trailing ones and k for the summation indices: what an
// expression with a product inside the sum is when one factor ignores n and the other one m.  The sum and its two
// derived gradients  dA(m, k) = sum_n g_mn B(k, n)  and  dB(k, n) = sum_m A(m, k) g_mn  are dense products then.
#pragma once
#include <cstddef>
#include <cstdint>

struct tad_plan;

namespace tad {

// One dense product C[r][c] = sum_q A(r, q) B(q, c) with 64-bit accumulation.  A(r, q) = a[r * ar + q * aq],
// B(q, c) = b[q * bq + c * bc] (element strides of any order), C row-major.
struct ProductDesc {
    int R = 0, C = 0, Q = 0;
    int64_t ar = 0, aq = 0, bq = 0, bc = 0;
    bool a64 = false, b64 = false;   // 64-bit operands
    int rows = 1;      // an output tile has 16 rows x kProductCols results
    bool flip = false; // ... of the product with its operands exchanged, whose results are stored transposed
    int pieces = 1;    // pieces of q computed by separate workgroups (few output tiles, long sum)
    int chunk = 0;     // values of q per piece (pieces > 1)
    int outer = 0;     // results per pass of the interpreter where a program is applied to them (0: none)
    bool scaled = false;   // results that are multiplied where they are stored, if the sum is not in pieces
    int pair_rows = 0; // `rows` of one launch for this product and the other gradient (0: a launch each)
    bool pair_flip = false;
};

// The products of a sum and of its gradients, with the workspace that their partial sums make it (lean: see tad_plan::ws_lean).
struct ProductSet {
    ProductDesc forward, grad[2];
    size_t ws_bytes = 0;
};

// One factor of the product.
struct ProductSide {
    int operand = -1;          // the tensor that is the factor
    int64_t sm = 0, sk = 0;    // element strides along m (first factor) or n (second one) and along k
    bool grad = false;         // its gradient is a dense product that fills the tensor in its own memory order
    bool k_major = false;      // ... whose rows run over k
};

struct ProductPlan {
    bool on = false;
    int64_t M = 0, N = 0, K = 0;
    bool forward_on = false;   // the sum itself is a dense product (else the gradients alone)
    ProductSide side[2];
    ProductSet set, lean;      // (ws_bytes: partial sums of shared tiles, behind the workspace of the other kernels)
    bool lean_on = false;
    size_t ws_offset = 0;
};

// Extents from which the dense products are used, and the least number of terms of the whole sum: below that the
// general kernels take a few microseconds as well.
constexpr int64_t kProductExtent = 16, kProductSum = 8;

// Offset of one tensor along a group of extended indices as a single stride: the group's indices, the last one
// fastest, count through 0 .. n - 1 and the offset is stride * that number.  False if it is not linear in it.
bool product_group_stride(const int64_t *off, const int64_t *extent, int count, int64_t &stride);
// The kernels address the elements of a stage (up to 112 rows, 32 values of q) with 32-bit byte offsets from
// a 64-bit base.
bool product_addressable(const ProductDesc &d);
// Columns of an output tile.
constexpr int kProductCols = 64;
// Values of q per stage: two stages of the tallest tile take 96 KB of LDS, and the low ones leave room for a second and a third
// workgroup on a compute unit, which covers the beginning and end of the other one (stages of 64 there: both gradients of
// 512 x 1024 x 768 40.8 us instead of 36.2, a product that is one round of tiles the same).
constexpr int kProductStage = 32;
// Tile and pieces for a product of these extents and operands, with no more than `most` bytes of partial sums.
void product_shape(ProductDesc &d, size_t most);
// Two products that run one after the other: would they be faster in one launch (pair_rows of both)?
void product_pair(ProductDesc &x, ProductDesc &y);
// The product with its operands exchanged: the transposed result.
ProductDesc product_turned(const ProductDesc &d);
// Bytes of partial sums a product needs (0: none).
size_t product_partial_bytes(const ProductDesc &d);
// Is a forward sum of K terms for M x N results so short that a thread per result of the general kernels is the faster one?
bool product_sum_short(bool f64, int64_t M, int64_t N, int64_t K);
// Does the expression separate, and which of its products run as dense products (plan.prod)?
void match_product(tad_plan &plan);

}  // namespace tad
