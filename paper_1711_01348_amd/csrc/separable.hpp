// Sums whose terms are products of two functions,
//
//     f_mn = outer( s_mn, operands at (m, n) ),   s_mn = sum_k A(m, k) B(k, n),
//
// where m stands for the leading function indices, n for the trailing ones and k for the summation indices, and A and B
// are what the factors of the inner function that ignore n and m multiply to.  A and B are evaluated once per pair of
// indices instead of once per term, the sum is a dense product, and so are the derivatives of the factors,
//
//     dA(m, k) = sum_n g_mn B(k, n),   dB(k, n) = sum_m A(m, k) g_mn,   g = df * d outer / d s;
//
// the gradient of an operand of A is the gather of an expression over (m, k) without a sum of its own:
// dx_beta = sum over the pairs (m, k) that read x_beta of dA(m, k) * (dA / dx)(operands at (m, k)).
#pragma once
#include <cstddef>
#include <cstdint>
#include <memory>
#include <vector>

#include "product.hpp"
#include "program.hpp"

struct tad_plan;

namespace tad {

struct SepSide {
    int operand = -1;            // the tensor that is the factor; -1: a function of operands, evaluated into the workspace
    bool fills = false;          // ... whose elements are exactly the pairs of indices: its gradient is the product itself
    int64_t X = 0;               // values of the side's function index
    int64_t sm = 0, sk = 0;      // element strides of the factor along the function index and along k
    bool k_major = false;        // rows of the factor's derivative run over k
    // the factor as an expression over its pairs of indices, in the order of its derivative's elements; null if the tensor
    // is the factor and its gradient is the product (or not wanted)
    std::shared_ptr<tad_plan> sub;
    std::vector<int> operands;   // operand of sub -> operand of the expression
    // a factor that is a function of operands: its value and the partial derivatives of the operands with a gradient in one program, if
    // that has a register form; joint_place[0]: which of its results is the value, [1 + p]: the derivative by operand p (-1: none)
    bool joint_on = false;
    DevProg joint;
    int joint_place[1 + TAD_MAX_ARGS];
    std::vector<char> aligned;   // ... every pair of indices reads an element of its own, numbered alike
    // workspace, all in 64 bits
    size_t value_offset = 0;     // the evaluated factor
    size_t d_offset = 0;         // its derivative
    std::vector<size_t> h_offset;   // per operand: terms of a gradient that several pairs of indices add to (in a large
                                    // workspace one of them in the place of the evaluated factor)
};

struct SepPlan {
    bool on = false;
    int64_t M = 0, N = 0, K = 0;
    ProductSet set, lean;        // the sums, and the derivatives of the factors
    bool lean_on = false;
    bool forward_on = false;     // the forward pass too runs on the dense product (else the gradients alone)
    SepSide side[2];
    ProgramBody prog;            // outer function and its derivatives
    bool identity = false;       // the outer function is the sum
    bool term_is_g[TAD_MAX_ARGS] = {};   // d outer / d operand and d outer / d sum are the same program
    // offsets of the outer function's operands along the two function indices, if these are single strides
    bool outer_linear = true;
    int64_t outer_r[TAD_MAX_ARGS] = {}, outer_c[TAD_MAX_ARGS] = {};
    // workspace
    size_t s_offset = 0;         // sums
    size_t g_offset = 0;         // g = df * d outer / d s
    size_t h_offset = 0;         // 64-bit terms of an operand of the outer function
    size_t part_offset = 0;      // partial sums of the products and of the gathers
};

// Workspace the dense form may ask for beyond four times the operands and f.  A factor's pairs of indices can be any number of
// times the elements it is made of (x_{i+k} at 40000 x 40000 pairs: 13 GB per matrix of pairs from 0.3 MB); where they are the
// elements, the matrices of either side (values, derivatives) take four times the operand.  2^30 bytes are 0.4 % of the
// memory; 262144 x 64 pairs of x_{i+k} fit.
constexpr double kSeparableWorkspace = 1073741824.0;

// Does the inner function separate, is the sum large enough for the dense form and its workspace in proportion (plan.sep)?
void match_separable(tad_plan &plan);

}  // namespace tad
