// Declarations shared by the kernel translation units and the C ABI front end.
#pragma once
#include <hip/hip_runtime.h>

#include "plan.hpp"

namespace tad {

struct ArgPtrs {
    const void *p[kMaxArgs];
};

int generic_forward(const tad_plan &pl, const void *const *args, void *f, void *ws, hipStream_t s);
int generic_backward(const tad_plan &pl, const void *const *args, const void *f, const void *df,
                     void *const *dx, void *ws, hipStream_t s);

int worked_forward(const tad_plan &pl, const void *const *args, void *f, hipStream_t s);
int worked_backward(const tad_plan &pl, const void *const *args, const void *f, const void *df,
                    void *const *dx, void *ws, hipStream_t s);

// worked expression in either precision, rows of any length, K <= 16: sums in 64 bits
int worked_wide_forward(const tad_plan &pl, const void *const *args, void *f, hipStream_t s);
int worked_wide_backward(const tad_plan &pl, const void *const *args, const void *f, const void *df, void *const *dx, void *ws, hipStream_t s);

int mfma_forward(const tad_plan &pl, const void *const *args, void *f, void *ws, bool full, hipStream_t s);
int mfma_backward(const tad_plan &pl, const void *const *args, const void *f, const void *df, void *const *dx,
                  void *ws, bool full, hipStream_t s);
int pattern_forward(const tad_plan &pl, const void *const *args, void *f, hipStream_t s);
int pattern_backward(const tad_plan &pl, const void *const *args, const void *df, void *const *dx, void *ws,
                     hipStream_t s);

// row reduce and antidiagonal patterns in either precision, rows of any length: sums in 64 bits
int pattern_wide_forward(const tad_plan &pl, const void *const *args, void *f, hipStream_t s);
int pattern_wide_backward(const tad_plan &pl, const void *const *args, const void *df, void *const *dx, void *ws, hipStream_t s);

// sums over a moving window
int window_forward(const tad_plan &pl, const void *const *args, void *f, hipStream_t s);
int window_backward(const tad_plan &pl, const void *const *args, const void *df, void *const *dx, void *ws, hipStream_t s);

int strided_forward(const tad_plan &pl, const void *const *args, void *f, hipStream_t s);
int strided_backward(const tad_plan &pl, const void *const *args, const void *f, const void *df,
                     void *const *dx, void *ws, hipStream_t s);

int contract_forward(const tad_plan &pl, const void *const *args, void *f, void *ws, bool full, hipStream_t s);
int contract_backward(const tad_plan &pl, const void *const *args, const void *df, void *const *dx, void *ws, bool full, hipStream_t s);
// one of their products on the bf16 matrix cores; *range: what the 32-bit kernel looks at to see whether it is still to be done
int split_product(const GemmDesc &g, const float *a, const float *b, float *c, void *ws, const int **range, hipStream_t s);

// Sums of products as dense products.  product_backward writes the gradients it is responsible for and clears their
// entries of dx; the rest is left to the family's kernels.
int product_forward(const tad_plan &pl, const ProductSet &set, const void *const *args, void *f, void *ws, hipStream_t s);
int product_backward(const tad_plan &pl, const ProductSet &set, const void *const *args, const void *df, void **dx, void *ws, hipStream_t s);

// One product and its operands; a64, b64, c64: 64-bit elements; turned: the result is stored [c][r].
struct ProductDesc;
struct ProductJob {
    const ProductDesc *desc;
    const void *a;
    bool a64;
    const void *b;
    bool b64;
    void *c;
    bool c64;
    bool turned = false;
    // not 0: instead of the result v itself, to[n] = v * by[n] for n < scaled, element by element (a product of a single piece)
    int scaled = 0;
    const double *by[2] = {};
    void *to[2] = {};
    bool to64[2] = {};
};
struct ProductOuter;
// Column sums out[c] = sum_r g[r][c] beside a product (64 bits on the way; wide: 64-bit elements)
struct ProductColumns {
    const void *g;
    void *out;
    int R, C;
    bool wide;
};
// ws: partial sums of shared tiles; columns: null, or sums that the first launch does as well
int product_run(const ProductJob &j, void *ws, hipStream_t s, const ProductColumns *columns = nullptr);
int product_run_two(const ProductJob &x, const ProductJob &y, void *ws, hipStream_t s, const ProductColumns *columns = nullptr);
// can the results of this product, run alone or as one of two, be scaled?
bool product_scales(const ProductDesc &d, bool one_of_two);
// the product's results through a program in register form (only where product_outer_fits)
bool product_outer_fits(const ProductDesc &d);
int product_run_outer(const ProductJob &j, const ProductOuter &o, hipStream_t s);

// sums of products of two functions (separable.hpp)
int separable_forward(const tad_plan &pl, const ProductSet &set, const void *const *args, void *f, void *ws, hipStream_t s);
int separable_backward(const tad_plan &pl, const ProductSet &set, const void *const *args, const void *f, const void *df, void *const *dx, void *ws, hipStream_t s);

int program_forward(const tad_plan &pl, const void *const *args, void *f, void *ws, hipStream_t s);
// out = prog(s, operands), times df if that is given, for every function element; pb: the body `prog` belongs to
int program_outer(const tad_plan &pl, const ProgramBody &pb, const DevProg &prog, const void *const *args, const void *s, const void *df,
                  void *out, hipStream_t stream);
// Can the derivatives of the outer function that these gradients need be written in f?
bool outer_in_f(const tad_plan &pl, const ProgramBody &pb, void *const *dx);
int program_backward(const tad_plan &pl, const void *const *args, const void *f, const void *df, void *const *dx, void *ws,
                     hipStream_t s);

}  // namespace tad
